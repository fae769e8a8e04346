// Isolated k-hop neighbour sampling inside one partition (mini-batch mode), on the GPU.
//
// Per destination node v with d local in-edges: all of them if d <= fanout, otherwise a uniformly
// random fanout-subset of the positions 0..d-1 of its CSR row, grown one element at a time:
//   for t = 0..fanout-1:  top = d - fanout + t,  r = floor(u_t * (top + 1) / 2^64),
//                         the subset gains r if it does not hold r yet, else top;
//   u_t = M(M(M(M(M(sampler_seed) ^ batch_id) ^ layer) ^ global_id(v)) ^ t),
//   M(x) = SplitMix64 finaliser of x + 0x9E3779B97F4A7C15.
// Every subset is equally likely; the draws depend only on (seed, batch, layer, node, t), so the
// selection is independent of scheduling and bit-reproducible; and a row costs O(fanout) whatever
// its length (the hub rows of a skewed graph hold 10^5..10^6 edges).  The chosen edges are kept
// in position order.
//
// Layers are built from the seeds inwards.  Above the input layer, new source nodes are
// found with a node bitmap and a prefix sum over its words (ascending local id), sources are
// relabelled to block-local indices and the block is also stored transposed for the backward pass.  The input layer keeps
// partition-local ids: they index the feature matrix directly, so no feature rows are copied.
//
// Every launch costs the device about 3.6 us, whatever its stream (a captured step of 70 launches replayed alone 450 us, on two streams
// 508 for two, on four 1030 for four), so the work is cut into as few as its dependences allow: a layer is (1) the counts of its rows with
// their prefix sum, beside the relabelling of the layer before, (2) the choice of its edges, which marks the nodes they
// reach, (3) the prefix sum over the marks' words, which numbers them.  The transposed blocks of all layers take three more together.
// The prefix sums look back over the workgroups before theirs instead of taking launches of their own.  (23 launches
// on the caller's stream and 20 beside it became 9 and 3: a step of 1024 seeds, fanouts 15, 10, 5 on a 7e6-node store 415 -> 391 us, an epoch of
// 24 steps on four streams 6.2 -> 5.2 ms.)
//
// The host never learns a block's sizes.  They depend on the draws, so they exist on the device only
// (`sizes`, four numbers per layer); every launch is sized by the upper bounds that follow from the seeds
// and fanouts, reads the real sizes from device memory and leaves the slots between the two in a state
// that is harmless to read (empty rows, sentinel keys).  A step is therefore queued without waiting for
// the device, and can be captured in a graph.
#include "common.h"

#include <algorithm>
#include <vector>

namespace grp {

constexpr int SAMPLE_MAX_FANOUT = 64;         // one lane of a wavefront per chosen edge
// A layer's sizes on the device: destinations, sources (destinations first, then the newly reached nodes),
// edges, newly reached nodes.
enum { SZ_DST = 0, SZ_SRC = 1, SZ_NNZ = 2, SZ_NEW = 3, SZ_PER_LAYER = 4 };

// ---- prefix sums across the workgroups of one launch (the decoupled look-back of Merrill and Garland, "Single-pass parallel prefix scan
// with decoupled look-back", 2016).  A workgroup posts the sum of its part, then adds up what those before it have
// posted, 64 at a time, until it meets one that has posted its whole prefix, and posts its own.  Flag and value share a 64-bit word,
// cleared before the launch.
// Every wait ends: workgroups wait for lower-numbered ones of their launch only, which each XCD starts first, so a launch on its own
// cannot stall.  Launches side by side could, if those of others filled an XCD while they wait for parts that have no place there.  So a
// launch, whatever its layers and merged steps, has at most WAITING workgroups that wait, 48 on an XCD; an XCD holds at
// least 192 of them (six a CU: these kernels take at most 80 vector registers and next to no LDS), so that three of the four launches that four
// hardware queues run at a time leave room for the fourth.
constexpr int PARTS = 128;               // of one prefix sum
constexpr int WAITING = 384;             // of all prefix sums of a launch (256: an epoch in four merged lanes 1 % slower)
constexpr unsigned long long POSTED_SUM = 1ull << 62, POSTED_PREFIX = 2ull << 62, POSTED_VALUE = (1ull << 62) - 1;

// The sum before part `part`, for the lanes of one wavefront; `own`: this part's sum.
__device__ __forceinline__ unsigned long long look_back(unsigned long long* __restrict__ posted, int part, unsigned long long own) {
    const int lane = threadIdx.x & 63;
    auto post = [&](unsigned long long v) {
        if (lane == 0) __hip_atomic_store(&posted[part], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    post((part == 0 ? POSTED_PREFIX : POSTED_SUM) | own);
    unsigned long long before = 0;
    for (int at = part - 1; at >= 0; at -= 64) {
        unsigned long long v = POSTED_PREFIX;
        do {
            if (at - lane >= 0) v = __hip_atomic_load(&posted[at - lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } while (__ballot((v >> 62) == 0));
        const unsigned long long whole = __ballot((v >> 62) == 2);       // (lanes past part 0 count as whole, with nothing)
        const int last = whole ? __ffsll(whole) - 1 : 63;
        unsigned long long sum = lane <= last ? v & POSTED_VALUE : 0ull;
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        before += sum;
        if (whole) break;
    }
    if (part > 0) post(POSTED_PREFIX | (before + own));
    return before;
}

constexpr int CS_THREADS = 256;
constexpr int CS_PER = 4;
constexpr int CS_ROUND = CS_THREADS * CS_PER;                // rows of a part, taken that many at a time
// Rounds of a part and number of parts (workgroups) for `items` rows; sums: that share the launch (merged steps times the layers of one: 8
// times 15 are 120, fewer than WAITING).
struct ScanPlan { int rounds, parts; };
ScanPlan look_back_plan(int64_t items, int64_t round, int sums) {
    const int64_t parts = std::max(1, std::min(PARTS, WAITING / sums)), rounds = cdiv(items, round * parts);
    return {(int)rounds, (int)cdiv(items, round * rounds)};
}
static int steps_of_launch() { return g_recorder ? g_recorder->steps : 1; }

// Rows of a layer, counted: the number of edges row i keeps (CSR pointer ptr[0 .. bound], the rows between the real count and the bound
// empty), 1 / max(that, 1) and, above the input layer, its place at the head of the block's source list.  The seeds' layer reads
// the caller's list: seeds outside [0, n) are counted (`bad`; the step's statistics report it) and replaced by node 0 in the
// copy the sampler works on, so that no kernel reads outside the partition.
struct CountJob {
    const int64_t* rowptr;
    const int32_t* dst_nodes;
    const int32_t* raw_seeds;            // the seeds' layer only: the caller's list (dst_nodes receives the checked copy)
    int64_t n, n_seeds;
    int64_t* sizes;                      // of this layer
    int64_t bound;
    int fanout, rounds, parts;
    unsigned long long* posted;
    int64_t* ptr;
    int32_t* cnt32;
    float* inv;
    int32_t* mark;                       // the seeds' layer only (and above the input layer)
    int32_t* src_nodes;                  // above the input layer
    unsigned long long* bad;
};
// idx_blk[e] = block-local index of the source of edge e; arrival[e] = how many edges of that source came before it, in any order.
struct RelabelJob {
    const int64_t* ptr;                  // null: nothing to relabel
    const int64_t* sizes;
    int64_t dst_bound;
    const int32_t* idx_local;
    const int32_t* mark;
    int32_t* idx_blk;
    int32_t* arrival;
    uint32_t* count_t;                   // [sources] edges of each (cleared)
};

__device__ __forceinline__ void count_rows_kernel_body(unsigned gx, CountJob c, RelabelJob r) {
    __shared__ unsigned long long wave_sum[CS_THREADS / 64];
    __shared__ unsigned long long before_s;
    const int tid = threadIdx.x, lane = tid & 63;
    if ((int)blockIdx.x >= c.parts) {                        // relabelling: a wavefront per destination row
        const int64_t i = (int64_t)((int)blockIdx.x - c.parts) * 4 + tid / 64;
        if (i >= r.sizes[SZ_DST]) return;
        for (int64_t e = r.ptr[i] + lane; e < r.ptr[i + 1]; e += 64) {
            const int32_t s = r.mark[r.idx_local[e]] - 1;
            r.idx_blk[e] = s;
            r.arrival[e] = (int32_t)atomicAdd(&r.count_t[s], 1u);
        }
        return;
    }
    const int part = (int)blockIdx.x;
    const int64_t n_dst = c.raw_seeds ? c.n_seeds : c.sizes[SZ_DST];
    if (c.raw_seeds && part == 0 && tid == 0) c.sizes[SZ_DST] = n_dst;
    const int64_t part0 = (int64_t)part * c.rounds * CS_ROUND;
    int32_t cnt[CS_PER];
    auto count = [&](int round, bool first) {                // the counts of one round, in cnt
        unsigned long long sum = 0;
        int32_t v[CS_PER];
#pragma unroll
        for (int q = 0; q < CS_PER; ++q) {
            const int64_t i = part0 + (int64_t)round * CS_ROUND + CS_PER * tid + q;
            v[q] = 0;
            if (i < n_dst) {
                if (c.raw_seeds) {
                    v[q] = c.raw_seeds[i];
                    const bool ok = v[q] >= 0 && (int64_t)v[q] < c.n;
                    if (!ok) v[q] = 0;
                    if (first && !ok) atomicAdd(c.bad, 1ull);
                    if (first) const_cast<int32_t*>(c.dst_nodes)[i] = v[q];
                } else {
                    v[q] = c.dst_nodes[i];
                }
            }
        }
#pragma unroll
        for (int q = 0; q < CS_PER; ++q) {
            const int64_t i = part0 + (int64_t)round * CS_ROUND + CS_PER * tid + q;
            cnt[q] = 0;
            if (i < n_dst) {
                const int64_t d = c.rowptr[v[q] + 1] - c.rowptr[v[q]];
                cnt[q] = (int32_t)(d < c.fanout ? d : c.fanout);
                if (first) {
                    if (c.cnt32) c.cnt32[i] = cnt[q];
                    c.inv[i] = 1.0f / (float)(cnt[q] > 1 ? cnt[q] : 1);
                    // (a lower layer's destinations are the sources of the layer above: the map holds the same places already)
                    if (c.mark) c.mark[v[q]] = (int32_t)i + 1;
                    if (c.src_nodes) c.src_nodes[i] = v[q];
                }
            }
            sum += (unsigned long long)cnt[q];
        }
        return sum;
    };
    unsigned long long mine = 0, total;
    for (int round = 0; round < c.rounds; ++round) mine += count(round, true);
    (void)block_scan<CS_THREADS / 64>(mine, wave_sum, total);
    if (tid < 64) {
        const unsigned long long b = look_back(c.posted, part, total);
        if (lane == 0) before_s = b;
    }
    __syncthreads();
    unsigned long long at0 = before_s;
    for (int round = 0; round < c.rounds; ++round) {
        const unsigned long long sum = c.rounds == 1 ? mine : count(round, false);
        unsigned long long at = at0 + block_scan<CS_THREADS / 64>(sum, wave_sum, total);
        at0 += total;
#pragma unroll
        for (int q = 0; q < CS_PER; ++q) {
            const int64_t i = part0 + (int64_t)round * CS_ROUND + CS_PER * tid + q;
            if (i <= c.bound) c.ptr[i] = (int64_t)at;
            at += (unsigned long long)cnt[q];
        }
    }
}
__global__ __launch_bounds__(CS_THREADS) void count_rows_kernel(CountJob c, RelabelJob r) {
    count_rows_kernel_body(gridDim.x, c, r);
}
struct count_rows_kernel_op {
    static constexpr int THREADS = CS_THREADS, WGS = 1;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { count_rows_kernel_body(gx, a...); }
};

// One wavefront per destination row.  Lane t computes draw t; the subset is grown in `fanout`
// wave-uniform steps with lane t keeping the t-th element; each lane then finds the rank of its
// element (they are distinct) and writes the edge to that output slot.
// Above the input layer the sources that the block does not have yet are marked in a bitmap over the partition's nodes (one bit each):
// the words' population counts are prefix-summed and every non-empty word then numbers its own nodes, which
// yields them in ascending local id while touching n / 8 bytes instead of per-node flag arrays.
// mark[u] - 1 is the place of a node that the block has; for any other node it is whatever the memory held, so a place counts
// only if it exists and names the node.  (Clearing the map first and after each layer cost the step of a 7e6-node store a fill of
// 28 MB and a launch per layer: 10.4 of 450 us for the fill and 2.5 for each of the launches.)
constexpr int SAMPLE_ROWS_PER_WG = 4;
constexpr int SAMPLE_THREADS = 64 * SAMPLE_ROWS_PER_WG;

__device__ __forceinline__ void sample_select_kernel_body(unsigned gx, const int64_t* __restrict__ rowptr,
                                                                                const int32_t* __restrict__ col,
                                                                                const int64_t* __restrict__ l2g,
                                                                                const int32_t* __restrict__ dst_nodes,
                                                                                int64_t* __restrict__ sizes /*of this layer*/,
                                                                                int fanout, uint64_t h0 /*M(sampler_seed)*/,
                                                                                uint64_t batch_id,
                                                                                const uint64_t* __restrict__ batch_id_dev,
                                                                                int layer,
                                                                                const int64_t* __restrict__ out_ptr,
                                                                                int32_t* __restrict__ out_idx,
                                                                                const int32_t* __restrict__ mark,
                                                                                uint32_t* __restrict__ bits /*null: input layer*/) {
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * SAMPLE_ROWS_PER_WG + (threadIdx.x >> 6);
    const int64_t n_dst = sizes[SZ_DST];
    if (blockIdx.x == 0 && threadIdx.x == 0) sizes[SZ_NNZ] = out_ptr[n_dst];      // the block's number of edges
    if (i >= n_dst) return;                              // uniform over the wavefront
    const int64_t v = dst_nodes[i];
    const int64_t b = rowptr[v];
    const int64_t d = rowptr[v + 1] - b;
    const int64_t o = out_ptr[i];
    auto take = [&](int64_t slot, int32_t u) {
        out_idx[slot] = u;
        if (!bits) return;
        const int32_t at = mark[u];
        const bool known = at > 0 && at <= n_dst && dst_nodes[at - 1] == u;
        if (!known) atomicOr(&bits[u >> 5], 1u << (u & 31));
    };
    if (d <= fanout) {
        for (int64_t j = lane; j < d; j += 64) take(o + j, col[b + j]);
        return;
    }
    const uint64_t h2 = mixM(mixM(h0 ^ (batch_id_dev ? *batch_id_dev : batch_id)) ^ (uint64_t)layer);
    const uint64_t h3 = mixM(h2 ^ (uint64_t)l2g[v]);
    const uint64_t my_bits = mixM(h3 ^ (uint64_t)lane);
    int64_t mine = -1;                                   // lane t < fanout: the t-th element of the subset
    for (int t = 0; t < fanout; ++t) {
        const uint64_t u = __shfl(my_bits, t, 64);
        const int64_t top = d - fanout + t;
        int64_t r = (int64_t)__umul64hi(u, (uint64_t)(top + 1));
        if (__ballot(lane < t && mine == r)) r = top;    // r is taken: top cannot be (earlier elements are below it)
        if (lane == t) mine = r;
    }
    int rank = 0;
    for (int t = 0; t < fanout; ++t) rank += __shfl(mine, t, 64) < mine ? 1 : 0;
    if (lane < fanout) take(o + rank, col[b + mine]);
}
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_select_kernel(const int64_t* __restrict__ rowptr,
                                                                                const int32_t* __restrict__ col,
                                                                                const int64_t* __restrict__ l2g,
                                                                                const int32_t* __restrict__ dst_nodes,
                                                                                int64_t* __restrict__ sizes /*of this layer*/,
                                                                                int fanout, uint64_t h0 /*M(sampler_seed)*/,
                                                                                uint64_t batch_id,
                                                                                const uint64_t* __restrict__ batch_id_dev,
                                                                                int layer,
                                                                                const int64_t* __restrict__ out_ptr,
                                                                                int32_t* __restrict__ out_idx,
                                                                                const int32_t* __restrict__ mark,
                                                                                uint32_t* __restrict__ bits /*null: input layer*/) {
    sample_select_kernel_body(gridDim.x, rowptr, col, l2g, dst_nodes, sizes, fanout, h0, batch_id, batch_id_dev, layer, out_ptr, out_idx, mark, bits);
}
struct sample_select_kernel_op {
    static constexpr int THREADS = SAMPLE_THREADS, WGS = 1;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { sample_select_kernel_body(gx, a...); }
};

// The bitmap's words: the new nodes of every word are numbered after the destinations and the new nodes of the words before it.
// Also clears the bitmap for the next layer, completes the layer's sizes and states the next layer's number of destinations (this
// layer's sources).  Parts of `rounds` rounds, a thread WD_PER consecutive words of each.
constexpr int WD_THREADS = 256;
constexpr int WD_PER = 16;
constexpr int WD_ROUND = WD_THREADS * WD_PER;
__device__ __forceinline__ void number_new_kernel_body(unsigned gx, int64_t n_words /*rounded up to WD_PER, the words past the last empty*/, int rounds,
                                                                unsigned long long* __restrict__ posted, uint32_t* __restrict__ bits,
                                                                int64_t* __restrict__ sizes, int64_t* __restrict__ next_n_dst,
                                                                int32_t* __restrict__ mark, int32_t* __restrict__ src_nodes) {
    __shared__ unsigned long long wave_sum[WD_THREADS / 64];
    __shared__ unsigned long long before_s;
    const int tid = threadIdx.x;
    const int64_t n_dst = sizes[SZ_DST];
    const int64_t part0 = (int64_t)blockIdx.x * rounds * WD_ROUND;
    uint4 w[WD_PER / 4];
    auto load = [&](int round) {
        const int64_t i = part0 + (int64_t)round * WD_ROUND + WD_PER * tid;
        unsigned long long sum = 0;
#pragma unroll
        for (int q = 0; q < WD_PER / 4; ++q) {
            w[q] = i < n_words ? reinterpret_cast<const uint4*>(bits + i)[q] : make_uint4(0u, 0u, 0u, 0u);
            sum += (unsigned long long)(__popc(w[q].x) + __popc(w[q].y) + __popc(w[q].z) + __popc(w[q].w));
        }
        return sum;
    };
    unsigned long long mine = 0, total, part_total;
    for (int round = 0; round < rounds; ++round) mine += load(round);
    (void)block_scan<WD_THREADS / 64>(mine, wave_sum, part_total);
    if (tid < 64) {
        const unsigned long long b = look_back(posted, (int)blockIdx.x, part_total);
        if (tid == 0) before_s = b;
    }
    __syncthreads();
    unsigned long long at0 = before_s;
    if (blockIdx.x == gx - 1 && tid == 0) {
        const int64_t n_new = (int64_t)(at0 + part_total);
        sizes[SZ_NEW] = n_new;
        sizes[SZ_SRC] = n_dst + n_new;
        *next_n_dst = n_dst + n_new;
    }
    for (int round = 0; round < rounds; ++round) {
        const unsigned long long sum = rounds == 1 ? mine : load(round);
        unsigned long long at = at0 + block_scan<WD_THREADS / 64>(sum, wave_sum, total);
        at0 += total;
        if (sum == 0) continue;
        const int64_t i = part0 + (int64_t)round * WD_ROUND + WD_PER * tid;
        int32_t p = (int32_t)(n_dst + (int64_t)at);
#pragma unroll
        for (int q = 0; q < WD_PER / 4; ++q) {
            const uint32_t word[4] = {w[q].x, w[q].y, w[q].z, w[q].w};
#pragma unroll
            for (int h = 0; h < 4; ++h)
                for (uint32_t left = word[h]; left; left &= left - 1) {
                    const int32_t u = (int32_t)((i + 4 * q + h) * 32) + (__ffs(left) - 1);
                    src_nodes[p] = u;
                    mark[u] = ++p;
                }
            reinterpret_cast<uint4*>(bits + i)[q] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
}
__global__ __launch_bounds__(WD_THREADS) void number_new_kernel(int64_t n_words /*rounded up to WD_PER, the words past the last empty*/, int rounds,
                                                                unsigned long long* __restrict__ posted, uint32_t* __restrict__ bits,
                                                                int64_t* __restrict__ sizes, int64_t* __restrict__ next_n_dst,
                                                                int32_t* __restrict__ mark, int32_t* __restrict__ src_nodes) {
    number_new_kernel_body(gridDim.x, n_words, rounds, posted, bits, sizes, next_n_dst, mark, src_nodes);
}
struct number_new_kernel_op {
    static constexpr int THREADS = WD_THREADS, WGS = 1;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { number_new_kernel_body(gx, a...); }
};

// ---- the transposed blocks, of all layers above the input layer in three launches (blockIdx.y: the layer).
struct TransposeJob {
    const int64_t* sizes;
    const int64_t* ptr;                  // the block
    const int32_t* idx_blk;
    const int32_t* arrival;
    const uint32_t* count_t;
    int64_t src_bound;
    int64_t* ptr_t;                      // [src_bound + 1]; the rows past the real sources are empty
    int32_t* loose;                      // the rows' edges in order of arrival
    int32_t* idx_t;
    int rounds, parts;                   // of the sources
    unsigned long long* posted;          // [2 PARTS] edges; long rows and their chunks
    int32_t *long_row, *long_first;      // the split schedule of the long rows, up to its capacities
    int64_t *chunk_begin, *chunk_end;
    int64_t cap_long, cap_chunks;
};
template <int MOST> struct TransposeJobsOf { TransposeJob d[MOST]; };
using TransposeJobs = TransposeJobsOf<GRP_MAX_LAYERS - 1>;

// Row pointers and the schedule of the long rows (as long_rows_emit_kernel makes it; places past the real ones do nothing).
template <int MOST>
__device__ __forceinline__ void transpose_rows_kernel_body(unsigned gx, const TransposeJobsOf<MOST>& jobs) {
    __shared__ unsigned long long wave_sum[CS_THREADS / 64];
    __shared__ unsigned long long before_s[2];
    const TransposeJob& t = jobs.d[blockIdx.y];
    if ((int)blockIdx.x >= t.parts) return;
    const int part = (int)blockIdx.x, tid = threadIdx.x;
    const int64_t part0 = (int64_t)part * t.rounds * CS_ROUND;
    uint32_t c[CS_PER];
    auto load = [&](int round, unsigned long long& longs) {
        unsigned long long sum = 0;
        longs = 0;
#pragma unroll
        for (int q = 0; q < CS_PER; ++q) {
            const int64_t i = part0 + (int64_t)round * CS_ROUND + CS_PER * tid + q;
            c[q] = i < t.src_bound ? t.count_t[i] : 0u;
            sum += c[q];
            if (c[q] > (uint32_t)SPMM_LONG_ROW) longs += (1ull << 31) + (c[q] + SPMM_CHUNK - 1) / SPMM_CHUNK;
        }
        return sum;
    };
    unsigned long long mine = 0, mine_long = 0, total[2], round_total, l;
    for (int round = 0; round < t.rounds; ++round) {
        mine += load(round, l);
        mine_long += l;
    }
    (void)block_scan<CS_THREADS / 64>(mine, wave_sum, total[0]);
    (void)block_scan<CS_THREADS / 64>(mine_long, wave_sum, total[1]);
    if (tid < 128) {                                         // a wavefront each
        const unsigned long long b = look_back(t.posted + (tid / 64) * PARTS, part, tid < 64 ? total[0] : total[1]);
        if ((tid & 63) == 0) before_s[tid / 64] = b;
    }
    __syncthreads();
    unsigned long long at0 = before_s[0], long0 = before_s[1];
    for (int round = 0; round < t.rounds; ++round) {
        const unsigned long long sum = t.rounds == 1 ? mine : load(round, l);
        if (t.rounds == 1) l = mine_long;
        unsigned long long at = at0 + block_scan<CS_THREADS / 64>(sum, wave_sum, round_total);
        at0 += round_total;
        unsigned long long slot = long0 + block_scan<CS_THREADS / 64>(l, wave_sum, round_total);
        long0 += round_total;
#pragma unroll
        for (int q = 0; q < CS_PER; ++q) {
            const int64_t i = part0 + (int64_t)round * CS_ROUND + CS_PER * tid + q;
            if (i <= t.src_bound) t.ptr_t[i] = (int64_t)at;
            if (c[q] > (uint32_t)SPMM_LONG_ROW) {
                const int64_t j = (int64_t)(slot >> 31);
                int64_t k = (int64_t)(slot & 0x7FFFFFFFull);
                slot += (1ull << 31) + (c[q] + SPMM_CHUNK - 1) / SPMM_CHUNK;
                if (j < t.cap_long) {
                    t.long_row[j] = (int32_t)i;
                    t.long_first[j] = (int32_t)k;
                }
                const int64_t end = (int64_t)(at + c[q]);
                for (int64_t e = (int64_t)at; e < end && k < t.cap_chunks; e += SPMM_CHUNK, ++k) {
                    t.chunk_begin[k] = e;
                    t.chunk_end[k] = e + SPMM_CHUNK < end ? e + SPMM_CHUNK : end;
                }
            }
            at += c[q];
        }
    }
    if (part == t.parts - 1) {                               // (long0 is the sum of all)
        const int64_t n_long = (int64_t)(long0 >> 31), n_chunks = (int64_t)(long0 & 0x7FFFFFFFull);
        for (int64_t j = n_long + tid; j <= t.cap_long; j += CS_THREADS) {
            if (j < t.cap_long) t.long_row[j] = -1;
            t.long_first[j] = (int32_t)(n_chunks < t.cap_chunks ? n_chunks : t.cap_chunks);
        }
        for (int64_t k = n_chunks + tid; k < t.cap_chunks; k += CS_THREADS) { t.chunk_begin[k] = 0; t.chunk_end[k] = 0; }
    }
}
template <int MOST>
__global__ __launch_bounds__(CS_THREADS) void transpose_rows_kernel(TransposeJobsOf<MOST> jobs) {
    transpose_rows_kernel_body<MOST>(gridDim.x, jobs);
}
template <int MOST>
struct transpose_rows_kernel_op {
    static constexpr int THREADS = CS_THREADS, WGS = 1;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { transpose_rows_kernel_body<MOST>(gx, a...); }
};

// Every edge to its source's row, in order of arrival.
template <int MOST>
__device__ __forceinline__ void transpose_scatter_kernel_body(unsigned gx, const TransposeJobsOf<MOST>& jobs) {
    const TransposeJob& t = jobs.d[blockIdx.y];
    const int64_t n_dst = t.sizes[SZ_DST];
    for (int64_t i = (int64_t)blockIdx.x * 4 + threadIdx.x / 64; i < n_dst; i += (int64_t)gx * 4)
        for (int64_t e = t.ptr[i] + (threadIdx.x & 63); e < t.ptr[i + 1]; e += 64) t.loose[t.ptr_t[t.idx_blk[e]] + t.arrival[e]] = (int32_t)i;
}
template <int MOST>
__global__ __launch_bounds__(256) void transpose_scatter_kernel(TransposeJobsOf<MOST> jobs) {
    transpose_scatter_kernel_body<MOST>(gridDim.x, jobs);
}
template <int MOST>
struct transpose_scatter_kernel_op {
    static constexpr int THREADS = 256, WGS = 1;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { transpose_scatter_kernel_body<MOST>(gx, a...); }
};

// Every source's row in ascending order, whatever the order of arrival was.  A workgroup owns TS_ROWS rows: as many of them as fit
// are taken into LDS, where an edge's place is the number of smaller ones in its row (of equal ones, by where they lie); a row of more
// than TS_RANK edges is counted id by id instead, TS_CAP destinations at a time.  (7.5 us for two blocks of 6e3 and 7e4 places; walking the
// rows one by one to see which fit took 27 us more.)
constexpr int TS_THREADS = 256;
constexpr int TS_ROWS = 256;
constexpr int TS_CAP = 8192;
constexpr int TS_RANK = 128;
template <int MOST>
__device__ __forceinline__ void transpose_sort_kernel_body(unsigned gx, const TransposeJobsOf<MOST>& jobs) {
    __shared__ uint32_t buf[TS_CAP];
    __shared__ uint32_t off[TS_ROWS + 1];
    __shared__ unsigned long long long_rows[TS_ROWS / 64];   // the rows that are too long to be ranked
    __shared__ uint32_t wave_sum[TS_THREADS / 64];
    static_assert(TS_ROWS == TS_THREADS, "a thread per row");
    const TransposeJob& t = jobs.d[blockIdx.y];
    const int64_t n_src = t.sizes[SZ_SRC], n_dst = t.sizes[SZ_DST];
    const int tid = threadIdx.x;
    for (int64_t row0 = (int64_t)blockIdx.x * TS_ROWS; row0 < n_src; row0 += (int64_t)gx * TS_ROWS) {
        const int rows = (int)(n_src - row0 < TS_ROWS ? n_src - row0 : TS_ROWS);
        const int64_t e0 = t.ptr_t[row0];
        const uint32_t mine = (uint32_t)(t.ptr_t[row0 + (tid < rows ? tid : rows)] - e0), next = (uint32_t)(t.ptr_t[row0 + (tid < rows ? tid + 1 : rows)] - e0);
        off[tid] = mine;
        if (tid == TS_ROWS - 1) off[TS_ROWS] = next;         // (rows past the last are empty)
        const unsigned long long too_long = __ballot(next - mine > (uint32_t)TS_RANK);
        if ((tid & 63) == 0) long_rows[tid / 64] = too_long;
        __syncthreads();
        const int32_t* const in = t.loose + e0;
        int32_t* const out = t.idx_t + e0;
        for (int ra = 0; ra < rows;) {                           // (uniform)
            const uint32_t base = off[ra];
            int rb = rows;                                       // rows ra .. rb - 1 fit, and none of them is too long to be ranked
            for (int q = TS_ROWS / 64 - 1; q >= ra / 64; --q) {
                const unsigned long long l = q == ra / 64 ? long_rows[q] & (~0ull << (ra & 63)) : long_rows[q];
                if (l) rb = 64 * q + __ffsll(l) - 1;
            }
            if (off[rb] - base > (uint32_t)TS_CAP) {
                int x = ra, y = rb;                              // off[x] - base <= TS_CAP < off[y] - base
                while (y - x > 1) {
                    const int mid = (x + y) >> 1;
                    if (off[mid] - base <= (uint32_t)TS_CAP) x = mid; else y = mid;
                }
                rb = x;
            }
            if (rb > ra) {
                const uint32_t m = off[rb] - base;
                for (uint32_t e = tid; e < m; e += TS_THREADS) buf[e] = (uint32_t)in[base + e];
                __syncthreads();
                for (uint32_t e = tid; e < m; e += TS_THREADS) {
                    int lo = ra, hi = rb;                        // the row of e: off[lo] <= base + e < off[lo + 1]
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (off[mid] <= base + e) lo = mid; else hi = mid;
                    }
                    const uint32_t b = off[lo] - base, z = off[lo + 1] - base, key = buf[e];
                    uint32_t rank = 0;
                    for (uint32_t j = b; j < z; j += 8) {    // (eight reads in flight)
                        uint32_t other[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) other[q] = buf[j + q < z ? j + q : e];
#pragma unroll
                        for (int q = 0; q < 8; ++q) rank += j + q < z && (other[q] < key || (other[q] == key && j + q < e)) ? 1u : 0u;
                    }
                    out[base + b + rank] = (int32_t)key;
                }
                __syncthreads();
                ra = rb;
                continue;
            }
            const uint32_t m = off[ra + 1] - base;               // one long row
            int32_t* o = out + base;
            for (int64_t d0 = 0; d0 < n_dst; d0 += TS_CAP) {
                for (int i = tid; i < TS_CAP; i += TS_THREADS) buf[i] = 0u;
                __syncthreads();
                constexpr int U = 8;
                for (uint32_t j0 = 0; j0 < m; j0 += U * TS_THREADS) {
                    int64_t d[U];
    #pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t j = j0 + u * TS_THREADS + tid;
                        d[u] = (int64_t)in[base + (j < m ? j : m - 1)] - d0;
                        if (j >= m) d[u] = -1;
                    }
    #pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (d[u] >= 0 && d[u] < TS_CAP) atomicAdd(&buf[d[u]], 1u);
                }
                __syncthreads();
                constexpr int PER = TS_CAP / TS_THREADS;
                uint32_t sum = 0, total;
                for (int i = 0; i < PER; ++i) sum += buf[tid * PER + i];
                uint32_t at = block_scan<TS_THREADS / 64>(sum, wave_sum, total);
                for (int i = 0; i < PER; ++i)
                    for (uint32_t c = buf[tid * PER + i]; c > 0; --c) o[at++] = (int32_t)(d0 + tid * PER + i);
                o += total;
                __syncthreads();
            }
            ra = ra + 1;
        }
        __syncthreads();                                     // off is filled anew
    }
}
template <int MOST>
__global__ __launch_bounds__(TS_THREADS) void transpose_sort_kernel(TransposeJobsOf<MOST> jobs) {
    transpose_sort_kernel_body<MOST>(gridDim.x, jobs);
}
template <int MOST>
struct transpose_sort_kernel_op {
    static constexpr int THREADS = TS_THREADS, WGS = 1;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { transpose_sort_kernel_body<MOST>(gx, a...); }
};

// A list of sources names every node once, but for the seeds: those that had to be replaced, and those that the caller repeated, stand in
// it as often as in the seed list.  So it may hold n_seeds - 1 more than the partition has nodes.
void sampler_bounds(int64_t n, int64_t n_seeds, const int32_t* fanouts, int k, SamplerBounds* out) {
    int64_t nd = n_seeds;
    for (int l = k - 1; l >= 0; --l) {
        out->dst[l] = nd;
        out->nnz[l] = nd * fanouts[l];
        int64_t ns = nd + out->nnz[l];
        if (ns > n + n_seeds - 1) ns = n + n_seeds - 1;
        out->src[l] = ns;
        nd = ns;
    }
}

struct SamplerLayerBufs {
    int64_t* ptr;        // [dst+1]
    int32_t* cnt32;      // [dst] (the seeds' layer)
    int32_t* idx_local;  // [nnz] partition-local source ids
    int32_t* idx_blk;    // [nnz] block-local (layers >= 1)
    int32_t* src_nodes;  // [src] (layers >= 1)
    int32_t *arrival, *loose;      // [nnz] (layers >= 1) scratch of the transposed block
    uint32_t* count_t;             // [src] (layers >= 1)
    int64_t* ptrT;       // [src+1]
    int32_t* idxT;       // [nnz]
    float* inv_in;       // [dst]
    int32_t *lr_row, *lr_first;    // long rows of the transposed block
    int64_t *lr_cb, *lr_ce;
    int64_t lr_cap_long, lr_cap_chunks;
    unsigned long long* posted;    // [4 PARTS] of the rows' counts, the new nodes and the transposed rows (two)
};

struct SamplerBufs {
    SamplerLayerBufs L[GRP_MAX_LAYERS];
    int32_t* seeds;                     // [n_seeds] the caller's seeds, range-checked
    int64_t* sizes;                     // [SZ_PER_LAYER * GRP_MAX_LAYERS] the blocks' real sizes (see the enum)
    int32_t* mark;                      // [n] block-local index + 1 of the current layer's nodes, anything elsewhere
    // what starts at zero, carved back to back: one fill clears it
    int64_t* bad;                       // [2] seeds outside the partition
    uint32_t* bits;                     // [n_words] bitmap of newly reached nodes
    int64_t n_words;                    // rounded up to what a thread of number_new_kernel takes
    char *clear_from, *clear_to;
    size_t total;
};

static SamplerBufs carve_sampler(int64_t n, const SamplerBounds& b, int k, void* ws, size_t ws_bytes) {
    SamplerBufs s;
    Bump bump(ws, ws_bytes);
    s.sizes = bump.take<int64_t>(SZ_PER_LAYER * GRP_MAX_LAYERS);
    s.seeds = bump.take<int32_t>((size_t)b.dst[k - 1]);
    for (int l = 0; l < k; ++l) {
        SamplerLayerBufs& L = s.L[l];
        L = SamplerLayerBufs{};
        L.ptr = bump.take<int64_t>((size_t)b.dst[l] + 1);
        if (l == k - 1) L.cnt32 = bump.take<int32_t>((size_t)b.dst[l]);
        L.idx_local = bump.take<int32_t>((size_t)b.nnz[l]);
        L.inv_in = bump.take<float>((size_t)b.dst[l]);
        if (l > 0) {
            L.idx_blk = bump.take<int32_t>((size_t)b.nnz[l]);
            L.src_nodes = bump.take<int32_t>((size_t)b.src[l]);
            L.arrival = bump.take<int32_t>((size_t)b.nnz[l]);
            L.loose = bump.take<int32_t>((size_t)b.nnz[l]);
            L.ptrT = bump.take<int64_t>((size_t)b.src[l] + 1);
            L.idxT = bump.take<int32_t>((size_t)b.nnz[l]);
            L.lr_cap_long = b.nnz[l] / SPMM_LONG_ROW + 1;
            L.lr_cap_chunks = b.nnz[l] / SPMM_CHUNK + L.lr_cap_long + 1;
            L.lr_row = bump.take<int32_t>((size_t)L.lr_cap_long);
            L.lr_first = bump.take<int32_t>((size_t)L.lr_cap_long + 1);
            L.lr_cb = bump.take<int64_t>((size_t)L.lr_cap_chunks);
            L.lr_ce = bump.take<int64_t>((size_t)L.lr_cap_chunks);
        }
    }
    s.mark = bump.take<int32_t>((size_t)n);
    s.n_words = round_up(cdiv(n, 32), WD_PER);
    s.bad = bump.take<int64_t>(2);
    for (int l = 0; l < k; ++l) {
        s.L[l].posted = bump.take<unsigned long long>(4 * PARTS);
        if (l > 0) s.L[l].count_t = bump.take<uint32_t>((size_t)b.src[l]);
    }
    s.bits = bump.take<uint32_t>(k > 1 ? (size_t)s.n_words : 1);
    s.clear_from = (char*)s.bad;
    s.clear_to = (char*)(s.bits + (k > 1 ? s.n_words : 1));
    s.total = bump.total();
    return s;
}

size_t sampler_workspace_bytes(int64_t n, const SamplerBounds& b, int k) { return carve_sampler(n, b, k, nullptr, 0).total; }

grp_status sample_blocks(const grp_partition_t* part, const grp_step_opts* o, int k, void* ws, size_t ws_bytes,
                         Block* blocks, LongRows* long_bwd_store, const int64_t** nnz_parts_dev,
                         const int32_t** seed_counts_dev, const int64_t** bad_seeds_dev, hipStream_t st,
                         hipEvent_t* transposed_ready) {
    const int64_t n = part->n;
    *transposed_ready = nullptr;
    if (o->n_seeds < 1 || !o->seeds) return fail(GRP_EINVAL, "mini-batch: need at least one seed node");
    if (n == 0) return fail(GRP_ERANGE, "mini-batch: seeds given for a partition without nodes");
    for (int l = 0; l < k; ++l)
        if (o->fanouts[l] < 1 || o->fanouts[l] > SAMPLE_MAX_FANOUT)
            return fail(GRP_EINVAL, "mini-batch: fanout %d outside [1, %d]", o->fanouts[l], SAMPLE_MAX_FANOUT);
    SamplerBounds bd;
    sampler_bounds(n, o->n_seeds, o->fanouts, k, &bd);
    SamplerBufs s = carve_sampler(n, bd, k, ws, ws_bytes);
    if (s.total > ws_bytes) return fail(GRP_EWORKSPACE, "mini-batch: sampler workspace %zu < %zu", ws_bytes, s.total);

    GRP_TRY(launch_fill_zero(s.clear_from, (size_t)(s.clear_to - s.clear_from), st));
    *bad_seeds_dev = s.bad;
    const uint64_t h0 = mixM(o->sampler_seed);
    const int32_t* dst_nodes = s.seeds;
    RelabelJob relabel{};                                // of the layer before
    TransposeJobs jobs{};
    for (int l = k - 1; l >= 0; --l) {
        SamplerLayerBufs& L = s.L[l];
        int64_t* const D = s.sizes + SZ_PER_LAYER * l;   // this layer's sizes; D[SZ_DST] is already there
        const int64_t dst_bound = bd.dst[l];
        const int f = o->fanouts[l];
        const bool top = l == k - 1;
        const ScanPlan cp = look_back_plan(dst_bound + 1, CS_ROUND, steps_of_launch());
        const CountJob count{part->rowptr, dst_nodes, top ? o->seeds : nullptr, n, (int64_t)o->n_seeds, D, dst_bound, f, cp.rounds, cp.parts, L.posted,
                             L.ptr, L.cnt32, L.inv_in, top && l > 0 ? s.mark : nullptr, L.src_nodes, (unsigned long long*)s.bad};
        launch(count_rows_kernel, count_rows_kernel_op(), dim3((unsigned)(cp.parts + (relabel.ptr ? cdiv(relabel.dst_bound, 4) : 0))), st, count, relabel);
        GRP_LAUNCH_CHECK();
        if (l == 0 && k > 1) {
            // The transposed blocks are read by the backward pass only: they are built on a helper stream, beside the choice of the input
            // layer's edges and the forward pass.
            SideLane* const lane = !(o->flags & GRP_STEP_ONE_STREAM) ? side_lane(st) : nullptr;
            hipStream_t bst = st;
            if (lane) {
                GRP_HIP(hipEventRecord(lane->fork[0], st));
                GRP_HIP(hipStreamWaitEvent(lane->stream, lane->fork[0], 0));
                bst = lane->stream;
            }
            int parts = 0;
            for (int q = 1; q < k; ++q) parts = std::max(parts, jobs.d[q - 1].parts);
            const int64_t dst_groups = std::min(cdiv(bd.dst[1], 4), (int64_t)1 << 18);             // (layer 1 is the largest)
            const int64_t src_groups = std::min(cdiv(bd.src[1], TS_ROWS), (int64_t)1 << 18);
            constexpr int FEW = 3;                       // arguments of several steps fit one launch
            if (k - 1 <= FEW) {
                TransposeJobsOf<FEW> few{};
                for (int q = 0; q < k - 1; ++q) few.d[q] = jobs.d[q];
                launch(transpose_rows_kernel<FEW>, transpose_rows_kernel_op<FEW>(), dim3((unsigned)parts, (unsigned)(k - 1)), bst, few);
                launch(transpose_scatter_kernel<FEW>, transpose_scatter_kernel_op<FEW>(), dim3((unsigned)dst_groups, (unsigned)(k - 1)), bst, few);
                launch(transpose_sort_kernel<FEW>, transpose_sort_kernel_op<FEW>(), dim3((unsigned)src_groups, (unsigned)(k - 1)), bst, few);
            } else {
                constexpr int ALL = GRP_MAX_LAYERS - 1;
                launch_alone(transpose_rows_kernel<ALL>, dim3((unsigned)parts, (unsigned)(k - 1)), dim3(CS_THREADS), 0, bst, jobs);
                launch_alone(transpose_scatter_kernel<ALL>, dim3((unsigned)dst_groups, (unsigned)(k - 1)), dim3(256), 0, bst, jobs);
                launch_alone(transpose_sort_kernel<ALL>, dim3((unsigned)src_groups, (unsigned)(k - 1)), dim3(TS_THREADS), 0, bst, jobs);
            }
            GRP_LAUNCH_CHECK();
            if (lane) {
                GRP_HIP(hipEventRecord(lane->join, lane->stream));
                *transposed_ready = lane->join;
            }
        }
        {
            ProfScope ps("sample_select", st);
            launch(sample_select_kernel, sample_select_kernel_op(), dim3((unsigned)cdiv(dst_bound, SAMPLE_ROWS_PER_WG)), st, part->rowptr, part->col, part->l2g, dst_nodes, D, f,
                               h0, (uint64_t)o->batch_id, o->batch_id_dev, l, (const int64_t*)L.ptr, L.idx_local, (const int32_t*)s.mark,
                               l > 0 ? s.bits : nullptr);
            GRP_LAUNCH_CHECK();
        }

        Block& B = blocks[l];
        B.n_dst = dst_bound;
        B.n_dst_dev = D + SZ_DST;
        B.nnz = bd.nnz[l];
        B.dst_nodes = dst_nodes;
        B.ptr = L.ptr;
        B.inv_in = L.inv_in;
        B.long_fwd = nullptr;                            // rows hold at most `fanout` edges
        nnz_parts_dev[l] = D + SZ_NNZ;
        if (top) *seed_counts_dev = L.cnt32;
        if (l == 0) {
            B.idx = L.idx_local;
            B.n_in = n;
            B.n_in_dev = nullptr;                        // the inputs are the partition's nodes
            B.self_rows = dst_nodes;
            B.ptrT = nullptr; B.idxT = nullptr; B.long_bwd = nullptr;
            break;
        }
        // new source nodes in ascending local id
        const int64_t src_bound = bd.src[l];
        const ScanPlan wp = look_back_plan(s.n_words, WD_ROUND, steps_of_launch());
        launch(number_new_kernel, number_new_kernel_op(), dim3((unsigned)wp.parts), st, s.n_words, wp.rounds, L.posted + PARTS, s.bits, D,
                           s.sizes + SZ_PER_LAYER * (l - 1) + SZ_DST, s.mark, L.src_nodes);
        GRP_LAUNCH_CHECK();
        relabel = RelabelJob{L.ptr, D, dst_bound, L.idx_local, s.mark, L.idx_blk, L.arrival, L.count_t};
        const ScanPlan tp = look_back_plan(src_bound + 1, CS_ROUND, (k - 1) * steps_of_launch());
        jobs.d[l - 1] = TransposeJob{D, L.ptr, L.idx_blk, L.arrival, L.count_t, src_bound, L.ptrT, L.loose, L.idxT, tp.rounds, tp.parts,
                                     L.posted + 2 * PARTS, L.lr_row, L.lr_first, L.lr_cb, L.lr_ce, L.lr_cap_long, L.lr_cap_chunks};
        LongRows& lr = long_bwd_store[l];
        lr.long_row = L.lr_row; lr.long_first = L.lr_first; lr.chunk_begin = L.lr_cb; lr.chunk_end = L.lr_ce;
        lr.n_long = (int32_t)L.lr_cap_long;              // (the launches cover the capacities)
        lr.n_chunks = (int32_t)L.lr_cap_chunks;
        B.idx = L.idx_blk;
        B.n_in = src_bound;
        B.n_in_dev = D + SZ_SRC;
        B.self_rows = nullptr;
        B.ptrT = L.ptrT;
        B.idxT = L.idxT;
        B.long_bwd = &lr;
        dst_nodes = L.src_nodes;
    }
    return GRP_OK;
}

// Where a finished step left block `layer` inside its sampler workspace (same partition size, seeds count,
// fanouts and depth).  Copies the block sizes from the device: synchronises the device.
grp_status sampler_block_view(const grp_partition_t* part, const grp_step_opts* o, int k, void* ws, size_t ws_bytes, int layer,
                              grp_block_view_t* out) {
    SamplerBounds bd;
    sampler_bounds(part->n, o->n_seeds, o->fanouts, k, &bd);
    const SamplerBufs s = carve_sampler(part->n, bd, k, ws, ws_bytes);
    if (s.total > ws_bytes) return fail(GRP_EWORKSPACE, "grp_step_block: sampler workspace %zu < %zu", ws_bytes, s.total);
    int64_t sizes[SZ_PER_LAYER * GRP_MAX_LAYERS] = {0};
    GRP_HIP(hipDeviceSynchronize());
    GRP_HIP(hipMemcpy(sizes, s.sizes, sizeof sizes, hipMemcpyDeviceToHost));
    const int64_t* const D = sizes + SZ_PER_LAYER * layer;
    const SamplerLayerBufs& L = s.L[layer];
    if (D[SZ_DST] < 0 || D[SZ_DST] > bd.dst[layer] || D[SZ_NNZ] < 0 || D[SZ_NNZ] > bd.nnz[layer])
        return fail(GRP_EINVAL, "grp_step_block: the workspace does not hold a step of this shape");
    out->n_dst = D[SZ_DST];
    out->nnz = D[SZ_NNZ];
    out->rowptr = L.ptr;
    out->dst_nodes = layer == k - 1 ? s.seeds : s.L[layer + 1].src_nodes;
    if (layer == 0) {
        out->n_src = part->n;
        out->col = L.idx_local;
        out->src_nodes = nullptr;
    } else {
        if (D[SZ_SRC] < D[SZ_DST] || D[SZ_SRC] > bd.src[layer])
            return fail(GRP_EINVAL, "grp_step_block: the workspace does not hold a step of this shape");
        out->n_src = D[SZ_SRC];
        out->col = L.idx_blk;
        out->src_nodes = L.src_nodes;
    }
    return GRP_OK;
}

}  // namespace grp
