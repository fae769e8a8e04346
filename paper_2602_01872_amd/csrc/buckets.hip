// CSR and CSC of an edge list from its unordered keys (destination << 32 | source), both at once.
//
// A device-wide radix sort of 64-bit keys reads and writes them once per digit, seven passes for a million nodes and half as many
// again for the transpose, each with its launches and clears.  Here a direction is cut into buckets of consecutive rows that hold
// a few thousand keys each: one pass counts the buckets of both directions, one writes every key to its two buckets (as 32 bits:
// row within the bucket, other end), and a workgroup per bucket sorts its keys in LDS and writes the pointers, the degrees and
// the indices.  Equal keys are indistinguishable, so the arrays are unique, whatever order the keys arrived in.
//
// What skewed graphs ask for: a bucket of a few more keys than LDS holds is sorted a range of rows at a time, one of many more puts them in
// order of their rows in memory and leaves the sorting to jobs, of a range of rows each or, where a single row has more keys than LDS holds
// (a hub), of a range of the other end's ids.  One workgroup orders a bucket, and every job of a hub reads all its keys: where either would
// take longer than a device-wide sort, the build is refused and goes there (bucket_build).
// Builds, ms, of graphs numbered so that heavy rows are neighbours (buckets / every range and hub reading its whole bucket again /
// radix sorts): R-MAT by degree, 3e5 nodes 3e6 edges 0.61 / 8.0 / 6.9, 2e6 3e7 3.0 / 203 / 57; all edges to 1000 nodes numbered first, 2e6 3e7
// 2.8 / 1133 / 52, 300 of 6e5 3.9e6 0.82 / 187 / 15.8; to one node, 1e6 2e7 3.6 / 72 / 20.  (The sorts took their time over the
// pointers of empty rows: csr_rows_kernel.)
#include "common.h"

namespace grp {

constexpr int BK_THREADS = 1024;
constexpr int BK_WAVES = BK_THREADS / 64;
constexpr int BK_PER = 8;                       // keys a thread sorts
constexpr int BK_CAP = BK_THREADS * BK_PER;     // keys sorted at a time: 32 KB of LDS
constexpr int BK_AIM = BK_CAP / 2;              // keys of a bucket, on average: room for twice as many
constexpr int BK_MAX = 4096;                    // buckets of a direction
constexpr int BK_ROW_BITS = 11;                 // rows of a bucket: at most 2048, two per thread
constexpr int BK_DIGIT = 6;                     // bits of a sorting pass: a wavefront's 64 counters
constexpr int BK_SUB = 8;                       // keys that share a part of their row, about
constexpr int BK_SUB_MAX = 64;                  // keys of a part that are ranked against each other
constexpr int BK_SUBS = (1 << BK_ROW_BITS) + 2 * BK_CAP / BK_SUB;
constexpr int HUB_SPAN = 8192;                  // ids that are counted at a time where a hub's keys crowd: 32 KB of LDS
constexpr int HUB_PART = 2048;                  // keys of a hub's job, if they are spread evenly: many short jobs, each of which reads all keys,
constexpr int HUB_LONG = 1 << 18;               // or, of a hub of more than this, BK_AIM keys
constexpr int JOB_GROUPS = 512;
constexpr int BK_ALONE = 2 * BK_CAP;            // keys that a bucket's workgroup sorts itself, reading them again for every range of rows
constexpr int JOB_KEYS = BK_CAP / 2;            // a range of rows: those that begin within so many keys, but for one of more keys at its end

// Fewest buckets of at most BK_AIM keys on average (more where there would be too many of them), 2048 rows and 32 bits of key.  Builds from
// n nodes and E local edges of a skewed graph, destroy included (us; radix sorts of 64-bit keys -> buckets): 1e3, 4e3 180 -> 110;
// 2e4, 1.6e5 280 -> 115; 1e5, 7e5 405 -> 178; 3e5, 3e6 585 -> 285; 1e6, 2e7 2290 -> 1530; 2.4e6, 5e7 4670 -> 3500; 4e6, 6e7 5700 -> 4110.
bool bucket_plan(int64_t n, int64_t nnz, BucketPlan* p) {
    if (n < 1 || nnz < 1 || n > ((int64_t)1 << 22) || nnz > ((int64_t)1 << 26)) return false;
    p->id_bits = 1;
    while (((int64_t)1 << p->id_bits) < n) ++p->id_bits;
    const int most = std::min(BK_ROW_BITS, 32 - p->id_bits);       // (2^22 nodes: 10, and as many buckets as there may be)
    int r = most;
    while (r > 0 && (nnz << r) > n * BK_AIM) --r;
    while (r < most && ((n - 1) >> r) >= BK_MAX) ++r;
    p->row_bits = r;
    p->n_buckets = (int)(((n - 1) >> r) + 1);
    return p->n_buckets <= BK_MAX;
}

struct BucketScratch {
    unsigned long long* totals;      // [5] sums: longs, edges of the CSR, of the CSC; keys that the hubs' jobs read (cleared)
    uint32_t* count;                 // [2 B] keys of the buckets (cleared)
    uint32_t* n_jobs;                // [1] (cleared)
    uint32_t* start;                 // [2 (B + 1)] first key of each bucket
    uint32_t* cursor;                // [2 B]
    unsigned long long* longs;       // [2 B] long rows << 32 | their chunks
    unsigned long long* edges;       // [2 B] edges of the long rows
    uint4* jobs;                     // direction << 31 | JOB_ROWS or first id, id after the last, first key, keys
    uint32_t bucket_most;            // keys of a bucket, and keys that the hubs' jobs read, beyond which the build is refused
    unsigned long long hubs_most;
    size_t bytes, clear_bytes;
};
constexpr unsigned long long REFUSED_AT_ONCE = 1ull << 62;       // in totals[4], before the keys are moved
constexpr uint32_t JOB_ROWS = 1u << 30;          // the job's keys are those of whole rows
static BucketScratch carve_scratch(const BucketPlan& p, int64_t nnz, void* base) {
    BucketScratch s;
    Bump b(base, 0);
    const size_t B = (size_t)p.n_buckets;
    s.totals = b.take<unsigned long long>(5 + B + 1);
    s.count = (uint32_t*)(s.totals + 5);
    s.n_jobs = s.count + 2 * B;
    s.clear_bytes = 5 * sizeof(unsigned long long) + (2 * B + 1) * sizeof(uint32_t);
    s.start = b.take<uint32_t>(2 * (B + 1));
    s.cursor = b.take<uint32_t>(2 * B);
    s.longs = b.take<unsigned long long>(2 * B);
    s.edges = b.take<unsigned long long>(2 * B);
    // a direction's jobs: ranges of rows, at most one more per crowded bucket than whole JOB_KEYS; rows of more than JOB_KEYS keys; parts of hubs
    s.jobs = b.take<uint4>(2 * (size_t)(2 * (nnz / JOB_KEYS) + nnz / HUB_PART + 2 * (nnz / BK_CAP)) + 1);
    // One workgroup reads a bucket's keys twice, some five a nanosecond each time, and the hubs' jobs read 128 times the edges in about
    // as long as the sorts take (30 hubs of 1e6 keys: 6.7 ms by jobs, 4.0 refused; of 1e5: 0.62 by jobs, 1.3 by sorts).
    s.bucket_most = (uint32_t)std::max<int64_t>((int64_t)1 << 20, nnz / 16);
    s.hubs_most = 128ull * (unsigned long long)nnz;
    s.bytes = b.total();
    return s;
}
size_t bucket_scratch_bytes(const BucketPlan& p, int64_t nnz) { return carve_scratch(p, nnz, nullptr).bytes; }

__global__ __launch_bounds__(BK_THREADS) void bucket_count_kernel(const uint64_t* __restrict__ keys, int64_t nnz, BucketPlan p, int dirs,
                                                                  uint32_t* __restrict__ count) {
    extern __shared__ uint32_t hist[];                     // [2 B]
    const int B = p.n_buckets;
    for (int i = threadIdx.x; i < 2 * B; i += BK_THREADS) hist[i] = 0u;
    __syncthreads();
    for (int64_t e = (int64_t)blockIdx.x * BK_THREADS + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * BK_THREADS) {
        const uint64_t k = keys[e];
        atomicAdd(&hist[(uint32_t)(k >> 32) >> p.row_bits], 1u);
        if (dirs > 1) atomicAdd(&hist[B + ((uint32_t)k >> p.row_bits)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * B; i += BK_THREADS)
        if (hist[i]) atomicAdd(&count[i], hist[i]);
}

__global__ __launch_bounds__(BK_THREADS) void bucket_start_kernel(BucketScratch s, int B) {
    __shared__ uint32_t wave_sum[BK_WAVES];
    constexpr int PER = BK_MAX / BK_THREADS;
    for (int dir = 0; dir < 2; ++dir) {
        uint32_t c[PER], sum = 0, total;
        bool too_many = false;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int b = PER * threadIdx.x + i;
            c[i] = b < B ? s.count[dir * B + b] : 0u;
            sum += c[i];
            too_many = too_many || c[i] > s.bucket_most;
        }
        if (too_many) s.totals[4] = REFUSED_AT_ONCE;
        uint32_t at = block_scan<BK_WAVES>(sum, wave_sum, total);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int b = PER * threadIdx.x + i;
            if (b < B) s.start[dir * (B + 1) + b] = s.cursor[dir * B + b] = at;
            at += c[i];
        }
        if (threadIdx.x == 0) s.start[dir * (B + 1) + B] = total;
    }
}

// A tile's keys to their buckets: places counted in LDS, one reservation per tile and bucket, and the keys put in the buckets' order in
// LDS first, so that a bucket's run leaves as neighbouring words (a store of 64 scattered words is 64 requests: 3.9e6 edges into
// 2 x 1170 buckets 89 us, this way 29).  packed: nnz keys of each direction.
constexpr int SC_PER = 16;                                 // (16 bits hold a place in a tile, and a bucket of either direction)
constexpr int SC_TILE = BK_THREADS * SC_PER;
__global__ __launch_bounds__(BK_THREADS) void bucket_scatter_kernel(const uint64_t* __restrict__ keys, int64_t nnz, BucketPlan p, int dirs, int per,
                                                                    const unsigned long long* __restrict__ refused, uint32_t* __restrict__ cursor,
                                                                    uint32_t* __restrict__ packed) {
    extern __shared__ uint32_t lds[];                      // [2 B] counts, then where a bucket's keys go; [tile] keys; [2 B] places; [tile] buckets
    __shared__ uint32_t wave_sum[BK_WAVES];
    if (*refused) return;
    const int B = p.n_buckets, tile = per * BK_THREADS;
    uint32_t* const to = lds;
    uint32_t* const buf = lds + 2 * B;
    uint16_t* const first = (uint16_t*)(buf + tile);
    uint16_t* const of = first + 2 * B;
    const int64_t e0 = (int64_t)blockIdx.x * tile + threadIdx.x;
    const int here = (int)(nnz - (int64_t)blockIdx.x * tile < tile ? nnz - (int64_t)blockIdx.x * tile : tile);
    uint32_t u[SC_PER], v[SC_PER], at[SC_PER];
#pragma unroll
    for (int i = 0; i < SC_PER; ++i) {
        const int64_t e = e0 + (int64_t)i * BK_THREADS;
        const uint64_t k = i < per ? keys[e < nnz ? e : nnz - 1] : 0;
        u[i] = (uint32_t)k;
        v[i] = (uint32_t)(k >> 32);
    }
    for (int i = threadIdx.x; i < 2 * B; i += BK_THREADS) to[i] = 0u;
    __syncthreads();
    auto on = [&](int i) { return i < per && (int)(threadIdx.x + i * BK_THREADS) < here; };
#pragma unroll
    for (int i = 0; i < SC_PER; ++i) {
        if (!on(i)) continue;
        at[i] = atomicAdd(&to[v[i] >> p.row_bits], 1u);
        if (dirs > 1) at[i] |= atomicAdd(&to[B + (u[i] >> p.row_bits)], 1u) << 16;
    }
    __syncthreads();
    {   // reservations (neighbouring lanes ask for neighbouring cursors: a line of them is one request), and places of both directions
        constexpr int PER = 2 * BK_MAX / BK_THREADS;
        uint32_t base[PER], sum = 0, total;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int b = threadIdx.x + q * BK_THREADS;
            const uint32_t c = b < 2 * B ? to[b] : 0u;
            base[q] = c ? atomicAdd(&cursor[b], c) : 0u;
        }
        uint32_t c[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int b = PER * threadIdx.x + q;
            c[q] = b < 2 * B ? to[b] : 0u;
            sum += c[q];
        }
        uint32_t place = block_scan<BK_WAVES>(sum, wave_sum, total);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int b = PER * threadIdx.x + q;           // (the second direction's places follow the first's `here` keys)
            if (b < 2 * B) first[b] = (uint16_t)(b < B ? place : place - (uint32_t)here);
            place += c[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int b = threadIdx.x + q * BK_THREADS;
            if (b < 2 * B) to[b] = base[q] - first[b];
        }
    }
    __syncthreads();
    const uint32_t low = (1u << p.row_bits) - 1u;
    for (int dir = 0; dir < dirs; ++dir) {
#pragma unroll
        for (int i = 0; i < SC_PER; ++i) {
            if (!on(i)) continue;
            const uint32_t r = dir ? u[i] : v[i], b = dir * B + (r >> p.row_bits);
            const uint32_t x = first[b] + (dir ? at[i] >> 16 : at[i] & 0xFFFFu);
            buf[x] = ((r & low) << p.id_bits) | (dir ? v[i] : u[i]);
            of[x] = (uint16_t)b;
        }
        __syncthreads();
        uint32_t* const out = packed + dir * nnz;
        for (int x = threadIdx.x; x < here; x += BK_THREADS) out[to[of[x]] + (uint32_t)x] = buf[x];
        __syncthreads();
    }
}

// f(on, key) for every key, by whole wavefronts (on: the lane has one); eight loads in flight per thread.
template <typename F> __device__ __forceinline__ void each_key(const uint32_t* __restrict__ in, uint32_t count, F f) {
    constexpr int U = 8;
    for (uint32_t i0 = 0; i0 < count; i0 += U * BK_THREADS) {
        uint32_t key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = i0 + u * BK_THREADS + threadIdx.x;
            key[u] = in[i < count ? i : count - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u * BK_THREADS >= count) break;       // (uniform)
            f(i0 + u * BK_THREADS + threadIdx.x < count, key[u]);
        }
    }
}

// counter[row] += 1 for every lane that is on; returns what the counter held, as if the lanes came one after another.  The lanes that have
// the first one's row are counted with one addition (a hub's keys come 64 at a time).
__device__ __forceinline__ uint32_t count_row(bool on, uint32_t row, uint32_t* counter) {
    const unsigned long long who = __ballot(on);
    if (!who) return 0u;
    const bool same = on && row == (uint32_t)__builtin_amdgcn_readlane((int)row, __ffsll(who) - 1);
    const unsigned long long group = __ballot(same);
    const int lane = threadIdx.x & 63, lead = __ffsll(group) - 1;
    uint32_t at = 0u;
    if (on && (!same || lane == lead)) at = atomicAdd(&counter[row], same ? (uint32_t)__popcll(group) : 1u);
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)at, lead);
    return same ? first + (uint32_t)__popcll(group & ((1ull << lane) - 1ull)) : at;
}

struct BucketOut {
    int64_t* ptr[2];
    int32_t* idx[2];
    int32_t* deg[2];
    int32_t* long_row[2];            // null: no row can be long
    int32_t* long_first[2];
    int64_t* chunk_begin[2];
    int64_t* chunk_end[2];
};

// The workgroup's keys k (a wavefront's are consecutive; per of them in each thread) in order of their low `bits` bits, into buf.
struct RadixLds {
    uint32_t digit[BK_WAVES << BK_DIGIT];
    uint32_t wave_sum[BK_WAVES];
};
__device__ __forceinline__ void radix_sort(uint32_t (&k)[BK_PER], int per, int bits, uint32_t* buf, RadixLds& l) {
    static_assert(BK_WAVES == 16 && BK_DIGIT == 6, "a thread per counter");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __syncthreads();
    l.digit[tid] = 0u;
    __syncthreads();
    for (int shift = 0;; shift += BK_DIGIT) {
        uint32_t rank[BK_PER];
#pragma unroll
        for (int i = 0; i < BK_PER; ++i) {
            if (i >= per) break;
            const uint32_t d = (k[i] >> shift) & 63u;
            unsigned long long same = ~0ull;               // lanes with this digit
#pragma unroll
            for (int q = 0; q < BK_DIGIT; ++q) {
                const bool set = (d >> q) & 1u;
                const unsigned long long v = __ballot(set);
                same &= set ? v : ~v;
            }
            const int lead = __ffsll(same) - 1;
            uint32_t old = 0;
            if (lane == lead) old = atomicAdd(&l.digit[wave * 64 + d], (uint32_t)__popcll(same));
            rank[i] = __shfl(old, lead, 64) + __popcll(same & ((1ull << lane) - 1ull));
        }
        __syncthreads();
        uint32_t* const mine = &l.digit[(tid & 15) * 64 + (tid >> 4)];           // by digit, then wavefront
        const uint32_t here = *mine;
        uint32_t incl = here;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) l.wave_sum[wave] = incl;
        __syncthreads();
        uint32_t before = incl - here;
#pragma unroll
        for (int w = 0; w < BK_WAVES; ++w)
            if (w < wave) before += l.wave_sum[w];
        *mine = before;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < BK_PER; ++i) {
            if (i >= per) break;
            buf[l.digit[wave * 64 + ((k[i] >> shift) & 63u)] + rank[i]] = k[i];
        }
        __syncthreads();
        if (shift + BK_DIGIT >= bits) return;
        l.digit[tid] = 0u;
#pragma unroll
        for (int i = 0; i < BK_PER; ++i) {
            if (i >= per) break;
            k[i] = buf[(wave * per + i) * 64 + lane];
        }
        __syncthreads();
    }
}

// One workgroup per bucket.  The keys of a row of d are dealt to the next power of two above d / BK_SUB equal ranges of the other
// end's ids, counted in LDS; each then finds its place among the few of its range by comparing.  Where a range is crowded (a graph
// whose numbering has locality) the rows are sorted digit by digit instead.  (3.9e6 edges of 6e5 nodes, both directions, digits
// alone 250 us, this way 160.)  A bucket of more than BK_CAP keys: see the top of the file.
__global__ __launch_bounds__(BK_THREADS) void bucket_sort_kernel(const uint32_t* __restrict__ packed, int64_t nnz, int64_t n, BucketPlan p,
                                                                 BucketScratch s, BucketOut out, uint32_t* __restrict__ by_row) {
    __shared__ __attribute__((aligned(16))) uint32_t buf[BK_CAP];
    __shared__ uint32_t off[(1 << BK_ROW_BITS) + 1];       // first key of each row of the bucket
    __shared__ uint32_t sub_of[1 << BK_ROW_BITS];          // a row's first range << 5 | how far an id is shifted to its range
    __shared__ union __attribute__((aligned(16))) {
        uint32_t sub[BK_SUBS + 4];                         // keys of each range, then where they begin
        RadixLds radix;
    } u;
    __shared__ uint32_t wave_sum[BK_WAVES];
    __shared__ unsigned long long stat[2];
    __shared__ uint32_t fill;
    const int B = p.n_buckets, dir = (int)blockIdx.x >= B, b = (int)blockIdx.x - dir * B;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t lo = s.start[dir * (B + 1) + b], count = s.start[dir * (B + 1) + b + 1] - lo;
    if (s.totals[4] == REFUSED_AT_ONCE) return;
    const uint32_t* const in = packed + dir * nnz + lo;
    const int64_t first = (int64_t)b << p.row_bits;
    const int rows = (int)(first + (1 << p.row_bits) <= n ? (int64_t)1 << p.row_bits : n - first);
    const uint32_t id_mask = p.id_bits == 32 ? ~0u : (1u << p.id_bits) - 1u;
    for (int i = tid; i < rows; i += BK_THREADS) off[i] = 0u;
    if (tid < 2) stat[tid] = 0ull;
    __syncthreads();
    uint32_t k[BK_PER];
    auto fetch = [&](const uint32_t* from, uint32_t m, int per) {      // a wavefront's keys are consecutive; places past the end sort last
#pragma unroll
        for (int i = 0; i < BK_PER; ++i) {
            const uint32_t at = (uint32_t)((wave * per + i) * 64 + lane);
            k[i] = i < per && at < m ? from[at] : ~0u;
        }
    };
    auto on = [&](int i, uint32_t m, int per) { return i < per && (uint32_t)((wave * per + i) * 64 + lane) < m; };
    const bool whole = count <= (uint32_t)BK_CAP;
    if (whole) {
        const int per = (int)((count + BK_THREADS - 1) / BK_THREADS);
        fetch(in, count, per);
#pragma unroll
        for (int i = 0; i < BK_PER; ++i)
            if (on(i, count, per)) atomicAdd(&off[k[i] >> p.id_bits], 1u);
    } else {
        const bool heavy = count > (uint32_t)BK_ALONE;
        each_key(in, count, [&](bool mine, uint32_t key) {
            if (heavy) (void)count_row(mine, key >> p.id_bits, off);
            else if (mine) atomicAdd(&off[key >> p.id_bits], 1u);
        });
    }
    __syncthreads();
    auto ranges_log = [&](uint32_t d) {                    // a row of d keys has 2^this ranges
        const uint32_t lg = d <= (uint32_t)BK_SUB ? 0u : 32u - __clz((d - 1u) / BK_SUB);
        return lg > (uint32_t)p.id_bits ? (uint32_t)p.id_bits : lg;
    };
    uint32_t n_sub = 0;
    {   // pointers, degrees, and what the schedule of the long rows needs; the ranges too where the bucket is sorted whole (one sum over both)
        static_assert(BK_CAP < 1 << 16 && BK_SUBS < 1 << 16, "16 bits each");
        uint32_t c[2], lg[2], total;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            c[q] = 2 * tid + q < rows ? off[2 * tid + q] : 0u;
            lg[q] = ranges_log(c[q]);
        }
        const uint32_t parts0 = whole && c[0] ? 1u << lg[0] : 0u, parts1 = whole && c[1] ? 1u << lg[1] : 0u;
        uint32_t at = block_scan<BK_WAVES>(c[0] + c[1] + (parts0 + parts1) * 65536u, wave_sum, total);
        if (whole) {
            n_sub = total >> 16;
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (2 * tid + q < rows) sub_of[2 * tid + q] = ((at >> 16) + (q ? parts0 : 0u)) << 5 | ((uint32_t)p.id_bits - lg[q]);
            for (uint32_t i = 4 * tid; i < n_sub; i += 4 * BK_THREADS) *reinterpret_cast<uint4*>(&u.sub[i]) = make_uint4(0u, 0u, 0u, 0u);
            at &= 0xFFFFu;
        }
        unsigned long long longs = 0, edges = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int r = 2 * tid + q;
            if (r < rows) {
                off[r] = at;
                out.ptr[dir][first + r] = (int64_t)lo + at;
                out.deg[dir][first + r] = (int32_t)c[q];
                if (c[q] > (uint32_t)SPMM_LONG_ROW) {
                    longs += (1ull << 32) + (c[q] + SPMM_CHUNK - 1) / SPMM_CHUNK;
                    edges += c[q];
                }
            }
            at += c[q];
        }
        if (longs) { atomicAdd(&stat[0], longs); atomicAdd(&stat[1], edges); }
        if (tid == 0) {
            off[rows] = count;
            if (b == B - 1) out.ptr[dir][n] = nnz;
        }
    }
    __syncthreads();
    if (tid == 0) { s.longs[dir * B + b] = stat[0]; s.edges[dir * B + b] = stat[1]; }

    uint32_t* const to = by_row + dir * nnz + lo;
    if (count > (uint32_t)BK_ALONE) {
        for (int i = tid; i < rows; i += BK_THREADS) sub_of[i] = 0u;       // the rows' keys placed so far
        __syncthreads();
        each_key(in, count, [&](bool mine, uint32_t key) {
            const uint32_t r = key >> p.id_bits, at = count_row(mine, r, sub_of);
            if (mine) to[off[r] + at] = key;
        });
        // Ranges of rows: the rows that begin among the same JOB_KEYS keys, but for a row of more than JOB_KEYS, which is the last of them and a
        // job, or several, of its own.  So a range has at most 2 JOB_KEYS = BK_CAP keys.  A thread looks at two rows, each of which
        // may be the first of a range, and heavy.
        uint32_t begin[2], end[2], parts[2], jobs = 0, total;
        unsigned long long reads = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int r = 2 * tid + q;
            begin[q] = end[q] = parts[q] = 0u;
            if (r >= rows) continue;
            const uint32_t at = off[r], m = off[r + 1] - at, window = at / JOB_KEYS;
            if (m > (uint32_t)BK_CAP) {
                const uint32_t aim = m <= (uint32_t)HUB_LONG ? HUB_PART : BK_AIM;
                parts[q] = (m + aim - 1) / aim;
                reads += (unsigned long long)parts[q] * m;
            } else if (m > (uint32_t)JOB_KEYS) {
                parts[q] = 1u;
            }
            if (r == 0 || off[r - 1] / JOB_KEYS != window) {
                int x = r, y = rows;                       // x begins in this window, y (or the end) does not
                while (y - x > 1) {
                    const int mid = (x + y) >> 1;
                    if (off[mid] / JOB_KEYS == window) x = mid; else y = mid;
                }
                begin[q] = at;
                end[q] = off[x + 1] - off[x] > (uint32_t)JOB_KEYS ? off[x] : off[x + 1];
            }
            jobs += parts[q] + (end[q] > begin[q] ? 1u : 0u);
        }
        const uint32_t mine = block_scan<BK_WAVES>(jobs, wave_sum, total);
        if (tid == 0) fill = atomicAdd(s.n_jobs, total);
        if (reads) atomicAdd(&s.totals[4], reads);
        __syncthreads();
        uint4* job = s.jobs + fill + mine;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int r = 2 * tid + q;
            if (end[q] > begin[q]) *job++ = make_uint4((uint32_t)dir << 31 | JOB_ROWS, 0u, lo + begin[q], end[q] - begin[q]);
            if (parts[q] == 0) continue;
            const uint32_t at = off[r], m = off[r + 1] - at;
            if (m <= (uint32_t)BK_CAP) *job++ = make_uint4((uint32_t)dir << 31 | JOB_ROWS, 0u, lo + at, m);
            else
                for (uint32_t x = 0; x < parts[q]; ++x)
                    *job++ = make_uint4((uint32_t)dir << 31 | (uint32_t)(n * x / parts[q]), (uint32_t)(n * (x + 1) / parts[q]), lo + at, m);
        }
        return;
    }

    for (int ra = 0; ra < rows;) {                         // (all of it uniform) the next rows that fit
        const uint32_t base = off[ra];
        int rb = rows;
        if (count - base > (uint32_t)BK_CAP) {
            int x = ra, y = rows;                          // off[x] - base <= BK_CAP < off[y] - base
            while (y - x > 1) {
                const int mid = (x + y) >> 1;
                if (off[mid] - base <= (uint32_t)BK_CAP) x = mid; else y = mid;
            }
            rb = x;
        }
        const bool hub = rb == ra;
        if (hub) rb = ra + 1;
        const uint32_t m = off[rb] - base;
        if (m == 0) { ra = rb; continue; }                 // empty rows, before a hub or at the end
        const int per = (int)((m + BK_THREADS - 1) / BK_THREADS);
        if (!whole) {                                      // those rows' keys among the bucket's
            if (tid == 0) fill = 0u;
            __syncthreads();
            each_key(in, count, [&](bool on, uint32_t key) {
                const uint32_t r = key >> p.id_bits;
                const bool mine = on && r >= (uint32_t)ra && r < (uint32_t)rb;
                const unsigned long long who = __ballot(mine);
                if (!who) return;
                const int lead = __ffsll(who) - 1;
                uint32_t at = 0;
                if (lane == lead) at = atomicAdd(&fill, (uint32_t)__popcll(who));
                at = __shfl(at, lead, 64) + __popcll(who & ((1ull << lane) - 1ull));
                if (mine) {
                    if (hub) to[base + at] = key;
                    else buf[at] = key;
                }
            });
            __syncthreads();
            if (hub) {
                const uint32_t parts = (m + HUB_PART - 1) / HUB_PART;      // (at most BK_ALONE keys: no strain on hubs_most)
                if (tid == 0) fill = atomicAdd(s.n_jobs, parts);
                __syncthreads();
                for (uint32_t q = tid; q < parts; q += BK_THREADS)
                    s.jobs[fill + q] = make_uint4((uint32_t)dir << 31 | (uint32_t)(n * q / parts), (uint32_t)(n * (q + 1) / parts), lo + base, m);
                __syncthreads();
                ra = rb;
                continue;
            }
            fetch(buf, m, per);
        }
        if (!whole) {
            uint32_t lg[2], parts = 0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int r = 2 * tid + q;
                const uint32_t d = r >= ra && r < rb ? off[r + 1] - off[r] : 0u;
                lg[q] = ranges_log(d);
                parts += d ? 1u << lg[q] : 0u;
            }
            uint32_t at = block_scan<BK_WAVES>(parts, wave_sum, n_sub);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int r = 2 * tid + q;
                if (r >= ra && r < rb) {
                    sub_of[r] = at << 5 | ((uint32_t)p.id_bits - lg[q]);
                    at += off[r + 1] > off[r] ? 1u << lg[q] : 0u;
                }
            }
            for (uint32_t i = tid; i < n_sub; i += BK_THREADS) u.sub[i] = 0u;
            __syncthreads();
        }
        auto range = [&](uint32_t key) {
            const uint32_t x = sub_of[key >> p.id_bits];
            return (x >> 5) + ((key & id_mask) >> (x & 31u));
        };
        uint32_t arrived[BK_PER];
#pragma unroll
        for (int i = 0; i < BK_PER; ++i)
            if (on(i, m, per)) arrived[i] = atomicAdd(&u.sub[range(k[i])], 1u);
        __syncthreads();
        static_assert(BK_SUBS == 4 * BK_THREADS, "four ranges a thread: one access of LDS");
        uint4 c = *reinterpret_cast<const uint4*>(&u.sub[4 * tid]);
        c.x = 4 * tid < n_sub ? c.x : 0u; c.y = 4 * tid + 1 < n_sub ? c.y : 0u;
        c.z = 4 * tid + 2 < n_sub ? c.z : 0u; c.w = 4 * tid + 3 < n_sub ? c.w : 0u;
        const uint32_t most = max(max(c.x, c.y), max(c.z, c.w));
        uint32_t total;
        const bool crowded = __syncthreads_or(most > (uint32_t)BK_SUB_MAX) != 0;
        if (crowded) {
            radix_sort(k, per, p.row_bits + p.id_bits, buf, u.radix);
            for (uint32_t i = tid; i < m; i += BK_THREADS) out.idx[dir][lo + base + i] = (int32_t)(buf[i] & id_mask);
        } else {
            const uint32_t at = block_scan<BK_WAVES>((c.x + c.y) + (c.z + c.w), wave_sum, total);
            *reinterpret_cast<uint4*>(&u.sub[4 * tid]) = make_uint4(at, at + c.x, at + c.x + c.y, at + c.x + c.y + c.z);
            if (tid == BK_THREADS - 1) u.sub[BK_SUBS] = m;
            if (tid < 3 && m + tid < (uint32_t)BK_CAP) buf[m + tid] = ~0u;       // (the last four that are read together)
            __syncthreads();
#pragma unroll
            for (int i = 0; i < BK_PER; ++i)
                if (on(i, m, per)) buf[u.sub[range(k[i])] + arrived[i]] = k[i];
            __syncthreads();
            // A key's place: behind the smaller ones, and behind its equals that stand before it.  Four keys at a time, whole aligned groups: what
            // stands before the range is smaller, what stands behind it larger.
            for (uint32_t i = tid; i < m; i += BK_THREADS) {
                const uint32_t key = buf[i], g = range(key), j0 = u.sub[g] & ~3u, j1 = u.sub[g + 1];
                uint32_t at_key = j0;
#pragma unroll 1
                for (uint32_t j = j0; j < j1; j += 4) {
                    const uint4 o = *reinterpret_cast<const uint4*>(&buf[j]);
                    at_key += (o.x < key || (o.x == key && j < i)) + (o.y < key || (o.y == key && j + 1 < i)) +
                              (o.z < key || (o.z == key && j + 2 < i)) + (o.w < key || (o.w == key && j + 3 < i));
                }
                out.idx[dir][lo + base + at_key] = (int32_t)(key & id_mask);
            }
        }
        __syncthreads();                                   // buf is filled anew
        ra = rb;
    }
}

// The first JOB_GROUPS workgroups take the jobs of crowded buckets (a chain of several memory latencies, so they start first): a range of
// rows is sorted in LDS; so are the keys of a hub that lie in one range of ids or, where they do not fit, they are counted id by id,
// HUB_SPAN ids at a time.  The others list their bucket's long rows and their chunks, in row order (as long_rows_emit_kernel does).
__global__ __launch_bounds__(BK_THREADS) void bucket_finish_kernel(int64_t nnz, int64_t n, BucketPlan p, BucketScratch s, BucketOut out,
                                                                   const uint32_t* __restrict__ by_row) {
    static_assert(HUB_SPAN == BK_CAP, "one array for both");
    __shared__ uint32_t buf[BK_CAP];
    __shared__ RadixLds radix;
    __shared__ uint32_t fill;
    __shared__ unsigned long long wave_sum64[BK_WAVES];
    __shared__ uint32_t wave_sum[BK_WAVES];
    const int B = p.n_buckets, tid = threadIdx.x;
    if (s.totals[4] > s.hubs_most) return;                 // refused
    if ((int)blockIdx.x >= JOB_GROUPS) {
        const int at_b = (int)blockIdx.x - JOB_GROUPS, dir = at_b >= B, b = at_b - dir * B;
        if (!out.long_row[dir]) {
            if (b == 0 && tid < 2) s.totals[2 * dir + tid] = 0ull;
            return;
        }
        const unsigned long long own = s.longs[dir * B + b];
        if (own == 0 && b != B - 1) return;
        unsigned long long before = 0, edges = 0, all, all_edges = 0;
        for (int i = tid; i <= b; i += BK_THREADS) {
            if (i < b) before += s.longs[dir * B + i];
            edges += s.edges[dir * B + i];
        }
        (void)block_scan<BK_WAVES>(before, wave_sum64, all);
        before = all;
        if (b == B - 1) {                                  // (uniform)
            (void)block_scan<BK_WAVES>(edges, wave_sum64, all_edges);
            if (tid == 0) {
                s.totals[2 * dir] = before + own;
                s.totals[2 * dir + 1] = all_edges;
                out.long_first[dir][(before + own) >> 32] = (int32_t)((before + own) & 0xFFFFFFFFull);
            }
        }
        if (own == 0) return;
        const int64_t first = (int64_t)b << p.row_bits;
        const int64_t* const ptr = out.ptr[dir];
        int64_t at[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int64_t r = first + 2 * tid + q;
            const int64_t end = first + ((int64_t)1 << p.row_bits) < n ? first + ((int64_t)1 << p.row_bits) : n;
            at[q] = ptr[r < end ? r : end];
        }
        unsigned long long mine[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t len = at[q + 1] - at[q];
            mine[q] = len > SPMM_LONG_ROW ? (1ull << 32) + (unsigned long long)((len + SPMM_CHUNK - 1) / SPMM_CHUNK) : 0ull;
        }
        unsigned long long slot = before + block_scan<BK_WAVES>(mine[0] + mine[1], wave_sum64, all);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (mine[q]) {
                int64_t c = (int64_t)(slot & 0xFFFFFFFFull);
                out.long_row[dir][slot >> 32] = (int32_t)(first + 2 * tid + q);
                out.long_first[dir][slot >> 32] = (int32_t)c;
                for (int64_t e = at[q]; e < at[q + 1]; e += SPMM_CHUNK, ++c) {
                    out.chunk_begin[dir][c] = e;
                    out.chunk_end[dir][c] = e + SPMM_CHUNK < at[q + 1] ? e + SPMM_CHUNK : at[q + 1];
                }
            }
            slot += mine[q];
        }
        return;
    }
    const uint32_t jobs = *s.n_jobs, id_mask = p.id_bits == 32 ? ~0u : (1u << p.id_bits) - 1u;
    const int lane = tid & 63, wave = tid >> 6;
    for (uint32_t job = blockIdx.x; job < jobs; job += JOB_GROUPS) {
        const uint4 h = s.jobs[job];
        const int dir = (int)(h.x >> 31);
        const bool whole_rows = (h.x & JOB_ROWS) != 0;
        const uint32_t id0 = h.x & (JOB_ROWS - 1u), id1 = h.y;
        const uint32_t* const in = by_row + dir * nnz + h.z;
        uint32_t m = h.w, below = 0, all_below = 0;
        if (!whole_rows) {
            if (tid == 0) fill = 0u;
            __syncthreads();
            each_key(in, h.w, [&](bool on, uint32_t key) {
                const uint32_t id = key & id_mask;
                below += on && id < id0 ? 1u : 0u;
                const bool mine = on && id >= id0 && id < id1;
                const unsigned long long who = __ballot(mine);
                if (!who) return;
                const int lead = __ffsll(who) - 1;
                uint32_t at = 0;
                if (lane == lead) at = atomicAdd(&fill, (uint32_t)__popcll(who));
                at = __shfl(at, lead, 64) + __popcll(who & ((1ull << lane) - 1ull));
                if (mine && at < (uint32_t)BK_CAP) buf[at] = id;
            });
            (void)block_scan<BK_WAVES>(below, wave_sum, all_below);
            m = fill;                                      // (block_scan's barriers are between)
        }
        int32_t* o = out.idx[dir] + h.z + all_below;
        if (m <= (uint32_t)BK_CAP) {
            uint32_t k[BK_PER];
            const int per = (int)((m + BK_THREADS - 1) / BK_THREADS);
#pragma unroll
            for (int i = 0; i < BK_PER; ++i) {
                const uint32_t at = (uint32_t)((wave * per + i) * 64 + lane);
                k[i] = i < per && at < m ? (whole_rows ? in[at] : buf[at]) : ~0u;
            }
            radix_sort(k, per, whole_rows ? p.row_bits + p.id_bits : p.id_bits, buf, radix);
            for (uint32_t i = tid; i < m; i += BK_THREADS) o[i] = (int32_t)(buf[i] & id_mask);
            __syncthreads();
            continue;
        }
        constexpr int PER = HUB_SPAN / BK_THREADS;
        for (uint32_t a = id0; a < id1; a += HUB_SPAN) {
            const uint32_t z = a + HUB_SPAN < id1 ? a + HUB_SPAN : id1;
            __syncthreads();
            for (int i = tid; i < HUB_SPAN; i += BK_THREADS) buf[i] = 0u;
            __syncthreads();
            each_key(in, h.w, [&](bool on, uint32_t key) {
                const uint32_t id = key & id_mask;
                if (on && id >= a && id < z) atomicAdd(&buf[id - a], 1u);
            });
            __syncthreads();
            uint32_t sum = 0, total;
            for (int i = 0; i < PER; ++i) sum += buf[tid * PER + i];
            uint32_t at = block_scan<BK_WAVES>(sum, wave_sum, total);
            for (int i = 0; i < PER; ++i)
                for (uint32_t c = buf[tid * PER + i]; c > 0; --c) o[at++] = (int32_t)(a + tid * PER + i);
            o += total;
        }
        __syncthreads();
    }
}

// The 64-bit keys again, from the CSR's packed ones.
__global__ __launch_bounds__(256) void bucket_unpack_kernel(const uint32_t* __restrict__ packed, int64_t nnz, BucketPlan p,
                                                            const uint32_t* __restrict__ start /*[B + 1]*/, uint64_t* __restrict__ keys) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= nnz) return;
    int x = 0, y = p.n_buckets;                            // start[x] <= e < start[y]
    while (y - x > 1) {
        const int mid = (x + y) >> 1;
        if ((int64_t)start[mid] <= e) x = mid; else y = mid;
    }
    const uint32_t k = packed[e], id_mask = p.id_bits == 32 ? ~0u : (1u << p.id_bits) - 1u;
    keys[e] = (uint64_t)(((uint32_t)x << p.row_bits) + (k >> p.id_bits)) << 32 | (uint64_t)(k & id_mask);
}

// keys: nnz of them, clobbered; packed: scratch of the same size; scratch: bucket_scratch_bytes.  Fills the handle's CSR, CSC and
// degrees and the lists of its long rows (arrays of the worst case's size, or null where no row can be long); waits for the lists'
// lengths.  long_edges: the edges of each direction's long rows.  *done = false: the build was refused, keys holds them again.
// csc_alone: the keys are source << 32 | destination, and the CSC is all that is filled (as the first direction of what is below); keys of a
// refused build are lost (its caller makes them anew, a range at a time).
grp_status bucket_build(grp_partition_t* h, const BucketPlan& p, uint64_t* keys, uint64_t* packed, void* scratch, int64_t (&long_edges)[2],
                        bool* done, hipStream_t st, bool csc_alone) {
    const int64_t n = h->n, nnz = h->nnz;
    const BucketScratch s = carve_scratch(p, nnz, scratch);
    const int dirs = csc_alone ? 1 : 2;
    LongRows* const lr[2] = {csc_alone ? &h->csc_long : &h->csr_long, &h->csc_long};
    const BucketOut out{{csc_alone ? h->colptr : h->rowptr, h->colptr}, {csc_alone ? h->row : h->col, h->row},
                        {csc_alone ? h->d_local_out : h->d_local_in, h->d_local_out}, {lr[0]->long_row, lr[1]->long_row},
                        {lr[0]->long_first, lr[1]->long_first}, {lr[0]->chunk_begin, lr[1]->chunk_begin}, {lr[0]->chunk_end, lr[1]->chunk_end}};
    const size_t hist_bytes = 2 * (size_t)p.n_buckets * sizeof(uint32_t);
    GRP_TRY(launch_fill_zero(s.totals, s.clear_bytes, st));
    const int64_t count_groups = cdiv(nnz, 8 * BK_THREADS);
    hipLaunchKernelGGL(bucket_count_kernel, dim3((unsigned)(count_groups < 512 ? count_groups : 512)), dim3(BK_THREADS), hist_bytes, st, keys, nnz,
                       p, dirs, s.count);
    hipLaunchKernelGGL(bucket_start_kernel, dim3(1), dim3(BK_THREADS), 0, st, s, p.n_buckets);
    // Long tiles make long runs in the buckets, short ones more workgroups.
    const int per = (int)(nnz >= (int64_t)256 * SC_TILE ? SC_PER : nnz <= (int64_t)256 * 4 * BK_THREADS ? 4 : cdiv(nnz, 256 * BK_THREADS));
    const size_t scatter_bytes = hist_bytes / 2 * 3 + (size_t)per * BK_THREADS * 6;
    hipLaunchKernelGGL(bucket_scatter_kernel, dim3((unsigned)cdiv(nnz, per * BK_THREADS)), dim3(BK_THREADS), scatter_bytes, st, keys, nnz, p, dirs, per,
                       (const unsigned long long*)(s.totals + 4), s.cursor, (uint32_t*)packed);
    GRP_LAUNCH_CHECK();
    hipLaunchKernelGGL(bucket_sort_kernel, dim3(dirs * p.n_buckets), dim3(BK_THREADS), 0, st, (const uint32_t*)packed, nnz, n, p, s, out, (uint32_t*)keys);
    hipLaunchKernelGGL(bucket_finish_kernel, dim3(dirs * p.n_buckets + JOB_GROUPS), dim3(BK_THREADS), 0, st, nnz, n, p, s, out, (const uint32_t*)keys);
    GRP_LAUNCH_CHECK();
    unsigned long long totals[5];
    GRP_HIP(hipMemcpyAsync(totals, s.totals, sizeof totals, hipMemcpyDeviceToHost, st));
    GRP_HIP(hipStreamSynchronize(st));
    *done = totals[4] <= s.hubs_most;
    if (!*done) {
        if (csc_alone || totals[4] == REFUSED_AT_ONCE) return GRP_OK;      // (keys are untouched if refused at once)
        hipLaunchKernelGGL(bucket_unpack_kernel, dim3((unsigned)cdiv(nnz, 256)), dim3(256), 0, st, (const uint32_t*)packed, nnz, p, (const uint32_t*)s.start,
                           keys);
        GRP_LAUNCH_CHECK();
        return GRP_OK;
    }
    for (int d = 0; d < dirs; ++d) {
        lr[d]->n_long = (int32_t)(totals[2 * d] >> 32);
        lr[d]->n_chunks = (int32_t)(totals[2 * d] & 0xFFFFFFFFull);
        long_edges[csc_alone ? 1 : d] = (int64_t)totals[2 * d + 1];
    }
    return GRP_OK;
}

}  // namespace grp
