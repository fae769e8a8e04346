// Random node assignment and the isolated local subgraph, built on the GPU.
//
// owner(v) = SplitMix64_output(seed, v) mod K.  A partition keeps the edges whose two
// endpoints it owns, renumbers nodes by ascending global id and stores the edge multiset
// twice in canonical order: CSR by destination (sources ascending) and CSC by source
// (destinations ascending).  Canonical order comes from a sort of the 64-bit keys (row << 32 | column): by buckets of rows
// (buckets.hip), or a device-wide radix sort where weights travel with the keys, there are more than 2^22 nodes or 2^26
// edges, or a few rows hold most of them.  Equal keys are indistinguishable, so the arrays are unique and can
// be compared bit for bit.  Everything is integer work: counters use integer atomics only.
//
// The device-wide radix sort and prefix sum are rocPRIM's; the hashing, filtering,
// relabelling and pointer construction are the kernels below.
#include "common.h"

#include <cstring>
#include <new>
#include <vector>

#include <rocprim/rocprim.hpp>

namespace grp {

__device__ __forceinline__ uint64_t splitmix64_output(uint64_t seed, uint64_t index) {
    uint64_t z = seed + (index + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// splitmix64_output(seed, v) mod K == part, without a division: K = 2^rot * odd divides z - part exactly if the product with the
// inverse of odd (mod 2^64), rotated right by rot, does not exceed (2^64 - 1) / K (Granlund and Montgomery, "Division by invariant
// integers using multiplication", 1994, section 9).
struct OwnerTest {
    uint64_t seed, inv, limit;
    uint32_t part;
    int rot;
    // POW2: K = 2^rot, whose remainder is the low bits
    template <bool POW2 = false> __device__ __forceinline__ bool owns(uint64_t v) const {
        const uint64_t z = splitmix64_output(seed, v);
        if (POW2) return ((uint32_t)z & ((1u << rot) - 1u)) == part;
        uint64_t q = (z - part) * inv;
        q = (q >> rot) | (q << ((64 - rot) & 63));
        return z >= part && q <= limit;
    }
    __device__ __forceinline__ bool operator()(int64_t v) const { return owns((uint64_t)v); }
};
static OwnerTest owner_test(uint64_t seed, uint32_t K, uint32_t part) {
    OwnerTest t{seed, 1, ~0ull / K, part, 0};
    uint64_t odd = K;
    while ((odd & 1) == 0) { odd >>= 1; ++t.rot; }
    for (int i = 0; i < 6; ++i) t.inv *= 2 - odd * t.inv;       // Newton: twice the bits each time
    return t;
}

// owner[v] for every node and (optionally) the number of nodes per partition.
__global__ __launch_bounds__(256) void node_owners_kernel(int64_t N, uint32_t K, uint64_t seed, int32_t* __restrict__ owner,
                                                          unsigned long long* __restrict__ hist) {
    constexpr int LDS_BINS = 1024;
    __shared__ unsigned int bins[LDS_BINS];
    const bool local = hist && K <= LDS_BINS;
    if (local) {
        for (int i = threadIdx.x; i < (int)K; i += 256) bins[i] = 0u;
        __syncthreads();
    }
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < N; v += (int64_t)gridDim.x * 256) {
        const uint32_t o = (uint32_t)(splitmix64_output(seed, (uint64_t)v) % K);
        owner[v] = (int32_t)o;
        if (local) atomicAdd(&bins[o], 1u);
        else if (hist) atomicAdd(&hist[o], 1ull);
    }
    if (local) {
        __syncthreads();
        for (int i = threadIdx.x; i < (int)K; i += 256)
            if (bins[i]) atomicAdd(&hist[i], (unsigned long long)bins[i]);
    }
}

// Edges e and e + 1 (e even) of an id array with one 16-byte load when the array allows it; `fill` past the end.
typedef int64_t i64x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void load_edge_pair(const int64_t* __restrict__ p, int64_t e, int64_t E, bool vec, int64_t fill,
                                               int64_t& a, int64_t& b) {
    if (vec && e + 1 < E) {
        const i64x2 t = *reinterpret_cast<const i64x2*>(p + e);
        a = t.x;
        b = t.y;
    } else {
        a = e < E ? p[e] : fill;
        b = e + 1 < E ? p[e + 1] : fill;
    }
}

// A node set as a bitmap, every 32-node word beside the number of members before it: membership and the
// member's rank (its local id) from one small array that stays in the L2 caches (N / 4 bytes in all),
// where per-node flag and position arrays (12 bytes per node) cost a cache line from HBM per lookup.  What a lookup costs is its line's
// way from the L2, so a word and its count lie together.
struct NodeSet {
    const uint2* words;                  // bits, members before
};
// The words of the set of the nodes v < N that member(v) holds for, and one empty word after the last; the grid covers their nodes.
template <typename Member>
__global__ __launch_bounds__(256) void node_bits_kernel(int64_t N, int64_t n_words, Member member, uint32_t* __restrict__ bits) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const unsigned long long m = __ballot(v < N && member(v));
    const int64_t w = v >> 5;
    if ((threadIdx.x & 31) == 0 && w <= n_words) bits[w] = (uint32_t)(m >> (threadIdx.x & 32));
}
__global__ __launch_bounds__(256) void count_bits_kernel(const uint32_t* __restrict__ bits, int64_t n_words, unsigned long long* __restrict__ count) {
    unsigned long long c = 0;
    for (int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x; w < n_words; w += (int64_t)gridDim.x * 256) c += __popc(bits[w]);
    for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(count, c);
}
__device__ __forceinline__ bool word_has(const uint2& w, int64_t v) { return (w.x >> (v & 31)) & 1u; }
__device__ __forceinline__ int32_t word_rank(const uint2& w, int64_t v) { return (int32_t)w.y + __popc(w.x & ((1u << (v & 31)) - 1u)); }
__device__ __forceinline__ bool set_has(const NodeSet& s, int64_t v) { return word_has(s.words[v >> 5], v); }
__device__ __forceinline__ int32_t set_rank(const NodeSet& s, int64_t v) { return word_rank(s.words[v >> 5], v); }

// Node v's word, which its first node also puts into the set.
__device__ __forceinline__ uint2 set_word(const uint32_t* __restrict__ bits, const int32_t* __restrict__ before, int64_t v,
                                          uint2* __restrict__ words) {
    const uint2 w = make_uint2(bits[v >> 5], (uint32_t)before[v >> 5]);
    if ((v & 31) == 0) words[v >> 5] = w;
    return w;
}
__global__ __launch_bounds__(256) void set_nodes_kernel(int64_t N, const uint32_t* __restrict__ bits, const int32_t* __restrict__ before,
                                                        uint2* __restrict__ words, int64_t* __restrict__ l2g) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= N) return;
    const uint2 w = set_word(bits, before, v, words);
    if (word_has(w, v)) l2g[word_rank(w, v)] = v;
}

// ---- weighted partitions: the selected edges are compacted in edge-list order, so that equal
// (dst, src) pairs keep their order through the stable sorts and the result does not depend on
// scheduling.  A tile is 2048 consecutive edges, eight consecutive edges per thread; a first pass counts
// the selected edges of every tile, a prefix sum over the tiles gives each its first slot, a second pass
// repeats the selection and places every edge at the tile's slot plus its rank inside the tile.
// WHICH = 0: edges with both endpoints in the set; WHICH = 1: edges whose destination is in the set.
constexpr int OC_PER = 8;
constexpr int OC_TILE = 256 * OC_PER;

template <int WHICH>
__device__ __forceinline__ int oc_select(const int64_t* __restrict__ src, const int64_t* __restrict__ dst, int64_t E,
                                         bool vec, const NodeSet& own, int64_t e0, int64_t (&us)[OC_PER],
                                         int64_t (&vs)[OC_PER], bool (&on)[OC_PER]) {
#pragma unroll
    for (int i = 0; i < OC_PER; i += 2) {
        load_edge_pair(src, e0 + i, E, vec, 0, us[i], us[i + 1]);
        load_edge_pair(dst, e0 + i, E, vec, -1, vs[i], vs[i + 1]);       // -1: past the end
    }
    int count = 0;
#pragma unroll
    for (int i = 0; i < OC_PER; ++i) {
        on[i] = vs[i] >= 0 && set_has(own, vs[i]) && (WHICH == 1 || set_has(own, us[i]));
        count += on[i] ? 1 : 0;
    }
    return count;
}

template <int WHICH>
__global__ __launch_bounds__(256) void ordered_count_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                            int64_t E, NodeSet own, int64_t n_tiles,
                                                            int64_t* __restrict__ tile_count /*[n_tiles + 1]*/) {
    __shared__ int wave_count[4];
    const bool vec = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        int64_t us[OC_PER], vs[OC_PER];
        bool on[OC_PER];
        int c = oc_select<WHICH>(src, dst, E, vec, own, tile * OC_TILE + (int64_t)threadIdx.x * OC_PER, us, vs, on);
        for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
        if (lane == 0) wave_count[wave] = c;
        __syncthreads();
        if (threadIdx.x == 0) tile_count[tile] = wave_count[0] + wave_count[1] + wave_count[2] + wave_count[3];
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) tile_count[n_tiles] = 0;
}

template <int WHICH>
__global__ __launch_bounds__(256) void ordered_emit_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                           const float* __restrict__ w, int64_t E, NodeSet own,
                                                           int64_t n_tiles, const int64_t* __restrict__ tile_base,
                                                           uint64_t* __restrict__ keys, uint32_t* __restrict__ keys32,
                                                           float* __restrict__ vals) {
    __shared__ int wave_count[4];
    const bool vec = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t e0 = tile * OC_TILE + (int64_t)threadIdx.x * OC_PER;
        int64_t us[OC_PER], vs[OC_PER];
        bool on[OC_PER];
        const int mine = oc_select<WHICH>(src, dst, E, vec, own, e0, us, vs, on);
        int incl = mine;                                 // inclusive prefix over the wavefront, then over the four
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wave_count[wave] = incl;
        __syncthreads();
        int before = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q < wave) before += wave_count[q];
        int64_t slot = tile_base[tile] + before + incl - mine;
#pragma unroll
        for (int i = 0; i < OC_PER; ++i) {
            if (!on[i]) continue;
            if (WHICH == 0) keys[slot] = ((uint64_t)(uint32_t)set_rank(own, vs[i]) << 32) | (uint64_t)(uint32_t)set_rank(own, us[i]);
            else keys32[slot] = (uint32_t)set_rank(own, vs[i]);
            vals[slot] = w[e0 + i];
            ++slot;
        }
        __syncthreads();                                 // wave_count is reused by the next tile
    }
}

// Pass 1 over the edges: id range check, global in-degree of owned destinations, count of kept edges.
// The in-degree counts go through a table in LDS first (open addressing on the local id, a few probes,
// LDS atomics) and reach memory once per workgroup and node: a hub of a skewed graph receives 10^5..10^6
// edges, and that many atomics on one address serialise in the L2 (they set the time of this pass before).
// An edge that finds no slot adds to memory directly.
constexpr int DG_SLOTS = 4096;
constexpr int DG_PROBES = 4;
constexpr int EDGE_SCAN_GRID = 4096;      // fat workgroups: more edges of a hub meet in one table

__device__ __forceinline__ void dg_table_add(int32_t* slot_key, uint32_t* slot_count, unsigned long long* __restrict__ dg,
                                             int32_t r) {
    uint32_t h = (uint32_t)r * 2654435761u >> 20;        // top 12 bits of a multiplicative hash
    for (int probe = 0; probe < DG_PROBES; ++probe, h = (h + 1) & (DG_SLOTS - 1)) {
        const int32_t seen = atomicCAS(&slot_key[h], -1, r);
        if (seen == -1 || seen == r) {
            atomicAdd(&slot_count[h], 1u);
            return;
        }
    }
    atomicAdd(&dg[r], 1ull);
}

// KEYS: the keys of the kept edges too, into a buffer of `cap` of them (as edge_scan_keys_kernel does).  counters: [1] += bad ids,
// and += kept edges to [2], the slot cursor, or else [0].
template <bool KEYS>
__global__ __launch_bounds__(256) void edge_scan_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                        int64_t E, int64_t N, NodeSet own,
                                                        unsigned long long* __restrict__ dg,
                                                        unsigned long long* __restrict__ counters,
                                                        uint64_t* __restrict__ keys, unsigned long long cap) {
    const bool vec = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    __shared__ int32_t slot_key[DG_SLOTS];
    __shared__ uint32_t slot_count[DG_SLOTS];
    __shared__ uint32_t wave_sum[4];
    __shared__ unsigned long long tile_base;
    for (int i = threadIdx.x; i < DG_SLOTS; i += 256) { slot_key[i] = -1; slot_count[i] = 0u; }
    __syncthreads();
    unsigned long long kept = 0, bad = 0;
    constexpr int PER = 8;                               // edges per thread and tile: their loads are in flight together
    const int64_t n_tiles = (E + 256 * PER - 1) / (256 * PER);
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t e0 = tile * (256 * PER) + 2 * threadIdx.x;
        int64_t us[PER], vs[PER];
#pragma unroll
        for (int i = 0; i < PER; i += 2) {               // a thread takes pairs of consecutive edges
            const int64_t e = e0 + (int64_t)i * 256;
            load_edge_pair(src, e, E, vec, 0, us[i], us[i + 1]);
            load_edge_pair(dst, e, E, vec, -1, vs[i], vs[i + 1]);     // past the end: out of range, and looked at again below
        }
        // Eight edges' lookups are requested together, in two stages; a lane that has no need of one reads word 0 (one line for all of
        // them).
        uint2 wv[PER], wu[PER];
        bool odd = false;                                // an id out of range, or no edge
        uint32_t has = 0, both = 0;                      // bit i: the destination, and also the source, of edge i is in the set
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const bool ok = us[i] >= 0 && vs[i] >= 0 && us[i] < N && vs[i] < N;
            odd = odd || !ok;
            if (!ok) us[i] = vs[i] = 0;
            wv[i] = own.words[vs[i] >> 5];
            has |= (ok ? 1u : 0u) << i;
        }
        if (__any(odd))                                  // (read again, by place, as an id may have any value; counted with the others 595 -> 628 us, 62e6 edges)
            for (int i = 0; i < PER; ++i) {
                const int64_t e = e0 + (i & ~1) * 256 + (i & 1);
                bad += e < E && !(src[e] >= 0 && dst[e] >= 0 && src[e] < N && dst[e] < N);
            }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (!word_has(wv[i], vs[i])) has &= ~(1u << i);
            wu[i] = own.words[(has >> i) & 1u ? us[i] >> 5 : 0];
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (!((has >> i) & 1u)) continue;
            dg_table_add(slot_key, slot_count, dg, word_rank(wv[i], vs[i]));
            if (word_has(wu[i], us[i])) both |= 1u << i;
        }
        if (KEYS) {
            uint32_t total;
            const uint32_t before = block_scan<4>((uint32_t)__popc(both), wave_sum, total);
            if (threadIdx.x == 0) tile_base = total ? atomicAdd(&counters[2], (unsigned long long)total) : 0ull;
            __syncthreads();
            unsigned long long slot = tile_base + before;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (!((both >> i) & 1u)) continue;
                if (slot < cap) keys[slot] = ((uint64_t)(uint32_t)word_rank(wv[i], vs[i]) << 32) | (uint64_t)(uint32_t)word_rank(wu[i], us[i]);
                ++slot;
            }
            // (tile_base is written anew behind the next tile's barriers, which every thread reaches with its base read)
        } else {
            kept += (unsigned long long)__popc(both);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < DG_SLOTS; i += 256)
        if (slot_key[i] >= 0) atomicAdd(&dg[slot_key[i]], (unsigned long long)slot_count[i]);
    for (int o = 32; o > 0; o >>= 1) {
        kept += __shfl_down(kept, o, 64);
        bad += __shfl_down(bad, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        if (kept) atomicAdd(&counters[0], kept);
        if (bad) atomicAdd(&counters[1], bad);
    }
}

// Which edges a partition keeps and their key (dst_local << 32 | src_local).
struct SetSelect {                        // both endpoints in the node set
    NodeSet own;
    __device__ __forceinline__ bool operator()(int64_t u, int64_t v, uint64_t& key) const {
        if (!set_has(own, v) || !set_has(own, u)) return false;
        key = ((uint64_t)(uint32_t)set_rank(own, v) << 32) | (uint64_t)(uint32_t)set_rank(own, u);
        return true;
    }
};
struct HaloSelect {                       // destination in `inner`, a part of the set; its source then is in the set
    NodeSet own;
    const uint32_t* inner;
    __device__ __forceinline__ bool operator()(int64_t u, int64_t v, uint64_t& key) const {
        if (!((inner[v >> 5] >> (v & 31)) & 1u)) return false;
        key = ((uint64_t)(uint32_t)set_rank(own, v) << 32) | (uint64_t)(uint32_t)set_rank(own, u);
        return true;
    }
};

// Pass 2: write the key of every kept edge.  The slot order is
// arbitrary; the sort that follows makes the result canonical.  A workgroup takes tiles of
// 256 x 8 edges, counts its kept edges through LDS and reserves their slots with one atomic
// per tile (one atomic per kept edge on a single address would serialise the whole pass).
template <typename Select>
__global__ __launch_bounds__(256) void edge_keys_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                        int64_t E, Select select,
                                                        unsigned long long* __restrict__ cursor,
                                                        uint64_t* __restrict__ keys) {
    constexpr int PER = 8;
    const bool vec = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    __shared__ int wave_count[4];
    __shared__ unsigned long long tile_base;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n_tiles = (E + 256 * PER - 1) / (256 * PER);
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t e0 = tile * (256 * PER) + 2 * tid;
        int64_t us[PER], vs[PER];
#pragma unroll
        for (int i = 0; i < PER; i += 2) {               // a thread takes pairs of consecutive edges
            const int64_t e = e0 + (int64_t)i * 256;
            load_edge_pair(src, e, E, vec, 0, us[i], us[i + 1]);
            load_edge_pair(dst, e, E, vec, -1, vs[i], vs[i + 1]);     // -1: past the end
        }
        uint64_t key[PER];
        int mine = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            key[i] = ~0ull;
            uint64_t k;
            if (vs[i] >= 0 && select(us[i], vs[i], k)) { key[i] = k; ++mine; }
        }
        // exclusive prefix of `mine` over the workgroup: inside the wavefront by shuffles, across the four by LDS
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wave_count[wave] = incl;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) before += wave_count[w];
            total += wave_count[w];
        }
        if (tid == 0) tile_base = total ? atomicAdd(cursor, (unsigned long long)total) : 0ull;
        __syncthreads();
        unsigned long long slot = tile_base + (unsigned long long)(before + incl - mine);
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (key[i] != ~0ull) keys[slot++] = key[i];
        __syncthreads();                                 // wave_count / tile_base are reused by the next tile
    }
}

// Both passes in one (unweighted builds): range check, the keys of the kept edges, written into a buffer of `cap` keys, and the local
// ids of all owned destinations, from which rank_count_kernel counts the global in-degrees.  counters: [1] += bad ids, [2] += kept
// edges, [3] += local ids (the cursors).  If the kept edges end above cap the keys are incomplete and the caller runs
// edge_keys_kernel with a buffer of the exact size; local ids past id_cap are counted here, one by one.
// What sets the time is what is asked of the L2 beside the edges: a membership lookup per edge (a bitmap larger than the L1: a line
// each) and, worst, the in-degrees' additions, scattered words that are a request each even after a table in LDS (62e6
// edges, an eighth of the nodes: 547 us with either of a lookup and a computed membership).  So membership is computed, and a tile's ids
// leave in ranges of SPAN ids, as neighbouring words; counting a range takes LDS only.  Then it is the vector instructions (89 an edge and
// wavefront, 11 of them at a quarter of the rate, beside a read that alone would take 190 us): so remainders of a power of
// two are the low bits, bounds are checked on the halves of the ids, and the edges whose destination is owned are lined up in LDS before they
// are looked up, ranked and counted, instead of all eight of a lane's in turn with most lanes idle.  (62e6 edges, 8 parts: 286 -> 250 us.)
constexpr int SPAN_BITS = 14;            // 64 KB of counters
constexpr int SPANS_MAX = 256;           // ranges: partitions of up to 2^22 nodes
constexpr int SCAN_THREADS = 512;
constexpr int SCAN_PER = 8;              // edges per thread and tile: their loads are in flight together
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_PER;
constexpr int SCAN_GRID = 1536;
// Which edges are looked at (by their destination: its in-degree counts) and which of them are kept.
template <bool POW2> struct OwnedEdges {   // destination owned, which is computed; source owned too
    OwnerTest owned;
    static constexpr bool LOOKUP = false;
    static constexpr int WAVES = 5;          // a SIMD's (4: 492 us, 6: 500, some registers spilled)
};
struct HaloEdges {                         // destination in the set; destination in the set as it was before the last hop (its sources then are)
    const uint32_t* inner;
    static constexpr bool LOOKUP = true;
    static constexpr int WAVES = 4;          // (2e7 edges, 2.4e6 nodes, one hop: a build 807 us; 3: 847, 5: 1232, spilled)
};
template <bool POW2> __device__ __forceinline__ bool select_counted(const OwnedEdges<POW2>& s, uint32_t v) { return s.owned.template owns<POW2>(v); }
__device__ __forceinline__ bool select_counted(const HaloEdges&, uint32_t) { return true; }
template <bool POW2> __device__ __forceinline__ uint32_t select_inner(const OwnedEdges<POW2>&, uint32_t) { return 0u; }
__device__ __forceinline__ uint32_t select_inner(const HaloEdges& s, uint32_t word) { return s.inner[word]; }
template <typename Select>
__global__ __launch_bounds__(SCAN_THREADS, Select::WAVES) void edge_scan_keys_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst, int64_t E,
                                                                      uint32_t N, NodeSet own, Select select, int spans,
                                                                      unsigned long long* __restrict__ dg, unsigned long long* __restrict__ counters,
                                                                      uint64_t* __restrict__ keys, unsigned long long cap,
                                                                      uint32_t* __restrict__ ids, unsigned long long id_cap,
                                                                      uint32_t* __restrict__ heads /*[tiles][spans + 1]*/) {
    __shared__ union {
        uint2 line[SCAN_TILE];                               // (source, destination) of the edges in question, 64 * SCAN_PER places a wavefront
        uint32_t buf[SCAN_TILE];
    } sh;
    uint32_t* const buf = sh.buf;
    __shared__ uint32_t first[SPANS_MAX + 1];
    __shared__ uint32_t kept, id_total;
    __shared__ unsigned long long base[2];
    const bool vec = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    const int tid = threadIdx.x, lane = tid & 63;
    uint2* const line = sh.line + (tid >> 6) * (64 * SCAN_PER);
    unsigned long long bad = 0;
    const int64_t n_tiles = (E + SCAN_TILE - 1) / SCAN_TILE;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        for (int i = tid; i < spans; i += SCAN_THREADS) first[i] = 0u;
        if (tid == 0) kept = 0u;
        const int64_t e0 = tile * SCAN_TILE + 2 * tid;
        uint32_t here = 0;                                   // edges of the wavefront whose destination is owned
        {
            int64_t us[SCAN_PER], vs[SCAN_PER];
            if (vec && (tile + 1) * SCAN_TILE <= E) {        // (uniform)
#pragma unroll
                for (int i = 0; i < SCAN_PER; i += 2) {
                    const i64x2 a = *reinterpret_cast<const i64x2*>(src + e0 + (int64_t)i * SCAN_THREADS);
                    const i64x2 b = *reinterpret_cast<const i64x2*>(dst + e0 + (int64_t)i * SCAN_THREADS);
                    us[i] = a.x; us[i + 1] = a.y;
                    vs[i] = b.x; vs[i + 1] = b.y;
                }
            } else {
#pragma unroll
                for (int i = 0; i < SCAN_PER; i += 2) {
                    const int64_t e = e0 + (int64_t)i * SCAN_THREADS;
                    load_edge_pair(src, e, E, vec, 0, us[i], us[i + 1]);
                    load_edge_pair(dst, e, E, vec, -1, vs[i], vs[i + 1]);      // past the end: out of range, and looked at again below
                }
            }
            bool odd = false;                                // an id out of range, or no edge
            auto in_range = [&](int i) {
                const uint32_t u = (uint32_t)us[i], v = (uint32_t)vs[i], high = (uint32_t)(us[i] >> 32) | (uint32_t)(vs[i] >> 32);
                return high == 0u && (u > v ? u : v) < N;
            };
            uint2 of_v[Select::LOOKUP ? SCAN_PER : 1];       // LOOKUP: the lookups of all destinations at once, here
            uint32_t inner[Select::LOOKUP ? SCAN_PER : 1];
#pragma unroll
            for (int i = 0; Select::LOOKUP && i < SCAN_PER; ++i) {
                const uint32_t word = in_range(i) ? (uint32_t)vs[i] >> 5 : 0u;
                of_v[i] = own.words[word];
                inner[i] = select_inner(select, word);
            }
#pragma unroll
            for (int i = 0; i < SCAN_PER; ++i) {
                const uint32_t u = (uint32_t)us[i];
                uint32_t v = (uint32_t)vs[i];
                const bool ok = in_range(i);
                odd = odd || !ok;
                const unsigned long long in = __ballot(ok && (Select::LOOKUP ? word_has(of_v[Select::LOOKUP ? i : 0], v) : select_counted(select, v)));
                if (Select::LOOKUP)                          // in line: the destination's local id, and at the top whether the edge is kept
                    v = (uint32_t)word_rank(of_v[Select::LOOKUP ? i : 0], v) | ((inner[Select::LOOKUP ? i : 0] >> (v & 31u)) & 1u) << 31;
                if ((in >> lane) & 1ull) line[__builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, here))] = make_uint2(u, v);
                here += (uint32_t)__popcll(in);
                __builtin_amdgcn_sched_barrier(0);           // (an edge at a time: registers)
            }
            if (__any(odd)) {                                // (read again: registers)
                for (int i = 0; i < SCAN_PER; i += 2)
                    for (int64_t e = e0 + (int64_t)i * SCAN_THREADS, z = e + 2; e < z; ++e)
                        bad += e < E && !(src[e] >= 0 && dst[e] >= 0 && src[e] < (int64_t)N && dst[e] < (int64_t)N);
            }
        }
        here = (uint32_t)__builtin_amdgcn_readfirstlane((int)here);
        __builtin_amdgcn_wave_barrier();                     // (a wavefront's accesses to LDS are made in order)
        uint32_t u[SCAN_PER], v[SCAN_PER], at[SCAN_PER];      // local ids of edge 64 i + lane of them (NOT_KEPT: a source that is not owned)
        constexpr uint32_t NOT_KEPT = ~0u;
        auto on = [&](int i) { return (uint32_t)(64 * i + lane) < here; };
#pragma unroll
        for (int i = 0; i < SCAN_PER; i += 2) {
            if (64u * i >= here) break;                      // (uniform, here and below)
            const uint2 a = line[on(i) ? 64 * i + lane : 0], b = line[on(i + 1) ? 64 * (i + 1) + lane : 0];
            if constexpr (Select::LOOKUP) {
                const bool ka = a.y >> 31, kb = b.y >> 31;
                const uint2 au = own.words[ka ? a.x >> 5 : 0u], bu = own.words[kb ? b.x >> 5 : 0u];
                v[i] = a.y & ~(1u << 31);
                u[i] = ka ? (uint32_t)word_rank(au, a.x) : NOT_KEPT;
                v[i + 1] = b.y & ~(1u << 31);
                u[i + 1] = kb ? (uint32_t)word_rank(bu, b.x) : NOT_KEPT;
                continue;
            }
            const uint2 av = own.words[a.y >> 5], au = own.words[a.x >> 5], bv = own.words[b.y >> 5], bu = own.words[b.x >> 5];
            v[i] = (uint32_t)word_rank(av, a.y);
            u[i] = word_has(au, a.x) ? (uint32_t)word_rank(au, a.x) : NOT_KEPT;
            v[i + 1] = (uint32_t)word_rank(bv, b.y);
            u[i + 1] = word_has(bu, b.x) ? (uint32_t)word_rank(bu, b.x) : NOT_KEPT;
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();                                     // the counters are clear; the line has been read
#pragma unroll
        for (int i = 0; i < SCAN_PER; ++i) {
            if (64u * i >= here) break;
            if (!on(i)) continue;
            at[i] = atomicAdd(&first[v[i] >> SPAN_BITS], 1u);
            if (u[i] != NOT_KEPT) at[i] |= atomicAdd(&kept, 1u) << 16;
        }
        __syncthreads();
        if (tid < 64) {                                      // the ranges' places in the tile, and the tile's in the arrays
            constexpr int PER = SPANS_MAX / 64;
            uint32_t c[PER], sum = 0;
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                c[q] = PER * lane + q < spans ? first[PER * lane + q] : 0u;
                sum += c[q];
            }
            uint32_t incl = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_up(incl, o, 64);
                if (lane >= o) incl += t;
            }
            const uint32_t total = __shfl(incl, 63, 64);
            unsigned long long b = 0;
            if (lane < 2) {
                const uint32_t want = lane == 0 ? total : kept;
                if (want) b = atomicAdd(&counters[3 - lane], (unsigned long long)want);
                base[lane] = b;
            }
            if (lane == 0) id_total = total;
            b = __shfl(b, 0, 64);
            uint32_t place = incl - sum;
            auto head = [&](uint32_t x) { return (uint32_t)(b + x < id_cap ? b + x : id_cap); };
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                if (PER * lane + q < spans) {
                    first[PER * lane + q] = place;
                    heads[tile * (spans + 1) + PER * lane + q] = head(place);
                }
                place += c[q];
            }
            if (lane == 0) heads[tile * (spans + 1) + spans] = head(total);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SCAN_PER; ++i) {
            if (64u * i >= here) break;
            if (on(i)) buf[first[v[i] >> SPAN_BITS] + (at[i] & 0xFFFFu)] = v[i];
            if (on(i) && u[i] != NOT_KEPT) {
                const unsigned long long slot = base[1] + (at[i] >> 16);
                if (slot < cap) keys[slot] = ((uint64_t)v[i] << 32) | (uint64_t)u[i];
            }
        }
        __syncthreads();
        for (uint32_t x = tid; x < id_total; x += SCAN_THREADS) {
            if (base[0] + x < id_cap) ids[base[0] + x] = buf[x];
            else atomicAdd(&dg[buf[x]], 1ull);
        }
        __syncthreads();                                     // the arrays in LDS are used anew
    }
    for (int o = 32; o > 0; o >>= 1) bad += __shfl_down(bad, o, 64);
    if (lane == 0 && bad) atomicAdd(&counters[1], bad);
}

// dg[i] += how often i is among the tiles' local ids.  A workgroup counts a part of the tiles (blockIdx.y) for one range of ids
// (blockIdx.x) in LDS and adds its counts to memory as neighbouring words.  A wavefront takes the runs of `at_once` tiles together,
// whatever their lengths: id j of them lies in the run that a search over the runs' prefix sum finds.
__global__ __launch_bounds__(1024) void rank_count_kernel(const uint32_t* __restrict__ ids, const uint32_t* __restrict__ heads, int64_t n_tiles,
                                                          int spans, int at_once, int64_t n, unsigned long long* __restrict__ dg) {
    __shared__ uint32_t count[1 << SPAN_BITS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < (1 << SPAN_BITS); i += 1024) count[i] = 0u;
    __syncthreads();
    for (int64_t t0 = ((int64_t)blockIdx.y * 16 + wave) * at_once; t0 < n_tiles; t0 += (int64_t)gridDim.y * 16 * at_once) {
        const bool mine = lane < at_once && t0 + lane < n_tiles;
        const int64_t t = mine ? t0 + lane : t0;
        const uint32_t b = heads[t * (spans + 1) + blockIdx.x], e = heads[t * (spans + 1) + blockIdx.x + 1];
        uint32_t end = mine ? e - b : 0u;                    // of the lane's run, in the runs laid end to end
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t x = __shfl_up(end, o, 64);
            if (lane >= o) end += x;
        }
        const uint32_t total = __shfl(end, 63, 64), from = e - end;      // id j of this run is ids[from + j]
        constexpr int U = 8;
        for (uint32_t j0 = 0; j0 < total; j0 += 64 * U) {
            uint32_t id[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const uint32_t j = j0 + q * 64 + lane < total ? j0 + q * 64 + lane : total - 1;
                int run = 0;                                 // runs that end at or before j
#pragma unroll
                for (int o = 32; o > 0; o >>= 1)
                    if (__shfl(end, run + o - 1, 64) <= j) run += o;
                id[q] = ids[__shfl(from, run, 64) + j];
            }
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (j0 + q * 64 + lane < total) atomicAdd(&count[id[q] & ((1u << SPAN_BITS) - 1u)], 1u);
        }
    }
    __syncthreads();
    const int64_t id0 = (int64_t)blockIdx.x << SPAN_BITS;
    for (int i = tid; i < (1 << SPAN_BITS); i += 1024)
        if (count[i] && id0 + i < n) atomicAdd(&dg[id0 + i], (unsigned long long)count[i]);
}

template <typename Select>
static grp_status launch_scan_keys(const Select& select, const int64_t* src, const int64_t* dst, int64_t E, int64_t N, NodeSet own, int64_t n, int64_t spans,
                                   unsigned long long* dg, unsigned long long* counters, uint64_t* keys, int64_t cap, uint32_t* ids, int64_t id_cap,
                                   uint32_t* heads, hipStream_t st) {
    const int64_t tiles = cdiv(E, SCAN_TILE);
    hipLaunchKernelGGL(edge_scan_keys_kernel<Select>, dim3((unsigned)(tiles < SCAN_GRID ? tiles : SCAN_GRID)), dim3(SCAN_THREADS), 0, st, src, dst, E, (uint32_t)N,
                       own, select, (int)spans, dg, counters, keys, (unsigned long long)cap, ids, (unsigned long long)id_cap, heads);
    int64_t parts = cdiv(256, spans);                        // a workgroup per CU, a tile at least for each of its wavefronts
    if (parts > cdiv(tiles, 16)) parts = cdiv(tiles, 16);
    int at_once = 64;
    while (at_once > 1 && parts * 16 * at_once > tiles) at_once /= 2;
    hipLaunchKernelGGL(rank_count_kernel, dim3((unsigned)spans, (unsigned)parts), dim3(1024), 0, st, (const uint32_t*)ids, (const uint32_t*)heads, tiles, (int)spans,
                       at_once, n, dg);
    GRP_LAUNCH_CHECK();
    return GRP_OK;
}

// Local edge list: range check + keys in place order.
__global__ __launch_bounds__(256) void local_keys_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                         int64_t E, int64_t n, uint64_t* __restrict__ keys,
                                                         unsigned long long* __restrict__ bad) {
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < E; e += (int64_t)gridDim.x * 256) {
        const int64_t u = src[e], v = dst[e];
        if (u < 0 || v < 0 || u >= n || v >= n) {
            atomicAdd(bad, 1ull);
            keys[e] = 0;
        } else {
            keys[e] = ((uint64_t)v << 32) | (uint64_t)u;
        }
    }
}

// From sorted keys: idx[i] = low half; ptr[r] = first position whose high half is >= r (null: left to csr_rows_kernel).  SWAPPED: the
// halves change places.
template <bool SWAPPED>
__global__ __launch_bounds__(256) void csr_from_keys_kernel(const uint64_t* __restrict__ keys, int64_t nnz, int64_t n,
                                                            int64_t* __restrict__ ptr, int32_t* __restrict__ idx) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i <= nnz; i += (int64_t)gridDim.x * 256) {
        auto row = [&](int64_t k) { return (int64_t)(SWAPPED ? keys[k] & 0xFFFFFFFFull : keys[k] >> 32); };
        const int64_t hi = i < nnz ? row(i) : n;
        const int64_t prev = i > 0 ? row(i - 1) : -1;
        if (ptr)
            for (int64_t r = prev + 1; r <= hi; ++r) ptr[r] = i;
        if (i < nnz) idx[i] = (int32_t)(SWAPPED ? keys[i] >> 32 : keys[i] & 0xFFFFFFFFull);
    }
}

// The pointers alone, a search for each: where most rows are empty, one key after another would have a thread write all the pointers of
// a gap (2e6 rows of which 1000 have the 3e7 edges: 50 ms).
template <bool SWAPPED>
__global__ __launch_bounds__(256) void csr_rows_kernel(const uint64_t* __restrict__ keys, int64_t nnz, int64_t n, int64_t* __restrict__ ptr) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r > n) return;
    int64_t lo = 0, hi = nnz;                            // first position whose row is >= r
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)(SWAPPED ? keys[mid] & 0xFFFFFFFFull : keys[mid] >> 32) < r) lo = mid + 1; else hi = mid;
    }
    ptr[r] = lo;
}

__global__ __launch_bounds__(256) void degree_from_ptr_kernel(const int64_t* __restrict__ ptr, int64_t n,
                                                              int32_t* __restrict__ deg) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < n) deg[v] = (int32_t)(ptr[v + 1] - ptr[v]);
}

__global__ __launch_bounds__(256) void iota_kernel(int64_t n, int64_t* __restrict__ out) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < n) out[v] = v;
}

__global__ __launch_bounds__(256) void widen_kernel(const int32_t* __restrict__ in, int64_t n, int64_t* __restrict__ out) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < n) out[v] = in[v];
}

__global__ __launch_bounds__(256) void weight_check_kernel(const float* __restrict__ w, int64_t E,
                                                           unsigned long long* __restrict__ bad) {
    unsigned long long b = 0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < E; e += (int64_t)gridDim.x * 256)
        if (!(w[e] > 0.f) || !(w[e] <= 3.402823466e+38f)) b++;
    if (b) atomicAdd(bad, b);
}

// mass[r] = sum of vals over [ptr[r], ptr[r+1]) in fp64.  Rows of at most ROW_MASS_SERIAL entries are added in
// stored order by one thread.  Longer rows (hubs: 10^5 entries and more, which one thread would take
// milliseconds over) are left to row_mass_long_kernel: one workgroup per row, every thread adds a contiguous
// run in stored order and the 256 partial sums are added in thread order, a fixed order that does not depend
// on scheduling (and the same value as the serial sum whenever the partial sums are exact in fp64, as they
// are for float weights of similar magnitude).
constexpr int ROW_MASS_SERIAL = 1024;

__global__ __launch_bounds__(256) void row_mass_kernel(const int64_t* __restrict__ ptr, const float* __restrict__ vals,
                                                       int64_t n, double* __restrict__ mass,
                                                       int32_t* __restrict__ long_rows, int32_t* __restrict__ n_long) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    const int64_t b = ptr[r], e = ptr[r + 1];
    if (e - b > ROW_MASS_SERIAL) {
        long_rows[atomicAdd(n_long, 1)] = (int32_t)r;    // any order: each row is summed on its own
        return;
    }
    double s = 0.0;
    for (int64_t k = b; k < e; ++k) s += (double)vals[k];
    mass[r] = s;
}

__global__ __launch_bounds__(256) void row_mass_long_kernel(const int64_t* __restrict__ ptr, const float* __restrict__ vals,
                                                            const int32_t* __restrict__ long_rows,
                                                            const int32_t* __restrict__ n_long, double* __restrict__ mass) {
    __shared__ double part[256];
    const int count = *n_long;
    for (int j = blockIdx.x; j < count; j += gridDim.x) {
        const int64_t r = long_rows[j];
        const int64_t b = ptr[r], e = ptr[r + 1];
        const int64_t per = (e - b + 255) / 256;
        int64_t lo = b + threadIdx.x * per, hi = lo + per;
        if (lo > e) lo = e;
        if (hi > e) hi = e;
        double s = 0.0;
        for (int64_t k = lo; k < hi; ++k) s += (double)vals[k];
        part[threadIdx.x] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int q = 0; q < 256; ++q) t += part[q];
            mass[r] = t;
        }
        __syncthreads();
    }
}

// Row masses of a CSR-like (ptr, vals) pair; `scratch`: [n + 1] int32 device words (list of long rows + their count).
static grp_status launch_row_mass(const int64_t* ptr, const float* vals, int64_t n, double* mass, int32_t* scratch,
                                  hipStream_t st) {
    if (n == 0) return GRP_OK;
    GRP_HIP(hipMemsetAsync(scratch + n, 0, sizeof(int32_t), st));
    hipLaunchKernelGGL(row_mass_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, ptr, vals, n, mass, scratch, scratch + n);
    GRP_LAUNCH_CHECK();
    hipLaunchKernelGGL(row_mass_long_kernel, dim3(1024), dim3(256), 0, st, ptr, vals, (const int32_t*)scratch,
                       (const int32_t*)(scratch + n), mass);
    GRP_LAUNCH_CHECK();
    return GRP_OK;
}

static unsigned grid_for(int64_t work) {
    int64_t b = cdiv(work > 0 ? work : 1, 256);
    return (unsigned)(b > 16384 ? 16384 : b);
}

struct DevBuf {
    void* p = nullptr;
    ~DevBuf() { free(); }
    void free() { if (p) pool_free(p); p = nullptr; }    // (nothing on the device may still use it)
    grp_status alloc(size_t bytes) {
        if (pool_alloc(&p, bytes ? bytes : 4) != hipSuccess) {
            p = nullptr;
            (void)hipGetLastError();
            return fail(GRP_ENOMEM, "device allocation of %zu bytes failed", bytes);
        }
        return GRP_OK;
    }
    template <typename T> T* as() { return (T*)p; }
};

static void free_partition(grp_partition_t* h) {
    if (!h) return;
    if (h->borrowed_csr) { h->rowptr = nullptr; h->col = nullptr; }
    void* ptrs[] = {h->l2g, h->rowptr, h->col, h->colptr, h->row, h->d_local_in, h->d_local_out, h->d_global_in,
                    h->csr_long.long_row, h->csr_long.long_first, h->csr_long.chunk_begin, h->csr_long.chunk_end,
                    h->csc_long.long_row, h->csc_long.long_first, h->csc_long.chunk_begin, h->csc_long.chunk_end,
                    h->base_mask, h->csr_long.tasks, h->csr_long.row_task, h->csc_long.tasks, h->csc_long.row_task, h->csr_w, h->csc_w, h->w_local_in, h->w_global_in};
    const char* lo = (const char*)h->slab;
    for (void* q : ptrs)
        if (q && !(lo && (const char*)q >= lo && (const char*)q < lo + h->slab_bytes)) pool_free(q);
    if (h->slab) pool_free(h->slab);
    delete h;
}

template <typename T>
static grp_status halloc(T** out, int64_t count) {
    void* p = nullptr;
    const size_t bytes = (size_t)(count > 0 ? count : 1) * sizeof(T);
    if (pool_alloc(&p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return fail(GRP_ENOMEM, "device allocation of %zu bytes failed", bytes);
    }
    *out = (T*)p;
    return GRP_OK;
}

static int bits_for(int64_t n) {
    int b = 1;
    while (b < 32 && ((int64_t)1 << b) < n) ++b;
    return b;
}

// Split schedule of the rows longer than SPMM_LONG_ROW edges (a function of the pointer
// array only), built on the device into arrays sized for the worst case (out->long_row .. chunk_end,
// cap_long / cap_chunks entries); the two counts come back to the host (the launches that use the
// schedule are sized by them).  scanned: [n + 1] int64 scratch.
static grp_status build_long_rows(const int64_t* ptr_dev, int64_t n, LongRows* out, int64_t cap_long, int64_t cap_chunks,
                                  int64_t* scanned, void* tmp, size_t tmp_bytes, hipStream_t st) {
    out->n_long = out->n_chunks = 0;
    if (n == 0 || cap_long == 0) return GRP_OK;          // no row can be long
    GRP_TRY(build_long_rows_device(ptr_dev, n, out, cap_long, cap_chunks, scanned, tmp, tmp_bytes, st));
    int64_t total = 0;
    GRP_HIP(hipMemcpyAsync(&total, scanned + n, sizeof total, hipMemcpyDeviceToHost, st));
    GRP_HIP(hipStreamSynchronize(st));
    out->n_long = (int32_t)(total >> 32);
    out->n_chunks = (int32_t)(total & 0xFFFFFFFFll);
    return GRP_OK;
}

// The arrays build_csr_csc fills, carved from one allocation (base null: only measures).
static size_t carve_csr_csc(grp_partition_t* h, bool weighted, int64_t cap_long, int64_t cap_chunks, void* base, size_t cap) {
    Bump b(base, cap);
    const size_t n1 = (size_t)(h->n > 0 ? h->n : 1), z1 = (size_t)(h->nnz > 0 ? h->nnz : 1);
    if (weighted) {
        h->csr_w = b.take<float>(z1);
        h->csc_w = b.take<float>(z1);
    }
    h->rowptr = b.take<int64_t>(n1 + 1);
    h->colptr = b.take<int64_t>(n1 + 1);
    h->col = b.take<int32_t>(z1);
    h->row = b.take<int32_t>(z1);
    h->d_local_in = b.take<int32_t>(n1);
    h->d_local_out = b.take<int32_t>(n1);
    for (LongRows* lr : {&h->csr_long, &h->csc_long}) {
        if (cap_long == 0) continue;
        lr->long_row = b.take<int32_t>((size_t)cap_long);
        lr->long_first = b.take<int32_t>((size_t)cap_long + 1);
        lr->chunk_begin = b.take<int64_t>((size_t)cap_chunks);
        lr->chunk_end = b.take<int64_t>((size_t)cap_chunks);
    }
    return b.total();
}

// Sorts of the bits [begin, end) of 64-bit keys, with a value each if vals is given (temp null: sizes only), for the builds that
// buckets.hip does not take.  The library merges below 2^20 keys, in two launches per doubling; its digit passes are already faster
// from SORT_BY_DIGITS_FROM on (unweighted builds that once came here, us: 3e4, 2.5e5 edges 330 and 332; 4e4, 3e5 368 -> 293; 1e5,
// 7e5 466 -> 364; 1.2e5, 1e6 505 -> 396).
template <unsigned long LIMIT>
static hipError_t sort_bits_as(void* temp, size_t& bytes, uint64_t* in, uint64_t* out, float* vin, float* vout, int64_t count, unsigned begin,
                               unsigned end, hipStream_t st) {
    using Config = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config, rocprim::default_config, LIMIT>;
    if (vin) return rocprim::radix_sort_pairs<Config>(temp, bytes, in, out, vin, vout, (size_t)count, begin, end, st);
    return rocprim::radix_sort_keys<Config>(temp, bytes, in, out, (size_t)count, begin, end, st);
}
constexpr unsigned long SORT_BY_DIGITS_FROM = 1ul << 18;
static hipError_t sort_bits(void* temp, size_t& bytes, uint64_t* in, uint64_t* out, float* vin, float* vout, int64_t count, unsigned begin,
                            unsigned end, hipStream_t st) {
    return sort_bits_as<SORT_BY_DIGITS_FROM>(temp, bytes, in, out, vin, vout, count, begin, end, st);
}

// keys (unsorted, nnz of them; clobbered) -> h->rowptr/col/d_local_in and h->colptr/row/d_local_out.
// vals / vals_alt (optional, nnz floats each; clobbered): a value per key that travels through the
// (stable) sorts into h->csr_w and h->csc_w.
static grp_status build_csr_csc(grp_partition_t* h, uint64_t* keys, uint64_t* keys_alt, hipStream_t st,
                                float* vals = nullptr, float* vals_alt = nullptr) {
    const int64_t n = h->n, nnz = h->nnz;
    const int64_t cap_long = nnz > SPMM_LONG_ROW ? nnz / SPMM_LONG_ROW + 1 : 0;
    const int64_t cap_chunks = cap_long ? nnz / SPMM_CHUNK + cap_long + 1 : 0;
    if (cap_chunks >= ((int64_t)1 << 31)) return fail(GRP_ERANGE, "more than 2^31 row chunks");
    h->slab_bytes = carve_csr_csc(h, vals != nullptr, cap_long, cap_chunks, nullptr, 0);
    if (pool_alloc(&h->slab, h->slab_bytes) != hipSuccess) {
        (void)hipGetLastError();
        h->slab = nullptr;
        return fail(GRP_ENOMEM, "device allocation of %zu bytes failed", h->slab_bytes);
    }
    (void)carve_csr_csc(h, vals != nullptr, cap_long, cap_chunks, h->slab, h->slab_bytes);
    BucketPlan plan;
    bool uneven = false;                                 // few rows hold most edges
    if (!vals && bucket_plan(n, nnz, &plan)) {
        DevBuf scratch;
        int64_t long_edges[2];
        bool done = false;
        GRP_TRY(scratch.alloc(bucket_scratch_bytes(plan, nnz)));
        GRP_TRY(bucket_build(h, plan, keys, keys_alt, scratch.p, long_edges, &done, st));
        if (done) return build_slice_tasks(h, long_edges, st);
        uneven = true;
    }
    const unsigned id_bits = bits_for(n > 1 ? n : 2);
    // one scratch allocation: the sorts' temporary storage, later the long-row pass's prefix sums
    size_t sort_bytes = 0, transpose_bytes = 0;
    if (nnz > 0) {
        GRP_HIP(sort_bits(nullptr, sort_bytes, keys, keys_alt, vals, vals_alt, nnz, 0u, 32u + id_bits, st));
        GRP_HIP(sort_bits(nullptr, transpose_bytes, keys_alt, keys, vals_alt, vals, nnz, 0u, id_bits, st));
        sort_bytes = std::max(sort_bytes, transpose_bytes);
    }
    const size_t scan_bytes = cap_long ? scan_temp_bytes(n + 1) : 0;
    const size_t scanned_bytes = cap_long ? (((size_t)n + 1) * sizeof(int64_t) + 255) & ~(size_t)255 : 0;
    size_t tmp_bytes = sort_bytes > scanned_bytes + scan_bytes ? sort_bytes : scanned_bytes + scan_bytes;
    DevBuf tmp;
    GRP_TRY(tmp.alloc(tmp_bytes));
    if (nnz > 0) {
        GRP_HIP(sort_bits(tmp.p, sort_bytes, keys, keys_alt, vals, vals_alt, nnz, 0u, 32u + id_bits, st));
        if (vals) GRP_HIP(hipMemcpyAsync(h->csr_w, vals_alt, (size_t)nnz * sizeof(float), hipMemcpyDeviceToDevice, st));
    }
    if (uneven) hipLaunchKernelGGL(csr_rows_kernel<false>, dim3((unsigned)cdiv(n + 1, 256)), dim3(256), 0, st, (const uint64_t*)keys_alt, nnz, n, h->rowptr);
    hipLaunchKernelGGL(csr_from_keys_kernel<false>, dim3(grid_for(nnz + 1)), dim3(256), 0, st, keys_alt, nnz, n, uneven ? nullptr : h->rowptr, h->col);
    GRP_LAUNCH_CHECK();
    // The transpose: the keys are in order of (destination, source), so that a stable sort by source alone gives the order of
    // (source, destination): half the digits.
    if (nnz > 0) {
        GRP_HIP(sort_bits(tmp.p, sort_bytes, keys_alt, keys, vals_alt, vals, nnz, 0u, id_bits, st));
        if (vals) GRP_HIP(hipMemcpyAsync(h->csc_w, vals, (size_t)nnz * sizeof(float), hipMemcpyDeviceToDevice, st));
    }
    if (uneven) hipLaunchKernelGGL(csr_rows_kernel<true>, dim3((unsigned)cdiv(n + 1, 256)), dim3(256), 0, st, (const uint64_t*)keys, nnz, n, h->colptr);
    hipLaunchKernelGGL(csr_from_keys_kernel<true>, dim3(grid_for(nnz + 1)), dim3(256), 0, st, keys, nnz, n, uneven ? nullptr : h->colptr, h->row);
    GRP_LAUNCH_CHECK();
    if (n > 0) {
        hipLaunchKernelGGL(degree_from_ptr_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, h->rowptr, n, h->d_local_in);
        GRP_LAUNCH_CHECK();
        hipLaunchKernelGGL(degree_from_ptr_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, h->colptr, n, h->d_local_out);
        GRP_LAUNCH_CHECK();
    }
    int64_t* const scanned = (int64_t*)tmp.p;            // the sorts are done (stream order): their scratch is free
    void* const scan_tmp = (char*)tmp.p + scanned_bytes;
    GRP_TRY(build_long_rows(h->rowptr, n, &h->csr_long, cap_long, cap_chunks, scanned, scan_tmp, scan_bytes, st));
    GRP_TRY(build_long_rows(h->colptr, n, &h->csc_long, cap_long, cap_chunks, scanned, scan_tmp, scan_bytes, st));
    GRP_HIP(hipStreamSynchronize(st));
    return vals ? GRP_OK : build_slice_tasks(h, {-1, -1}, st);      // weighted partitions keep the chunk schedule
}

static grp_status weighted_build(const int64_t* src, const int64_t* dst, const float* w, int64_t E, NodeSet own,
                                 hipStream_t st, grp_partition_t* h);

// A node set and what building it needs, from one allocation.
struct SetScratch {
    unsigned long long* counters;        // [4]; the last: members
    uint32_t* bits;                      // [n_words + 1]
    int32_t* before;                     // [n_words + 1]
    uint2* words;                        // [n_words]
    char* scan;
    int64_t n_words;
    size_t scan_bytes;
    grp_status alloc(int64_t N, DevBuf& slab) {
        n_words = cdiv(N > 0 ? N : 1, 32);
        scan_bytes = scan_temp_bytes(n_words + 1);
        for (int pass = 0; pass < 2; ++pass) {
            Bump b(slab.p, 0);
            counters = b.take<unsigned long long>(4);
            bits = b.take<uint32_t>((size_t)n_words + 1);
            before = b.take<int32_t>((size_t)n_words + 1);
            words = b.take<uint2>((size_t)n_words);
            scan = b.take<char>(scan_bytes);
            if (pass == 0) GRP_TRY(slab.alloc(b.total()));
        }
        return GRP_OK;
    }
};
static grp_status count_node_set(int64_t N, const SetScratch& t, int64_t* n, hipStream_t st);      // the rest, from bits
// bits and before of the nodes that member(v) holds for, and their number n (waits for it).
template <typename Member>
static grp_status build_node_set(int64_t N, Member member, const SetScratch& t, int64_t* n, hipStream_t st) {
    *n = 0;
    if (N <= 0) return GRP_OK;
    hipLaunchKernelGGL(node_bits_kernel<Member>, dim3((unsigned)cdiv((t.n_words + 1) * 32, 256)), dim3(256), 0, st, N, t.n_words, member, t.bits);
    GRP_LAUNCH_CHECK();
    return count_node_set(N, t, n, st);
}
static grp_status count_node_set(int64_t N, const SetScratch& t, int64_t* n, hipStream_t st) {
    GRP_TRY(exclusive_scan_popcount(t.scan, t.scan_bytes, t.bits, t.before, t.n_words + 1, st));
    if (N >= ((int64_t)1 << 31)) {       // more than 32 bits may be needed to see that there are too many
        hipLaunchKernelGGL(count_bits_kernel, dim3(4096), dim3(256), 0, st, (const uint32_t*)t.bits, t.n_words, t.counters + 3);
        GRP_LAUNCH_CHECK();
        GRP_HIP(hipMemcpyAsync(n, t.counters + 3, sizeof *n, hipMemcpyDeviceToHost, st));
        GRP_HIP(hipStreamSynchronize(st));
        return GRP_OK;
    }
    int32_t count = 0;
    GRP_HIP(hipMemcpyAsync(&count, t.before + t.n_words, sizeof count, hipMemcpyDeviceToHost, st));
    GRP_HIP(hipStreamSynchronize(st));
    *n = count;
    return GRP_OK;
}

static grp_status partition_impl(const int64_t* src, const int64_t* dst, int64_t E, int64_t N, int32_t K, uint64_t seed,
                                 int32_t part_id, hipStream_t st, grp_partition_t* h, const float* w = nullptr,
                                 bool weighted = false) {
    // every N-sized temporary from one allocation: the node set, counters, scan scratch
    SetScratch t;
    DevBuf slab;
    GRP_TRY(t.alloc(N, slab));
    GRP_HIP(hipMemsetAsync(t.counters, 0, 4 * sizeof(unsigned long long), st));
    const OwnerTest owned = owner_test(seed, (uint32_t)K, (uint32_t)part_id);
    int64_t n = 0;
    GRP_TRY(build_node_set(N, owned, t, &n, st));
    if (n >= ((int64_t)1 << 31)) return fail(GRP_ERANGE, "partition has %lld >= 2^31 local nodes", (long long)n);
    h->n = n;
    GRP_TRY(halloc(&h->l2g, n));
    GRP_TRY(halloc(&h->d_global_in, n));
    GRP_HIP(hipMemsetAsync(h->d_global_in, 0, (size_t)(n > 0 ? n : 1) * sizeof(int64_t), st));
    const NodeSet own{t.words};
    if (N > 0) {
        hipLaunchKernelGGL(set_nodes_kernel, dim3((unsigned)cdiv(N, 256)), dim3(256), 0, st, N, (const uint32_t*)t.bits, (const int32_t*)t.before,
                           t.words, h->l2g);
        GRP_LAUNCH_CHECK();
    }
    unsigned long long host_counters[3] = {0, 0, 0};
    const unsigned scan_grid = grid_for(E) < (unsigned)EDGE_SCAN_GRID ? grid_for(E) : (unsigned)EDGE_SCAN_GRID;
    // Unweighted: one pass writes the keys too, into a buffer sized for twice the expected E / K^2 kept edges, and the local ids of twice
    // the expected E / K edges that end in the partition.  Ids beyond 32 bits and more ranges of local ids than that pass
    // orders are counted through a table in LDS instead (a build from 62e6 edges, one of 2 parts of 1e7 nodes: 4.5 ms; with a second pass
    // over the edges for the keys 5.4).
    const int64_t spans = cdiv(n > 0 ? n : 1, (int64_t)1 << SPAN_BITS), scan_tiles = cdiv(E, SCAN_TILE);
    const bool ranged = !weighted && N < ((int64_t)1 << 31) && spans <= SPANS_MAX;
    int64_t cap = weighted ? 0 : 2 * (E / K / K) + (1 << 20), id_cap = ranged ? 2 * (E / K) + (1 << 20) : 0;
    if (cap > E) cap = E;
    if (id_cap > E) id_cap = E;
    if (id_cap > (int64_t)0xFFFFFFF0) id_cap = 0xFFFFFFF0;
    DevBuf keybuf, idbuf;                                // both key arrays; the local ids and where the tiles' runs begin
    size_t key_pitch = (((size_t)(cap > 0 ? cap : 1) * sizeof(uint64_t)) + 255) & ~(size_t)255;
    const size_t id_pitch = (((size_t)id_cap * sizeof(uint32_t)) + 255) & ~(size_t)255;
    if (!weighted) GRP_TRY(keybuf.alloc(2 * key_pitch));
    if (ranged && E > 0) GRP_TRY(idbuf.alloc(id_pitch + (size_t)scan_tiles * (size_t)(spans + 1) * sizeof(uint32_t)));
    if (E > 0) {
        if (weighted) {
            ProfScope ps("partition_edge_scan", st, 0.0, 16.0 * (double)E);
            hipLaunchKernelGGL(edge_scan_kernel<false>, dim3(scan_grid), dim3(256), 0, st, src, dst, E, N, own,
                               (unsigned long long*)h->d_global_in, t.counters, (uint64_t*)nullptr, 0ull);
            GRP_LAUNCH_CHECK();
        } else if (!ranged) {
            ProfScope ps("partition_edge_scan_keys", st, 0.0, 16.0 * (double)E);
            hipLaunchKernelGGL(edge_scan_kernel<true>, dim3(scan_grid), dim3(256), 0, st, src, dst, E, N, own,
                               (unsigned long long*)h->d_global_in, t.counters, keybuf.as<uint64_t>(), (unsigned long long)cap);
            GRP_LAUNCH_CHECK();
        } else {
            ProfScope ps("partition_edge_scan_keys", st, 0.0, 16.0 * (double)E);
            uint32_t* const heads = (uint32_t*)((char*)idbuf.p + id_pitch);
            auto go = [&](auto select) {
                return launch_scan_keys(select, src, dst, E, N, own, n, spans, (unsigned long long*)h->d_global_in, t.counters, keybuf.as<uint64_t>(), cap,
                                        idbuf.as<uint32_t>(), id_cap, heads, st);
            };
            GRP_TRY((K & (K - 1)) == 0 ? go(OwnedEdges<true>{owned}) : go(OwnedEdges<false>{owned}));
        }
        GRP_HIP(hipMemcpyAsync(host_counters, t.counters, sizeof host_counters, hipMemcpyDeviceToHost, st));
        GRP_HIP(hipStreamSynchronize(st));
    }
    if (host_counters[1] != 0)
        return fail(GRP_ERANGE, "%llu edges have an endpoint outside [0, %lld)", host_counters[1], (long long)N);
    const int64_t nnz = (int64_t)(weighted ? host_counters[0] : host_counters[2]);
    h->nnz = nnz;
    if (weighted) return weighted_build(src, dst, w, E, own, st, h);
    DevBuf exact;                                        // only if the first buffer was too small
    uint64_t* keys = keybuf.as<uint64_t>();
    if (nnz > cap) {
        key_pitch = (((size_t)nnz * sizeof(uint64_t)) + 255) & ~(size_t)255;
        GRP_TRY(exact.alloc(2 * key_pitch));
        keys = exact.as<uint64_t>();
        GRP_HIP(hipMemsetAsync(t.counters + 2, 0, sizeof(unsigned long long), st));
        ProfScope ps("partition_edge_keys", st, 0.0, 16.0 * (double)E + 8.0 * (double)nnz);
        hipLaunchKernelGGL(edge_keys_kernel<SetSelect>, dim3(grid_for(E)), dim3(256), 0, st, src, dst, E, SetSelect{own},
                           t.counters + 2, keys);
        GRP_LAUNCH_CHECK();
    }
    uint64_t* const keys_alt = (uint64_t*)((char*)keys + key_pitch);
    return build_csr_csc(h, keys, keys_alt, st);
}

// ------------------------------------------------------------------ halo partitions
// One hop outwards: the source of every edge whose destination is already inside joins.
// The rest of a weighted partition build (h->n, h->nnz, h->l2g, h->d_global_in are set; the ids are
// range-checked): CSR/CSC with the edge weights carried along, then the weight masses.
static grp_status weighted_build(const int64_t* src, const int64_t* dst, const float* w, int64_t E, NodeSet own,
                                 hipStream_t st, grp_partition_t* h) {
    const int64_t n = h->n, nnz = h->nnz;
    DevBuf bad, tiles, scan_tmp;
    GRP_TRY(bad.alloc(sizeof(unsigned long long)));
    GRP_HIP(hipMemsetAsync(bad.p, 0, sizeof(unsigned long long), st));
    unsigned long long host_bad = 0;
    if (E > 0) {
        hipLaunchKernelGGL(weight_check_kernel, dim3(grid_for(E)), dim3(256), 0, st, w, E, bad.as<unsigned long long>());
        GRP_LAUNCH_CHECK();
        GRP_HIP(hipMemcpyAsync(&host_bad, bad.p, sizeof host_bad, hipMemcpyDeviceToHost, st));
        GRP_HIP(hipStreamSynchronize(st));
    }
    if (host_bad) return fail(GRP_EINVAL, "%llu edge weights are not positive finite numbers", host_bad);
    const int64_t n_tiles = cdiv(E, OC_TILE);
    const size_t tile_pitch = (((size_t)n_tiles + 1) * sizeof(int64_t) + 255) & ~(size_t)255;
    GRP_TRY(tiles.alloc(2 * tile_pitch));                 // per-tile counts, then their prefix sums
    int64_t* const tile_count = tiles.as<int64_t>();
    int64_t* const tile_base = (int64_t*)((char*)tiles.p + tile_pitch);
    const size_t scan_bytes = scan_temp_bytes(n_tiles + 1);
    GRP_TRY(scan_tmp.alloc(scan_bytes));
    const unsigned oc_grid = (unsigned)(n_tiles < 16384 ? (n_tiles > 0 ? n_tiles : 1) : 16384);
    // the slots of the selected edges, in edge-list order (which = 0: local edges, 1: every in-edge of an owned node)
    auto place = [&](int which) -> grp_status {
        if (E <= 0) return GRP_OK;
        if (which == 0)
            hipLaunchKernelGGL(ordered_count_kernel<0>, dim3(oc_grid), dim3(256), 0, st, src, dst, E, own, n_tiles, tile_count);
        else
            hipLaunchKernelGGL(ordered_count_kernel<1>, dim3(oc_grid), dim3(256), 0, st, src, dst, E, own, n_tiles, tile_count);
        GRP_LAUNCH_CHECK();
        return exclusive_scan_i64(scan_tmp.p, scan_bytes, tile_count, tile_base, n_tiles + 1, st);
    };
    // ---- local edges with their weights
    DevBuf keys, keys_alt, vals, vals_alt;
    GRP_TRY(keys.alloc((size_t)nnz * sizeof(uint64_t)));
    GRP_TRY(keys_alt.alloc((size_t)nnz * sizeof(uint64_t)));
    GRP_TRY(vals.alloc((size_t)nnz * sizeof(float)));
    GRP_TRY(vals_alt.alloc((size_t)nnz * sizeof(float)));
    if (nnz > 0) {
        GRP_TRY(place(0));
        hipLaunchKernelGGL(ordered_emit_kernel<0>, dim3(oc_grid), dim3(256), 0, st, src, dst, w, E, own, n_tiles,
                           (const int64_t*)tile_base, keys.as<uint64_t>(), (uint32_t*)nullptr, vals.as<float>());
        GRP_LAUNCH_CHECK();
    }
    GRP_TRY(build_csr_csc(h, keys.as<uint64_t>(), keys_alt.as<uint64_t>(), st, vals.as<float>(), vals_alt.as<float>()));
    GRP_TRY(halloc(&h->w_local_in, n));
    GRP_TRY(halloc(&h->w_global_in, n));
    if (n == 0) return GRP_OK;
    DevBuf mass_scratch;
    GRP_TRY(mass_scratch.alloc(((size_t)n + 1) * sizeof(int32_t)));
    GRP_TRY(launch_row_mass(h->rowptr, h->csr_w, n, h->w_local_in, mass_scratch.as<int32_t>(), st));
    // ---- every in-edge of an owned node, grouped by destination in edge-list order
    DevBuf cnt, off;
    GRP_TRY(cnt.alloc((size_t)(n + 1) * sizeof(int64_t)));
    GRP_TRY(off.alloc((size_t)(n + 1) * sizeof(int64_t)));
    GRP_HIP(hipMemsetAsync(cnt.p, 0, (size_t)(n + 1) * sizeof(int64_t), st));
    GRP_HIP(hipMemcpyAsync(cnt.p, h->d_global_in, (size_t)n * sizeof(int64_t), hipMemcpyDeviceToDevice, st));
    {
        size_t bytes = 0;
        DevBuf tmp;
        GRP_HIP(rocprim::exclusive_scan(nullptr, bytes, cnt.as<int64_t>(), off.as<int64_t>(), (int64_t)0, (size_t)(n + 1),
                                        rocprim::plus<int64_t>(), st));
        GRP_TRY(tmp.alloc(bytes));
        GRP_HIP(rocprim::exclusive_scan(tmp.p, bytes, cnt.as<int64_t>(), off.as<int64_t>(), (int64_t)0, (size_t)(n + 1),
                                        rocprim::plus<int64_t>(), st));
        GRP_HIP(hipStreamSynchronize(st));        // tmp is released at the end of this scope
    }
    int64_t total = 0;
    GRP_HIP(hipMemcpy(&total, off.as<int64_t>() + n, sizeof(int64_t), hipMemcpyDeviceToHost));
    DevBuf k32, k32_alt, vin, vin_alt, sort_tmp;
    GRP_TRY(k32.alloc((size_t)total * sizeof(uint32_t)));
    GRP_TRY(k32_alt.alloc((size_t)total * sizeof(uint32_t)));
    GRP_TRY(vin.alloc((size_t)total * sizeof(float)));
    GRP_TRY(vin_alt.alloc((size_t)total * sizeof(float)));
    if (total > 0) {
        GRP_TRY(place(1));
        hipLaunchKernelGGL(ordered_emit_kernel<1>, dim3(oc_grid), dim3(256), 0, st, src, dst, w, E, own, n_tiles,
                           (const int64_t*)tile_base, (uint64_t*)nullptr, k32.as<uint32_t>(), vin.as<float>());
        GRP_LAUNCH_CHECK();
        const unsigned end_bit = (unsigned)bits_for(n > 1 ? n : 2);
        size_t bytes = 0;
        GRP_HIP(rocprim::radix_sort_pairs(nullptr, bytes, k32.as<uint32_t>(), k32_alt.as<uint32_t>(), vin.as<float>(),
                                          vin_alt.as<float>(), (size_t)total, 0u, end_bit, st));
        GRP_TRY(sort_tmp.alloc(bytes));
        GRP_HIP(rocprim::radix_sort_pairs(sort_tmp.p, bytes, k32.as<uint32_t>(), k32_alt.as<uint32_t>(), vin.as<float>(),
                                          vin_alt.as<float>(), (size_t)total, 0u, end_bit, st));
    }
    GRP_TRY(launch_row_mass(off.as<int64_t>(), vin_alt.as<float>(), n, h->w_global_in, mass_scratch.as<int32_t>(), st));
    GRP_HIP(hipStreamSynchronize(st));
    return GRP_OK;
}

// The sources of edges whose destination is in `inner` are flagged.  (Memberships come from a bitmap in the L2, a flag is a byte: every
// writer stores the same value.  A bitmap of the new members would take an atomic each: 2e7 edges, 2.4e6 nodes 536 us, words of flags for both
// 228, this way 137.)
__global__ __launch_bounds__(256) void halo_grow_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                        int64_t E, int64_t N, const uint32_t* __restrict__ inner,
                                                        uint8_t* __restrict__ flag, unsigned long long* __restrict__ bad) {
    const bool vec = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    constexpr int PER = 8;
    unsigned long long odd = 0;
    for (int64_t t0 = (int64_t)blockIdx.x * (256 * PER); t0 < E; t0 += (int64_t)gridDim.x * (256 * PER)) {
        int64_t us[PER], vs[PER];
#pragma unroll
        for (int i = 0; i < PER; i += 2) {
            const int64_t e = t0 + (int64_t)i * 256 + 2 * threadIdx.x;
            load_edge_pair(src, e, E, vec, 0, us[i], us[i + 1]);
            load_edge_pair(dst, e, E, vec, -1, vs[i], vs[i + 1]);      // past the end: out of range, but no error
        }
        if (t0 + 256 * PER > E)                              // (uniform; by its place: an edge's id may have any value)
#pragma unroll
            for (int i = 0; i < PER; ++i) odd -= t0 + (i & ~1) * 256 + 2 * threadIdx.x + (i & 1) >= E;
        uint32_t in[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const bool ok = us[i] >= 0 && vs[i] >= 0 && us[i] < N && vs[i] < N;
            odd += !ok;
            in[i] = inner[ok ? vs[i] >> 5 : 0];
            if (!ok) in[i] = 0u;
        }
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if ((in[i] >> (vs[i] & 31)) & 1u) flag[us[i]] = 1;
    }
    for (int o = 32; o > 0; o >>= 1) odd += __shfl_down(odd, o, 64);
    if ((threadIdx.x & 63) == 0 && odd) atomicAdd(bad, odd);
}
struct GrownMember {
    const uint32_t* inner;
    const uint8_t* flag;
    __device__ __forceinline__ bool operator()(int64_t v) const { return ((inner[v >> 5] >> (v & 31)) & 1u) || flag[v]; }
};

// Global in-degree of the members and the number of kept edges (destination in `inner`): partitions of more nodes than
// edge_scan_keys_kernel orders.
__global__ __launch_bounds__(256) void halo_scan_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                        int64_t E, NodeSet own, const uint32_t* __restrict__ inner,
                                                        unsigned long long* __restrict__ dg,
                                                        unsigned long long* __restrict__ kept_out) {
    __shared__ int32_t slot_key[DG_SLOTS];               // in-degree counts go through an LDS table (see edge_scan_kernel)
    __shared__ uint32_t slot_count[DG_SLOTS];
    for (int i = threadIdx.x; i < DG_SLOTS; i += 256) { slot_key[i] = -1; slot_count[i] = 0u; }
    __syncthreads();
    unsigned long long kept = 0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < E; e += (int64_t)gridDim.x * 256) {
        const int64_t v = dst[e];
        if (set_has(own, v)) dg_table_add(slot_key, slot_count, dg, set_rank(own, v));
        kept += (inner[v >> 5] >> (v & 31)) & 1u;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < DG_SLOTS; i += 256)
        if (slot_key[i] >= 0) atomicAdd(&dg[slot_key[i]], (unsigned long long)slot_count[i]);
    for (int o = 32; o > 0; o >>= 1) kept += __shfl_down(kept, o, 64);
    if ((threadIdx.x & 63) == 0 && kept) atomicAdd(kept_out, kept);
}

__global__ __launch_bounds__(256) void halo_owned_kernel(int64_t N, NodeSet own, const uint32_t* __restrict__ owned, uint8_t* __restrict__ owned_mask) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < N && set_has(own, v)) owned_mask[set_rank(own, v)] = (uint8_t)((owned[v >> 5] >> (v & 31)) & 1u);
}

static grp_status halo_partition_impl(const int64_t* src, const int64_t* dst, int64_t E, int64_t N, int32_t K, uint64_t seed,
                                      int32_t part_id, int32_t hops, hipStream_t st, grp_partition_t* h) {
    SetScratch t;                                        // the members; counters: [0] kept, [1] bad ids, [2] key cursor, [3] ids
    DevBuf slab, bits;
    GRP_TRY(t.alloc(N, slab));
    GRP_TRY(bits.alloc(2 * ((size_t)t.n_words + 1) * sizeof(uint32_t) + (size_t)t.n_words * 32));
    uint32_t* const owned = bits.as<uint32_t>();
    uint32_t* const inner = owned + t.n_words + 1;       // the members before the last hop
    uint8_t* const flag = (uint8_t*)(inner + t.n_words + 1);
    const size_t bits_bytes = ((size_t)t.n_words + 1) * sizeof(uint32_t);
    GRP_HIP(hipMemsetAsync(t.counters, 0, 4 * sizeof(unsigned long long), st));
    int64_t n = 0;
    if (N > 0) {
        const OwnerTest test = owner_test(seed, (uint32_t)K, (uint32_t)part_id);
        hipLaunchKernelGGL(node_bits_kernel<OwnerTest>, dim3((unsigned)cdiv((t.n_words + 1) * 32, 256)), dim3(256), 0, st, N, t.n_words, test, owned);
        GRP_LAUNCH_CHECK();
        GRP_HIP(hipMemcpyAsync(t.bits, owned, bits_bytes, hipMemcpyDeviceToDevice, st));
        GRP_HIP(hipMemsetAsync(flag, 0, (size_t)t.n_words * 32, st));
        for (int hop = 0; hop < hops; ++hop) {
            GRP_HIP(hipMemcpyAsync(inner, t.bits, bits_bytes, hipMemcpyDeviceToDevice, st));
            if (E > 0) {
                hipLaunchKernelGGL(halo_grow_kernel, dim3(grid_for(cdiv(E, 8))), dim3(256), 0, st, src, dst, E, N, (const uint32_t*)inner, flag, t.counters + 1);
                hipLaunchKernelGGL(node_bits_kernel<GrownMember>, dim3((unsigned)cdiv((t.n_words + 1) * 32, 256)), dim3(256), 0, st, N, t.n_words,
                                   GrownMember{inner, flag}, t.bits);
                GRP_LAUNCH_CHECK();
            }
        }
        unsigned long long nbad = 0;
        GRP_HIP(hipMemcpyAsync(&nbad, t.counters + 1, sizeof nbad, hipMemcpyDeviceToHost, st));
        GRP_TRY(count_node_set(N, t, &n, st));           // (waits)
        if (nbad) return fail(GRP_ERANGE, "edges have an endpoint outside [0, %lld)", (long long)N);
    }
    if (n >= ((int64_t)1 << 31)) return fail(GRP_ERANGE, "partition has %lld >= 2^31 local nodes", (long long)n);
    h->n = n;
    GRP_TRY(halloc(&h->l2g, n));
    GRP_TRY(halloc(&h->d_global_in, n));
    GRP_TRY(halloc(&h->base_mask, n));
    GRP_HIP(hipMemsetAsync(h->d_global_in, 0, (size_t)(n > 0 ? n : 1) * sizeof(int64_t), st));
    GRP_HIP(hipMemsetAsync(t.counters, 0, 4 * sizeof(unsigned long long), st));
    const NodeSet own{t.words};
    if (N > 0) {
        hipLaunchKernelGGL(set_nodes_kernel, dim3((unsigned)cdiv(N, 256)), dim3(256), 0, st, N, (const uint32_t*)t.bits, (const int32_t*)t.before,
                           t.words, h->l2g);
        hipLaunchKernelGGL(halo_owned_kernel, dim3((unsigned)cdiv(N, 256)), dim3(256), 0, st, N, own, (const uint32_t*)owned, h->base_mask);
        GRP_LAUNCH_CHECK();
    }
    // As a hash build (partition_impl): one pass writes the keys too.  Room for twice the expected edges of a single hop, whose destinations are a
    // random part of the nodes; for all edges, up to 2^28, of several, and for the local ids of all, up to 2^30: halo nodes are those with
    // many edges (62e6 of a skewed graph, ids of the nodes' share of them: the rest, counted one by one, took the pass from 657 to 1037 us).  Where
    // that room is not to be had, edges and in-degrees are counted first, which needs none.
    const int64_t spans = cdiv(n > 0 ? n : 1, (int64_t)1 << SPAN_BITS);
    bool ranged = N < ((int64_t)1 << 31) && spans <= SPANS_MAX && E > 0;
    const HaloEdges select{inner};
    unsigned long long host[3] = {0, 0, 0};
    DevBuf keys, keys_alt, idbuf;
    int64_t cap = 0, id_cap = 0;
    size_t id_pitch = 0;
    if (ranged) {
        cap = std::min<int64_t>(E, hops == 1 ? 2 * (E / K) + (1 << 20) : (int64_t)1 << 28);
        id_cap = std::min<int64_t>(E, (int64_t)1 << 30);
        id_pitch = (((size_t)id_cap * sizeof(uint32_t)) + 255) & ~(size_t)255;
        ranged = keys.alloc((size_t)cap * sizeof(uint64_t)) == GRP_OK &&
                 idbuf.alloc(id_pitch + (size_t)cdiv(E, SCAN_TILE) * (size_t)(spans + 1) * sizeof(uint32_t)) == GRP_OK;
        if (!ranged) { keys.free(); idbuf.free(); cap = 0; }
    }
    if (ranged) {
        GRP_TRY(launch_scan_keys(select, src, dst, E, N, own, n, spans, (unsigned long long*)h->d_global_in, t.counters, keys.as<uint64_t>(), cap,
                                 idbuf.as<uint32_t>(), id_cap, (uint32_t*)((char*)idbuf.p + id_pitch), st));
    } else if (E > 0) {
        const unsigned scan_grid = grid_for(E) < (unsigned)EDGE_SCAN_GRID ? grid_for(E) : (unsigned)EDGE_SCAN_GRID;
        hipLaunchKernelGGL(halo_scan_kernel, dim3(scan_grid), dim3(256), 0, st, src, dst, E, own, (const uint32_t*)inner,
                           (unsigned long long*)h->d_global_in, t.counters);
        GRP_LAUNCH_CHECK();
    }
    GRP_HIP(hipMemcpyAsync(host, t.counters, sizeof host, hipMemcpyDeviceToHost, st));
    GRP_HIP(hipStreamSynchronize(st));
    if (host[1]) return fail(GRP_ERANGE, "%llu edges have an endpoint outside [0, %lld)", host[1], (long long)N);      // (edges of no nodes: not seen above)
    const int64_t nnz = (int64_t)(ranged ? host[2] : host[0]);
    h->nnz = nnz;
    idbuf.free();
    // not written yet, or not all of them, or in a buffer with more to spare than there is for the other
    if (nnz > cap || keys_alt.alloc((size_t)nnz * sizeof(uint64_t)) != GRP_OK) {
        keys.free();
        GRP_TRY(keys.alloc((size_t)nnz * sizeof(uint64_t)));
        GRP_TRY(keys_alt.alloc((size_t)nnz * sizeof(uint64_t)));
        GRP_HIP(hipMemsetAsync(t.counters + 2, 0, sizeof(unsigned long long), st));
        hipLaunchKernelGGL(edge_keys_kernel<HaloSelect>, dim3(grid_for(E)), dim3(256), 0, st, src, dst, E, HaloSelect{own, inner}, t.counters + 2,
                           keys.as<uint64_t>());
        GRP_LAUNCH_CHECK();
    }
    return build_csr_csc(h, keys.as<uint64_t>(), keys_alt.as<uint64_t>(), st);
}

// ------------------------------------------------------------------ chunks
constexpr int MAX_CHUNKS = 64;        // n_chunks^2 bucket counters must fit a workgroup's LDS

// Node -> chunk: the random split, or a caller-supplied assignment (any partitioner's output).
struct ChunkMap {
    uint64_t seed;
    uint32_t c;
    const int32_t* assign;            // [N] chunk ids in [0, c), or null
};
__device__ __forceinline__ uint32_t chunk_of(const ChunkMap& m, int64_t v) {
    return m.assign ? (uint32_t)m.assign[v] : (uint32_t)(splitmix64_output(m.seed, (uint64_t)v) % m.c);
}

__global__ __launch_bounds__(256) void assignment_check_kernel(const int32_t* __restrict__ assign, int64_t N, int32_t c,
                                                               unsigned long long* __restrict__ bad) {
    unsigned long long b = 0;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < N; v += (int64_t)gridDim.x * 256)
        if (assign[v] < 0 || assign[v] >= c) b++;
    if (b) atomicAdd(bad, b);
}

// Pass 1: range check, global in-degrees, size of every (chunk(dst), chunk(src)) bucket.
__global__ __launch_bounds__(256) void chunk_count_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                          int64_t E, int64_t N, ChunkMap cm,
                                                          unsigned long long* __restrict__ dg,
                                                          unsigned long long* __restrict__ bucket_count,
                                                          unsigned long long* __restrict__ bad) {
    extern __shared__ unsigned int hist[];            // c*c counters of this workgroup
    const uint32_t c = cm.c;
    for (int i = threadIdx.x; i < (int)(c * c); i += 256) hist[i] = 0;
    __syncthreads();
    unsigned long long nbad = 0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < E; e += (int64_t)gridDim.x * 256) {
        const int64_t u = src[e], v = dst[e];
        if (u < 0 || v < 0 || u >= N || v >= N) { nbad++; continue; }
        atomicAdd(&dg[v], 1ull);
        atomicAdd(&hist[chunk_of(cm, v) * c + chunk_of(cm, u)], 1u);
    }
    if (nbad) atomicAdd(bad, nbad);
    __syncthreads();
    for (int i = threadIdx.x; i < (int)(c * c); i += 256)
        if (hist[i]) atomicAdd(&bucket_count[i], (unsigned long long)hist[i]);
}

// Pass 2: every workgroup reserves a run in each bucket for the edges it holds, then writes
// them (the order inside a bucket is arbitrary; partitions are sorted when they are built).
__global__ __launch_bounds__(256) void chunk_scatter_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst,
                                                            int64_t E, ChunkMap cm,
                                                            unsigned long long* __restrict__ cursor,
                                                            int64_t* __restrict__ out_src, int64_t* __restrict__ out_dst) {
    extern __shared__ unsigned int lds_u32[];         // [0, c*c): counts, then run starts (low / high words)
    const uint32_t c = cm.c;
    unsigned int* cnt = lds_u32;
    unsigned long long* start = (unsigned long long*)(lds_u32 + ((c * c + 1) & ~1u));
    const int64_t per = (E + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * per, hi = lo + per < E ? lo + per : E;
    for (int i = threadIdx.x; i < (int)(c * c); i += 256) cnt[i] = 0;
    __syncthreads();
    for (int64_t e = lo + threadIdx.x; e < hi; e += 256)
        atomicAdd(&cnt[chunk_of(cm, dst[e]) * c + chunk_of(cm, src[e])], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < (int)(c * c); i += 256) {
        start[i] = cnt[i] ? atomicAdd(&cursor[i], (unsigned long long)cnt[i]) : 0ull;
        cnt[i] = 0;
    }
    __syncthreads();
    for (int64_t e = lo + threadIdx.x; e < hi; e += 256) {
        const int64_t u = src[e], v = dst[e];
        const uint32_t b = chunk_of(cm, v) * c + chunk_of(cm, u);
        const unsigned long long slot = start[b] + atomicAdd(&cnt[b], 1u);
        out_src[slot] = u;
        out_dst[slot] = v;
    }
}

struct PairMember {
    ChunkMap cm;
    uint32_t base, swept;
    __device__ __forceinline__ bool operator()(int64_t v) const {
        const uint32_t ch = chunk_of(cm, v);
        return ch == base || ch == swept;
    }
};

__global__ __launch_bounds__(256) void pair_nodes_kernel(int64_t N, ChunkMap cm, uint32_t base, const uint32_t* __restrict__ bits,
                                                         const int32_t* __restrict__ before, uint2* __restrict__ words,
                                                         const int64_t* __restrict__ dg_all, int64_t* __restrict__ l2g, int64_t* __restrict__ dg,
                                                         uint8_t* __restrict__ base_mask) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= N) return;
    const uint2 w = set_word(bits, before, v, words);
    if (word_has(w, v)) {
        const int64_t i = word_rank(w, v);
        l2g[i] = v;
        dg[i] = dg_all[v];
        base_mask[i] = chunk_of(cm, v) == base ? 1 : 0;
    }
}

// Keys of the edges of up to four buckets (blockIdx.y; both endpoints are members by construction).  Four edges a thread: their
// lookups are in flight together (3.9e6 edges in four launches of one edge a thread, ids looked up in an 8-byte array over all nodes, 71
// us; this way 60).
struct PairBuckets { int64_t from[4], count[4], to[4]; };
__global__ __launch_bounds__(256) void bucket_keys_kernel(const int64_t* __restrict__ src, const int64_t* __restrict__ dst, PairBuckets b,
                                                          NodeSet set, uint64_t* __restrict__ keys) {
    constexpr int PER = 4;
    const int64_t count = b.count[blockIdx.y];
    const int64_t* const s = src + b.from[blockIdx.y];
    const int64_t* const d = dst + b.from[blockIdx.y];
    for (int64_t e0 = (int64_t)blockIdx.x * (256 * PER) + threadIdx.x; e0 < count; e0 += (int64_t)gridDim.x * (256 * PER)) {
        int64_t u[PER], v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t e = e0 + i * 256 < count ? e0 + i * 256 : count - 1;
            u[i] = s[e];
            v[i] = d[e];
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint64_t key = ((uint64_t)(uint32_t)set_rank(set, v[i]) << 32) | (uint64_t)(uint32_t)set_rank(set, u[i]);
            if (e0 + i * 256 < count) keys[b.to[blockIdx.y] + e0 + i * 256] = key;
        }
    }
}

static void free_chunks(grp_chunks_t* h) {
    if (!h) return;
    for (void* q : {(void*)h->src, (void*)h->dst, (void*)h->d_global_all, (void*)h->assign})
        if (q) pool_free(q);
    delete h;
}

static grp_status chunks_impl(const int64_t* src, const int64_t* dst, int64_t E, int64_t N, int32_t c, uint64_t seed,
                              const int32_t* assignment, hipStream_t st, grp_chunks_t* h) {
    const int nb = c * c;
    h->n_chunks = c; h->seed = seed; h->N = N; h->E = E;
    h->bucket_ptr.assign((size_t)nb + 1, 0);
    if (assignment) {                                  // keep a checked copy: partitions are built from it later
        GRP_TRY(halloc(&h->assign, N));
        GRP_HIP(hipMemcpyAsync(h->assign, assignment, (size_t)N * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
        DevBuf bad;
        GRP_TRY(bad.alloc(sizeof(unsigned long long)));
        GRP_HIP(hipMemsetAsync(bad.p, 0, sizeof(unsigned long long), st));
        unsigned long long host_bad = 0;
        if (N > 0) {
            hipLaunchKernelGGL(assignment_check_kernel, dim3(grid_for(N)), dim3(256), 0, st, (const int32_t*)h->assign, N, c,
                               bad.as<unsigned long long>());
            GRP_LAUNCH_CHECK();
        }
        GRP_HIP(hipMemcpyAsync(&host_bad, bad.p, sizeof host_bad, hipMemcpyDeviceToHost, st));
        GRP_HIP(hipStreamSynchronize(st));
        if (host_bad) return fail(GRP_ERANGE, "%llu nodes are assigned to a chunk outside [0, %d)", host_bad, c);
    }
    const ChunkMap cm{seed, (uint32_t)c, h->assign};
    GRP_TRY(halloc(&h->src, E));
    GRP_TRY(halloc(&h->dst, E));
    GRP_TRY(halloc(&h->d_global_all, N));
    GRP_HIP(hipMemsetAsync(h->d_global_all, 0, (size_t)(N > 0 ? N : 1) * sizeof(int64_t), st));
    DevBuf counters;                                   // [0, nb): counts then cursors; [nb]: bad ids
    GRP_TRY(counters.alloc((size_t)(nb + 1) * sizeof(unsigned long long)));
    GRP_HIP(hipMemsetAsync(counters.p, 0, (size_t)(nb + 1) * sizeof(unsigned long long), st));
    if (E == 0) { GRP_HIP(hipStreamSynchronize(st)); return GRP_OK; }
    const unsigned grid = grid_for(E) > 2048 ? 2048 : grid_for(E);
    hipLaunchKernelGGL(chunk_count_kernel, dim3(grid), dim3(256), (size_t)nb * sizeof(unsigned int), st, src, dst, E, N,
                       cm, (unsigned long long*)h->d_global_all, counters.as<unsigned long long>(),
                       counters.as<unsigned long long>() + nb);
    GRP_LAUNCH_CHECK();
    std::vector<unsigned long long> host((size_t)nb + 1);
    GRP_HIP(hipMemcpyAsync(host.data(), counters.p, host.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    GRP_HIP(hipStreamSynchronize(st));
    if (host[nb] != 0) return fail(GRP_ERANGE, "%llu edges have an endpoint outside [0, %lld)", host[nb], (long long)N);
    for (int b = 0; b < nb; ++b) h->bucket_ptr[b + 1] = h->bucket_ptr[b] + (int64_t)host[b];
    std::vector<unsigned long long> cur((size_t)nb);
    for (int b = 0; b < nb; ++b) cur[b] = (unsigned long long)h->bucket_ptr[b];
    GRP_HIP(hipMemcpyAsync(counters.p, cur.data(), cur.size() * sizeof(unsigned long long), hipMemcpyHostToDevice, st));
    const size_t lds = (size_t)((nb + 1) & ~1) * sizeof(unsigned int) + (size_t)nb * sizeof(unsigned long long);
    hipLaunchKernelGGL(chunk_scatter_kernel, dim3(grid), dim3(256), lds, st, src, dst, E, cm,
                       counters.as<unsigned long long>(), h->src, h->dst);
    GRP_LAUNCH_CHECK();
    GRP_HIP(hipStreamSynchronize(st));
    return GRP_OK;
}

static grp_status pair_partition_impl(const grp_chunks_t* ck, int32_t base, int32_t swept, hipStream_t st,
                                      grp_partition_t* h) {
    const int64_t N = ck->N;
    const int c = ck->n_chunks;
    const ChunkMap cm{ck->seed, (uint32_t)c, ck->assign};
    SetScratch t;
    DevBuf slab;
    GRP_TRY(t.alloc(N, slab));
    if (N >= ((int64_t)1 << 31)) GRP_HIP(hipMemsetAsync(t.counters, 0, 4 * sizeof(unsigned long long), st));
    int64_t n = 0;
    GRP_TRY(build_node_set(N, PairMember{cm, (uint32_t)base, (uint32_t)swept}, t, &n, st));
    if (n >= ((int64_t)1 << 31)) return fail(GRP_ERANGE, "partition has %lld >= 2^31 local nodes", (long long)n);
    h->n = n;
    GRP_TRY(halloc(&h->l2g, n));
    GRP_TRY(halloc(&h->d_global_in, n));
    GRP_TRY(halloc(&h->base_mask, n));
    const NodeSet set{t.words};
    if (N > 0) {
        hipLaunchKernelGGL(pair_nodes_kernel, dim3((unsigned)cdiv(N, 256)), dim3(256), 0, st, N, cm, (uint32_t)base, (const uint32_t*)t.bits,
                           (const int32_t*)t.before, t.words, ck->d_global_all, h->l2g, h->d_global_in, h->base_mask);
        GRP_LAUNCH_CHECK();
    }
    // the partition's edges are exactly the buckets (x, y) with x, y in {base, swept}
    int chunks2[2] = {base, swept};
    const int nc = base == swept ? 1 : 2;
    PairBuckets buckets{};
    int64_t nnz = 0, most = 0;
    for (int a = 0; a < nc; ++a)
        for (int b = 0; b < nc; ++b) {
            const int bk = chunks2[a] * c + chunks2[b], i = a * nc + b;
            buckets.from[i] = ck->bucket_ptr[bk];
            buckets.count[i] = ck->bucket_ptr[bk + 1] - ck->bucket_ptr[bk];
            buckets.to[i] = nnz;
            nnz += buckets.count[i];
            most = buckets.count[i] > most ? buckets.count[i] : most;
        }
    h->nnz = nnz;
    DevBuf keys, keys_alt;
    GRP_TRY(keys.alloc((size_t)nnz * sizeof(uint64_t)));
    GRP_TRY(keys_alt.alloc((size_t)nnz * sizeof(uint64_t)));
    if (nnz > 0) {
        hipLaunchKernelGGL(bucket_keys_kernel, dim3(grid_for(cdiv(most, 4)), nc * nc), dim3(256), 0, st, ck->src, ck->dst, buckets, set,
                           keys.as<uint64_t>());
        GRP_LAUNCH_CHECK();
    }
    return build_csr_csc(h, keys.as<uint64_t>(), keys_alt.as<uint64_t>(), st);
}

}  // namespace grp

extern "C" grp_status grp_chunks_build(const int64_t* src, const int64_t* dst, int64_t E, int64_t N, int32_t n_chunks,
                                       uint64_t seed, void* stream, grp_chunks_t** out) {
    using namespace grp;
    if (!out) return fail(GRP_EINVAL, "grp_chunks_build: out is null");
    *out = nullptr;
    if (E < 0 || N < 0) return fail(GRP_EINVAL, "grp_chunks_build: negative size");
    if (E > 0 && (!src || !dst)) return fail(GRP_EINVAL, "grp_chunks_build: null edge arrays");
    if (n_chunks < 1 || n_chunks > MAX_CHUNKS)
        return fail(GRP_EINVAL, "grp_chunks_build: n_chunks = %d outside [1, %d]", n_chunks, MAX_CHUNKS);
    grp_chunks_t* h = new (std::nothrow) grp_chunks_t();
    if (!h) return fail(GRP_ENOMEM, "grp_chunks_build: host allocation failed");
    (void)hipGetDevice(&h->device);
    const grp_status s = chunks_impl(src, dst, E, N, n_chunks, seed, nullptr, (hipStream_t)stream, h);
    if (s != GRP_OK) {
        free_chunks(h);
        return s;
    }
    *out = h;
    return GRP_OK;
}

extern "C" grp_status grp_chunks_build_assigned(const int64_t* src, const int64_t* dst, int64_t E, int64_t N,
                                                int32_t n_chunks, const int32_t* chunk_of_node, void* stream,
                                                grp_chunks_t** out) {
    using namespace grp;
    if (!out) return fail(GRP_EINVAL, "grp_chunks_build_assigned: out is null");
    *out = nullptr;
    if (E < 0 || N < 0) return fail(GRP_EINVAL, "grp_chunks_build_assigned: negative size");
    if (E > 0 && (!src || !dst)) return fail(GRP_EINVAL, "grp_chunks_build_assigned: null edge arrays");
    if (N > 0 && !chunk_of_node) return fail(GRP_EINVAL, "grp_chunks_build_assigned: null assignment");
    if (n_chunks < 1 || n_chunks > MAX_CHUNKS)
        return fail(GRP_EINVAL, "grp_chunks_build_assigned: n_chunks = %d outside [1, %d]", n_chunks, MAX_CHUNKS);
    grp_chunks_t* h = new (std::nothrow) grp_chunks_t();
    if (!h) return fail(GRP_ENOMEM, "grp_chunks_build_assigned: host allocation failed");
    (void)hipGetDevice(&h->device);
    const grp_status s = chunks_impl(src, dst, E, N, n_chunks, 0, chunk_of_node, (hipStream_t)stream, h);
    if (s != GRP_OK) {
        free_chunks(h);
        return s;
    }
    *out = h;
    return GRP_OK;
}

extern "C" grp_status grp_chunks_destroy(grp_chunks_t* chunks) {
    grp::free_chunks(chunks);
    return GRP_OK;
}

extern "C" grp_status grp_partition_from_chunks(const grp_chunks_t* chunks, int32_t base, int32_t swept, void* stream,
                                                grp_partition_t** out) {
    using namespace grp;
    if (!out) return fail(GRP_EINVAL, "grp_partition_from_chunks: out is null");
    *out = nullptr;
    if (!chunks) return fail(GRP_EINVAL, "grp_partition_from_chunks: chunks is null");
    if (base < 0 || base >= chunks->n_chunks || swept < 0 || swept >= chunks->n_chunks)
        return fail(GRP_EINVAL, "grp_partition_from_chunks: chunk ids (%d, %d) outside [0, %d)", base, swept, chunks->n_chunks);
    grp_partition_t* h = new (std::nothrow) grp_partition_t();
    if (!h) return fail(GRP_ENOMEM, "grp_partition_from_chunks: host allocation failed");
    (void)hipGetDevice(&h->device);
    const grp_status s = pair_partition_impl(chunks, base, swept, (hipStream_t)stream, h);
    if (s != GRP_OK) {
        free_partition(h);
        return s;
    }
    *out = h;
    return GRP_OK;
}

extern "C" grp_status grp_partition_halo(const int64_t* src, const int64_t* dst, int64_t E, int64_t N, int32_t K, uint64_t seed,
                                         int32_t part_id, int32_t hops, void* stream, grp_partition_t** out) {
    using namespace grp;
    if (!out) return fail(GRP_EINVAL, "grp_partition_halo: out is null");
    *out = nullptr;
    if (E < 0 || N < 0) return fail(GRP_EINVAL, "grp_partition_halo: negative size");
    if (E > 0 && (!src || !dst)) return fail(GRP_EINVAL, "grp_partition_halo: null edge arrays");
    if (K < 1) return fail(GRP_EINVAL, "grp_partition_halo: K = %d < 1", K);
    if (part_id < 0 || part_id >= K) return fail(GRP_EINVAL, "grp_partition_halo: part_id %d outside [0, %d)", part_id, K);
    if (hops < 1 || hops > GRP_MAX_LAYERS) return fail(GRP_EINVAL, "grp_partition_halo: hops = %d outside [1, %d]", hops, GRP_MAX_LAYERS);
    grp_partition_t* h = new (std::nothrow) grp_partition_t();
    if (!h) return fail(GRP_ENOMEM, "grp_partition_halo: host allocation failed");
    (void)hipGetDevice(&h->device);
    const grp_status s = halo_partition_impl(src, dst, E, N, K, seed, part_id, hops, (hipStream_t)stream, h);
    if (s != GRP_OK) {
        free_partition(h);
        return s;
    }
    *out = h;
    return GRP_OK;
}

extern "C" grp_status grp_partition_base_mask(const grp_partition_t* part, const uint8_t** mask) {
    if (!part || !mask) return grp::fail(GRP_EINVAL, "grp_partition_base_mask: null argument");
    *mask = part->base_mask;
    return GRP_OK;
}

extern "C" grp_status grp_partition(const int64_t* src, const int64_t* dst, int64_t E, int64_t N, int32_t K, uint64_t seed,
                                    int32_t part_id, void* stream, grp_partition_t** out) {
    using namespace grp;
    if (!out) return fail(GRP_EINVAL, "grp_partition: out is null");
    *out = nullptr;
    if (E < 0 || N < 0) return fail(GRP_EINVAL, "grp_partition: negative size");
    if (E > 0 && (!src || !dst)) return fail(GRP_EINVAL, "grp_partition: null edge arrays");
    if (K < 1) return fail(GRP_EINVAL, "grp_partition: K = %d < 1", K);
    if (part_id < 0 || part_id >= K) return fail(GRP_EINVAL, "grp_partition: part_id %d outside [0, %d)", part_id, K);
    grp_partition_t* h = new (std::nothrow) grp_partition_t();
    if (!h) return fail(GRP_ENOMEM, "grp_partition: host allocation failed");
    (void)hipGetDevice(&h->device);
    const grp_status s = partition_impl(src, dst, E, N, K, seed, part_id, (hipStream_t)stream, h);
    if (s != GRP_OK) {
        free_partition(h);
        return s;
    }
    *out = h;
    return GRP_OK;
}

extern "C" grp_status grp_node_owners(int64_t N, int32_t K, uint64_t seed, int32_t* owner_out, int64_t* count_out,
                                      void* stream) {
    using namespace grp;
    if (N < 0 || K < 1) return fail(GRP_EINVAL, "grp_node_owners: N = %lld, K = %d", (long long)N, K);
    if (N > 0 && !owner_out) return fail(GRP_EINVAL, "grp_node_owners: null output");
    hipStream_t st = (hipStream_t)stream;
    if (count_out) GRP_TRY(launch_fill_zero(count_out, (size_t)K * sizeof(int64_t), st));    // a kernel: the call can be captured in a graph
    if (N == 0) return GRP_OK;
    int64_t blocks = cdiv(N, 256 * 8);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(node_owners_kernel, dim3((unsigned)blocks), dim3(256), 0, st, N, (uint32_t)K, seed, owner_out,
                       (unsigned long long*)count_out);
    GRP_LAUNCH_CHECK();
    return GRP_OK;
}

namespace grp {
// ---- seed order of an epoch: the training nodes sorted by M(M(M(seed) ^ epoch) ^ global id), ties by local id
__global__ __launch_bounds__(256) void train_flag_kernel(const uint8_t* __restrict__ mask, int64_t n,
                                                         int32_t* __restrict__ flag /*[n+1]*/) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v > n) return;
    flag[v] = v < n && (!mask || mask[v] != 0) ? 1 : 0;
}

__global__ __launch_bounds__(256) void seed_keys_kernel(const int32_t* __restrict__ flag, const int32_t* __restrict__ pos,
                                                        const int64_t* __restrict__ l2g, int64_t n, uint64_t h,
                                                        uint64_t* __restrict__ keys, int32_t* __restrict__ ids) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= n || !flag[v]) return;
    keys[pos[v]] = mixM(h ^ (uint64_t)l2g[v]);           // slots ascend with the local id: the stable sort keeps ties in that order
    ids[pos[v]] = (int32_t)v;
}

// The same order for up to SEEDS_MOST nodes: the keys are as good as uniform, so their top bits deal them to buckets of 128 on average
// (if every node trains), and a workgroup ranks a bucket's keys against each other in LDS.  Three launches and one wait instead of
// eleven and two (a radix sort passes over all 8 bytes of the key however few there are).  Buckets beyond SEEDS_BUCKET keys (nodes that
// share a global id) are left to the sort.  A call, us, sort / buckets: 2500 nodes, half of them trained on 68/43; 1.5e5, 4 % 83/44, all
// 130/94; 5e5, 10 % 101/66; 2^19, all 219/159; but 1e6, all 259/288 (256 keys a bucket, each compared with each): the line is at 2^19.
// (Buckets of 64: 51 and 84 us at 1.5e5; of 256: 42 and 113.)
constexpr int64_t SEEDS_MOST = (int64_t)1 << 19;
constexpr int SEEDS_BUCKET = 2048;
constexpr int SEEDS_BITS = 12;           // 4096 buckets at most
struct SeedJob {
    const uint8_t* mask;
    const int64_t* l2g;
    int64_t n;
    uint64_t h;
    int bits;
    uint32_t *count, *taken;             // [2^bits] keys of a bucket, places given out in it
    uint64_t* keys;
    int32_t* ids;
    int32_t* out;
    int32_t* totals;                     // keys, keys of the largest bucket
};
__device__ __forceinline__ uint32_t seed_bucket(uint64_t key, int bits) { return bits ? (uint32_t)(key >> (64 - bits)) : 0u; }
__global__ __launch_bounds__(256) void seed_count_kernel(SeedJob j) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < j.n && (!j.mask || j.mask[v])) atomicAdd(&j.count[seed_bucket(mixM(j.h ^ (uint64_t)j.l2g[v]), j.bits)], 1u);
}
__global__ __launch_bounds__(256) void seed_place_kernel(SeedJob j) {
    __shared__ uint32_t at[1 << SEEDS_BITS];
    __shared__ uint32_t wave_sum[4];
    const int buckets = 1 << j.bits, tid = threadIdx.x;
    uint32_t before = 0, largest = 0;
    for (int b0 = 0; b0 < buckets; b0 += 256) {
        const uint32_t c = b0 + tid < buckets ? j.count[b0 + tid] : 0u;
        uint32_t all;
        const uint32_t first = block_scan<4>(c, wave_sum, all);
        if (b0 + tid < buckets) at[b0 + tid] = before + first;
        before += all;
        largest = c > largest ? c : largest;
    }
    __syncthreads();
    if (blockIdx.x == 0) {
        if (tid == 0) j.totals[0] = (int32_t)before;
        atomicMax(&j.totals[1], (int32_t)largest);
    }
    const int64_t v = (int64_t)blockIdx.x * 256 + tid;
    if (v >= j.n || (j.mask && !j.mask[v])) return;
    const uint64_t key = mixM(j.h ^ (uint64_t)j.l2g[v]);
    const uint32_t b = seed_bucket(key, j.bits), to = at[b] + atomicAdd(&j.taken[b], 1u);
    j.keys[to] = key;
    j.ids[to] = (int32_t)v;
}
__global__ __launch_bounds__(256) void seed_rank_kernel(SeedJob j) {
    __shared__ uint64_t key_s[SEEDS_BUCKET];
    __shared__ int32_t id_s[SEEDS_BUCKET];
    __shared__ uint32_t sums[4];
    const int b = blockIdx.x, tid = threadIdx.x, m = (int)j.count[b];
    uint32_t before = 0;
    for (int q = tid; q < b; q += 256) before += j.count[q];
    uint32_t base;
    block_scan<4>(before, sums, base);
    if (m > SEEDS_BUCKET) return;
    for (int i = tid; i < m; i += 256) {
        key_s[i] = j.keys[base + i];
        id_s[i] = j.ids[base + i];
    }
    __syncthreads();
    for (int i = tid; i < m; i += 256) {
        const uint64_t key = key_s[i];
        const int32_t id = id_s[i];
        int rank = 0;
        for (int q = 0; q < m; ++q) rank += key_s[q] < key || (key_s[q] == key && id_s[q] < id) ? 1 : 0;
        j.out[base + rank] = id;
    }
}

// done: false if a bucket was too large (seeds_out is then unfinished).
static grp_status seeds_by_buckets(const grp_partition_t* part, const uint8_t* mask, uint64_t h, hipStream_t st, int32_t* seeds_out,
                                   int64_t* n_seeds_out, bool* done) {
    const int64_t n = part->n;
    int bits = 0;
    while (bits < SEEDS_BITS && ((int64_t)128 << bits) < n) ++bits;
    const size_t buckets = (size_t)1 << bits;
    DevBuf keys, ids, counts;
    GRP_TRY(keys.alloc((size_t)n * sizeof(uint64_t)));
    GRP_TRY(ids.alloc((size_t)n * sizeof(int32_t)));
    const size_t words = 2 * buckets + 2;
    GRP_TRY(counts.alloc(words * sizeof(uint32_t)));
    uint32_t* const c = counts.as<uint32_t>();
    GRP_TRY(launch_fill_zero(c, words * sizeof(uint32_t), st));
    const SeedJob j{mask, part->l2g, n, h, bits, c, c + buckets, keys.as<uint64_t>(), ids.as<int32_t>(), seeds_out, (int32_t*)(c + 2 * buckets)};
    hipLaunchKernelGGL(seed_count_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, j);
    hipLaunchKernelGGL(seed_place_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, j);
    hipLaunchKernelGGL(seed_rank_kernel, dim3((unsigned)buckets), dim3(256), 0, st, j);
    GRP_LAUNCH_CHECK();
    int32_t totals[2] = {0, 0};
    GRP_HIP(hipMemcpyAsync(totals, j.totals, sizeof totals, hipMemcpyDeviceToHost, st));
    GRP_HIP(hipStreamSynchronize(st));                   // (the temporaries are released on return)
    *done = totals[1] <= SEEDS_BUCKET;
    if (*done) *n_seeds_out = totals[0];
    return GRP_OK;
}
}  // namespace grp

extern "C" grp_status grp_epoch_seeds(const grp_partition_t* part, const uint8_t* train_mask, uint64_t sampler_seed,
                                      uint64_t epoch, void* stream, int32_t* seeds_out, int64_t* n_seeds_out) {
    using namespace grp;
    if (!part || !n_seeds_out) return fail(GRP_EINVAL, "grp_epoch_seeds: null argument");
    *n_seeds_out = 0;
    const int64_t n = part->n;
    if (n == 0) return GRP_OK;
    if (!seeds_out) return fail(GRP_EINVAL, "grp_epoch_seeds: null output");
    hipStream_t st = (hipStream_t)stream;
    const uint64_t h = mixM(mixM(sampler_seed) ^ epoch);
    if (n <= SEEDS_MOST) {
        bool done = false;
        GRP_TRY(seeds_by_buckets(part, train_mask, h, st, seeds_out, n_seeds_out, &done));
        if (done) return GRP_OK;
    }
    DevBuf flag, pos, keys, keys_alt, ids, tmp;
    GRP_TRY(flag.alloc(((size_t)n + 1) * sizeof(int32_t)));
    GRP_TRY(pos.alloc(((size_t)n + 1) * sizeof(int32_t)));
    GRP_TRY(keys.alloc((size_t)n * sizeof(uint64_t)));
    GRP_TRY(keys_alt.alloc((size_t)n * sizeof(uint64_t)));
    GRP_TRY(ids.alloc((size_t)n * sizeof(int32_t)));
    size_t sort_bytes = 0;
    GRP_HIP(rocprim::radix_sort_pairs(nullptr, sort_bytes, keys.as<uint64_t>(), keys_alt.as<uint64_t>(), ids.as<int32_t>(),
                                      seeds_out, (size_t)n, 0u, 64u, st));
    const size_t scan_bytes = scan_temp_bytes(n + 1);
    GRP_TRY(tmp.alloc(sort_bytes > scan_bytes ? sort_bytes : scan_bytes));
    hipLaunchKernelGGL(train_flag_kernel, dim3((unsigned)cdiv(n + 1, 256)), dim3(256), 0, st, train_mask, n, flag.as<int32_t>());
    GRP_LAUNCH_CHECK();
    GRP_TRY(exclusive_scan_i32(tmp.p, scan_bytes, flag.as<int32_t>(), pos.as<int32_t>(), n + 1, st));
    hipLaunchKernelGGL(seed_keys_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, (const int32_t*)flag.as<int32_t>(),
                       (const int32_t*)pos.as<int32_t>(), part->l2g, n, h, keys.as<uint64_t>(),
                       ids.as<int32_t>());
    GRP_LAUNCH_CHECK();
    int32_t total = 0;
    GRP_HIP(hipMemcpyAsync(&total, pos.as<int32_t>() + n, sizeof total, hipMemcpyDeviceToHost, st));
    GRP_HIP(hipStreamSynchronize(st));
    if (total > 0) {
        GRP_HIP(rocprim::radix_sort_pairs(tmp.p, sort_bytes, keys.as<uint64_t>(), keys_alt.as<uint64_t>(), ids.as<int32_t>(),
                                          seeds_out, (size_t)total, 0u, 64u, st));
        GRP_HIP(hipStreamSynchronize(st));               // the temporaries are released on return
    }
    *n_seeds_out = total;
    return GRP_OK;
}

extern "C" grp_status grp_partition_weighted(const int64_t* src, const int64_t* dst, const float* w, int64_t E, int64_t N,
                                             int32_t K, uint64_t seed, int32_t part_id, void* stream,
                                             grp_partition_t** out) {
    using namespace grp;
    if (!out) return fail(GRP_EINVAL, "grp_partition_weighted: out is null");
    *out = nullptr;
    if (E < 0 || N < 0) return fail(GRP_EINVAL, "grp_partition_weighted: negative size");
    if (E > 0 && (!src || !dst)) return fail(GRP_EINVAL, "grp_partition_weighted: null edge arrays");
    if (E > 0 && !w) return fail(GRP_EINVAL, "grp_partition_weighted: null weights");
    if (K < 1) return fail(GRP_EINVAL, "grp_partition_weighted: K = %d < 1", K);
    if (part_id < 0 || part_id >= K)
        return fail(GRP_EINVAL, "grp_partition_weighted: part_id %d outside [0, %d)", part_id, K);
    grp_partition_t* h = new (std::nothrow) grp_partition_t();
    if (!h) return fail(GRP_ENOMEM, "grp_partition_weighted: host allocation failed");
    (void)hipGetDevice(&h->device);
    const grp_status s = partition_impl(src, dst, E, N, K, seed, part_id, (hipStream_t)stream, h, w, true);
    if (s != GRP_OK) {
        free_partition(h);
        return s;
    }
    *out = h;
    return GRP_OK;
}

extern "C" grp_status grp_partition_weights(const grp_partition_t* part, grp_partition_weights_t* view) {
    if (!part || !view) return grp::fail(GRP_EINVAL, "grp_partition_weights: null argument");
    view->csr_w = part->csr_w;
    view->csc_w = part->csc_w;
    view->w_local_in = part->w_local_in;
    view->w_global_in = part->w_global_in;
    return GRP_OK;
}

extern "C" grp_status grp_partition_from_local_coo(const int64_t* src_local, const int64_t* dst_local, int64_t E, int64_t n,
                                                   const int64_t* d_global_in, const int64_t* l2g, void* stream,
                                                   grp_partition_t** out) {
    using namespace grp;
    if (!out) return fail(GRP_EINVAL, "grp_partition_from_local_coo: out is null");
    *out = nullptr;
    if (E < 0 || n < 0) return fail(GRP_EINVAL, "grp_partition_from_local_coo: negative size");
    if (E > 0 && (!src_local || !dst_local)) return fail(GRP_EINVAL, "grp_partition_from_local_coo: null edge arrays");
    if (n >= ((int64_t)1 << 31)) return fail(GRP_ERANGE, "n = %lld >= 2^31", (long long)n);
    hipStream_t st = (hipStream_t)stream;
    grp_partition_t* h = new (std::nothrow) grp_partition_t();
    if (!h) return fail(GRP_ENOMEM, "host allocation failed");
    (void)hipGetDevice(&h->device);
    h->n = n;
    h->nnz = E;
    auto body = [&]() -> grp_status {
        DevBuf keys, keys_alt, bad;
        GRP_TRY(keys.alloc((size_t)E * sizeof(uint64_t)));
        GRP_TRY(keys_alt.alloc((size_t)E * sizeof(uint64_t)));
        GRP_TRY(bad.alloc(sizeof(unsigned long long)));
        GRP_HIP(hipMemsetAsync(bad.p, 0, sizeof(unsigned long long), st));
        if (E > 0) {
            hipLaunchKernelGGL(local_keys_kernel, dim3(grid_for(E)), dim3(256), 0, st, src_local, dst_local, E, n,
                               keys.as<uint64_t>(), bad.as<unsigned long long>());
            GRP_LAUNCH_CHECK();
        }
        unsigned long long nbad = 0;
        GRP_HIP(hipMemcpyAsync(&nbad, bad.p, sizeof nbad, hipMemcpyDeviceToHost, st));
        GRP_HIP(hipStreamSynchronize(st));
        if (nbad) return fail(GRP_ERANGE, "%llu edges have an endpoint outside [0, %lld)", nbad, (long long)n);
        GRP_TRY(build_csr_csc(h, keys.as<uint64_t>(), keys_alt.as<uint64_t>(), st));
        GRP_TRY(halloc(&h->l2g, n));
        GRP_TRY(halloc(&h->d_global_in, n));
        if (n > 0) {
            const unsigned g = (unsigned)cdiv(n, 256);
            if (l2g) GRP_HIP(hipMemcpyAsync(h->l2g, l2g, (size_t)n * sizeof(int64_t), hipMemcpyDeviceToDevice, st));
            else hipLaunchKernelGGL(iota_kernel, dim3(g), dim3(256), 0, st, n, h->l2g);
            if (d_global_in)
                GRP_HIP(hipMemcpyAsync(h->d_global_in, d_global_in, (size_t)n * sizeof(int64_t), hipMemcpyDeviceToDevice, st));
            else hipLaunchKernelGGL(widen_kernel, dim3(g), dim3(256), 0, st, h->d_local_in, n, h->d_global_in);
            GRP_LAUNCH_CHECK();
        }
        GRP_HIP(hipStreamSynchronize(st));
        return GRP_OK;
    };
    const grp_status s = body();
    if (s != GRP_OK) {
        free_partition(h);
        return s;
    }
    *out = h;
    return GRP_OK;
}

extern "C" grp_status grp_partition_view(const grp_partition_t* part, grp_partition_view_t* view) {
    if (!part || !view) return grp::fail(GRP_EINVAL, "grp_partition_view: null argument");
    view->n = part->n;
    view->nnz = part->nnz;
    view->l2g = part->l2g;
    view->rowptr = part->rowptr;
    view->col = part->col;
    view->colptr = part->colptr;
    view->row = part->row;
    view->d_local_in = part->d_local_in;
    view->d_local_out = part->d_local_out;
    view->d_global_in = part->d_global_in;
    return GRP_OK;
}

extern "C" grp_status grp_partition_destroy(grp_partition_t* part) {
    grp::free_partition(part);
    return GRP_OK;
}

// ------------------------------------------------------------------ shared device primitives
namespace grp {

size_t scan_temp_bytes(int64_t count) {
    size_t bytes = 0;
    (void)rocprim::exclusive_scan(nullptr, bytes, (const int64_t*)nullptr, (int64_t*)nullptr, (int64_t)0,
                                  (size_t)(count > 0 ? count : 1), rocprim::plus<int64_t>(), (hipStream_t)0);
    return bytes + 256;
}

grp_status exclusive_scan_i64(void* temp, size_t temp_bytes, const int64_t* in, int64_t* out, int64_t count,
                              hipStream_t st) {
    if (count <= 0) return GRP_OK;
    size_t need = 0;
    GRP_HIP(rocprim::exclusive_scan(nullptr, need, in, out, (int64_t)0, (size_t)count, rocprim::plus<int64_t>(), st));
    if (need > temp_bytes) return fail(GRP_EWORKSPACE, "scan temp %zu < %zu", temp_bytes, need);
    GRP_HIP(rocprim::exclusive_scan(temp, need, in, out, (int64_t)0, (size_t)count, rocprim::plus<int64_t>(), st));
    return GRP_OK;
}

grp_status exclusive_scan_i32(void* temp, size_t temp_bytes, const int32_t* in, int32_t* out, int64_t count,
                              hipStream_t st) {
    if (count <= 0) return GRP_OK;
    size_t need = 0;
    GRP_HIP(rocprim::exclusive_scan(nullptr, need, in, out, (int32_t)0, (size_t)count, rocprim::plus<int32_t>(), st));
    if (need > temp_bytes) return fail(GRP_EWORKSPACE, "scan temp %zu < %zu", temp_bytes, need);
    GRP_HIP(rocprim::exclusive_scan(temp, need, in, out, (int32_t)0, (size_t)count, rocprim::plus<int32_t>(), st));
    return GRP_OK;
}

struct PopcountOf {
    __host__ __device__ int32_t operator()(uint32_t w) const {
#if defined(__HIP_DEVICE_COMPILE__)
        return __popc(w);
#else
        return __builtin_popcount(w);
#endif
    }
};

// out[i] = number of set bits in words[0 .. i), for i in [0, count)
grp_status exclusive_scan_popcount(void* temp, size_t temp_bytes, const uint32_t* words, int32_t* out, int64_t count,
                                   hipStream_t st) {
    if (count <= 0) return GRP_OK;
    auto in = rocprim::make_transform_iterator(words, PopcountOf());
    size_t need = 0;
    GRP_HIP(rocprim::exclusive_scan(nullptr, need, in, out, (int32_t)0, (size_t)count, rocprim::plus<int32_t>(), st));
    if (need > temp_bytes) return fail(GRP_EWORKSPACE, "scan temp %zu < %zu", temp_bytes, need);
    GRP_HIP(rocprim::exclusive_scan(temp, need, in, out, (int32_t)0, (size_t)count, rocprim::plus<int32_t>(), st));
    return GRP_OK;
}

// ---- split schedule of the long rows, built on the device (no host pass, no synchronisation).
// The exclusive prefix sum of (1 << 32 | chunks of row r) for a long row, 0 otherwise, gives every
// long row its slot (high half) and first chunk (low half), in ascending row order.
struct LongRowPack {
    const int64_t* ptr;
    int64_t n;
    __host__ __device__ int64_t operator()(int64_t r) const {
        if (r >= n) return 0;
        const int64_t len = ptr[r + 1] - ptr[r];
        return len > SPMM_LONG_ROW ? (((int64_t)1 << 32) | ((len + SPMM_CHUNK - 1) / SPMM_CHUNK)) : 0;
    }
};

// Slots past the real counts are made harmless: row -1 (skipped by the combine pass), empty chunks.
__global__ __launch_bounds__(256) void long_rows_emit_kernel(const int64_t* __restrict__ ptr, int64_t n,
                                                             const int64_t* __restrict__ scanned /*[n+1]*/,
                                                             int64_t cap_long, int64_t cap_chunks,
                                                             int32_t* __restrict__ long_row, int32_t* __restrict__ long_first,
                                                             int64_t* __restrict__ chunk_begin, int64_t* __restrict__ chunk_end) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t total = scanned[n];
    const int64_t n_long = total >> 32, n_chunks = total & 0xFFFFFFFFll;
    if (r < n) {
        const int64_t b = ptr[r], e = ptr[r + 1];
        if (e - b > SPMM_LONG_ROW) {
            const int64_t slot = scanned[r] >> 32;
            int64_t c = scanned[r] & 0xFFFFFFFFll;
            if (slot < cap_long) {
                long_row[slot] = (int32_t)r;
                long_first[slot] = (int32_t)c;
            }
            for (int64_t at = b; at < e; at += SPMM_CHUNK, ++c) {
                if (c >= cap_chunks) break;
                chunk_begin[c] = at;
                chunk_end[c] = at + SPMM_CHUNK < e ? at + SPMM_CHUNK : e;
            }
        }
    }
    if (r >= n_long && r <= cap_long) {
        if (r < cap_long) long_row[r] = -1;
        long_first[r] = (int32_t)(n_chunks < cap_chunks ? n_chunks : cap_chunks);
    }
    if (r >= n_chunks && r < cap_chunks) { chunk_begin[r] = 0; chunk_end[r] = 0; }
}

grp_status build_long_rows_device(const int64_t* ptr_dev, int64_t n, LongRows* out, int64_t cap_long, int64_t cap_chunks,
                                  int64_t* scanned, void* scan_tmp, size_t scan_bytes, hipStream_t st) {
    {
        auto in = rocprim::make_transform_iterator(rocprim::make_counting_iterator<int64_t>(0), LongRowPack{ptr_dev, n});
        size_t need = 0;
        GRP_HIP(rocprim::exclusive_scan(nullptr, need, in, scanned, (int64_t)0, (size_t)(n + 1), rocprim::plus<int64_t>(), st));
        if (need > scan_bytes) return fail(GRP_EWORKSPACE, "scan temp %zu < %zu", scan_bytes, need);
        GRP_HIP(rocprim::exclusive_scan(scan_tmp, need, in, scanned, (int64_t)0, (size_t)(n + 1), rocprim::plus<int64_t>(), st));
    }
    int64_t work = n;
    if (cap_long + 1 > work) work = cap_long + 1;
    if (cap_chunks > work) work = cap_chunks;
    hipLaunchKernelGGL(long_rows_emit_kernel, dim3((unsigned)cdiv(work, 256)), dim3(256), 0, st, ptr_dev, n,
                       (const int64_t*)scanned, cap_long, cap_chunks, out->long_row, out->long_first, out->chunk_begin,
                       out->chunk_end);
    GRP_LAUNCH_CHECK();
    out->n_long = (int32_t)cap_long;          // upper bounds: the launches cover them, the device arrays say which are real
    out->n_chunks = (int32_t)cap_chunks;
    return GRP_OK;
}

}  // namespace grp
