// Row-parallel neighbour aggregation (SpMM) for gfx950.
//
// Y[i,:] = a_i (sum_{e in row i} w_e c_{idx[e]} X[idx[e],:] + self * X[i,:]) (+ addend[i,:]) (+ bias) (ReLU)
// (w_e: optional per-edge values, the weighted-mean aggregator of weighted partitions)
//
// The same kernels serve the forward pass (rows of the CSR: destinations gathering their
// in-neighbours) and the backward pass (rows of the CSC: the transposed operator), so no
// floating-point atomics are needed and results are bit-reproducible.
//
// Mapping: a group of G lanes (G = 1..64, a power of two) owns one output row; lane t of
// the group owns columns 4*(t + G*j), j < NJ, as one 16-byte vector, so a group's gather of
// one neighbour row is a single fully coalesced request of F*sizeof(elem) bytes.  The
// group's lanes fetch G column indices with one coalesced load and hand them round with
// wavefront shuffles; four neighbour rows are requested before any is accumulated so that
// several gathers are in flight per lane.
//
// Degree skew: rows longer than SPMM_LONG_ROW edges are cut, when the partition is built,
// into chunks of at most SPMM_CHUNK edges.  A workgroup owns a chunk (its 256/G groups take
// contiguous slices and are summed through LDS in a fixed order) and writes one partial row;
// a third kernel adds a row's partials in chunk order and applies the epilogue.  The split
// depends only on the graph, so results do not depend on scheduling.
#include "common.h"

#include <mutex>
#include <type_traits>

namespace grp {

// Rows of X may start at any element: the vector loads below ask for no more than the element's own alignment (the hardware takes
// them at the full rate when the address happens to be 16-byte friendly, which it is for every pitch of whole vectors).
// A row of F columns whose pitch leaves no room for its last, partial vector is read with that vector moved back to end at the
// row's last element (SpmmEpilogue::last_x): the lane that owns it sums columns F-4 .. F-1 and turns them into place when
// the row is finished.
// (1e5 rows of 75 fp32 columns packed without padding, 1.4e6 edges: 1090 us a sweep with one lane per column, 73 us this way.)

template <typename T> struct Vec4Load;
template <> struct Vec4Load<float> {
    static __device__ __forceinline__ float4 ld(const float* p) {
        const u32x4_any r = *reinterpret_cast<const u32x4_any*>(p);
        return make_float4(__uint_as_float(r.x), __uint_as_float(r.y), __uint_as_float(r.z), __uint_as_float(r.w));
    }
};
template <> struct Vec4Load<__hip_bfloat16> {
    static __device__ __forceinline__ float4 ld(const __hip_bfloat16* p) {
        const u32x2_any r = *reinterpret_cast<const u32x2_any*>(p);
        float4 v;
        v.x = __uint_as_float(r.x << 16);
        v.y = __uint_as_float(r.x & 0xFFFF0000u);
        v.z = __uint_as_float(r.y << 16);
        v.w = __uint_as_float(r.y & 0xFFFF0000u);
        return v;
    }
};


__device__ __forceinline__ float row_scale(int mode, int64_t deg, int self_term) {
    if (mode == GRP_SCALE_MEAN) return 1.0f / (float)(deg > 1 ? deg : 1);
    if (mode == GRP_SCALE_RSQRT) {
        int64_t d = deg + self_term;
        return 1.0f / sqrtf((float)(d > 1 ? d : 1));
    }
    return 1.0f;
}

__device__ __forceinline__ void axpy4(float4& acc, float s, const float4& v) {
    acc.x = fmaf(s, v.x, acc.x); acc.y = fmaf(s, v.y, acc.y);
    acc.z = fmaf(s, v.z, acc.z); acc.w = fmaf(s, v.w, acc.w);
}
__device__ __forceinline__ void add4(float4& acc, const float4& v) {
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
}

// Sum of X rows over the edges [b, e), taken by S groups of G lanes (this one is number gi; lane t of its group; tl = gi * G + t).
// EV: every edge carries a value val[e] that multiplies its gathered row.
// The S * G lanes fetch a batch of column indices with one load (or U / G of them, where that is more than one: a batch holds at
// least one step of every group); edge k of the batch belongs to group k % S.  A group requests U of its rows before it
// adds any; places past the batch's end read its last row again (a hit in L1) and add zeros in its place (a select: 0 times an
// infinity would be NaN).  Fetched one by one, the last few rows of every batch cost a memory latency each, and narrow groups
// had no full step at all.
// A lone group of wide rows takes the last rows of a batch singly: a repeated gather of 512 bytes is not free (3.25 edges a row:
// F = 256 181 us, with repeats 185; F = 100 87 and 91; bf16 F = 128 83 and 86; but F = 47 67 us singly and 63 with repeats).
// WIDE (bf16 rows of whole 16-byte units, NJ = 2): a lane owns eight consecutive columns, fetched with one 16-byte load
// and kept as two adjacent 4-column slabs, so a row takes half the lanes and a wavefront gathers twice the rows.
template <int G, bool WIDE> __device__ __forceinline__ int slab_col(int t, int j) { return WIDE ? 8 * t + 4 * j : 4 * (t + G * j); }
__device__ __forceinline__ void bf16x8_to_float4s(const uint4& r, float4& lo, float4& hi) {
    lo = make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xFFFF0000u), __uint_as_float(r.y << 16),
                     __uint_as_float(r.y & 0xFFFF0000u));
    hi = make_float4(__uint_as_float(r.z << 16), __uint_as_float(r.z & 0xFFFF0000u), __uint_as_float(r.w << 16),
                     __uint_as_float(r.w & 0xFFFF0000u));
}
template <typename XT, int G, int S, int NJ, bool EV, bool WIDE = false>
__device__ __forceinline__ void gather_rows(const int32_t* __restrict__ idx, const float* __restrict__ val, int64_t b,
                                            int64_t e, const XT* __restrict__ X, int64_t ldx,
                                            const float* __restrict__ colscale, int t, int gi, const bool (&live)[NJ],
                                            const int (&colx)[NJ], float4 (&acc)[NJ]) {
    static_assert(!WIDE || (NJ == 2 && sizeof(XT) == 2), "eight bf16 columns per lane");
    constexpr int L = G * S;                               // lanes of a row
    constexpr int U = 4;                                   // (8: no faster for any width, with these batches)
    constexpr bool SINGLY = S == 1 && (G >= 32 || (WIDE && G >= 8));      // no places past a batch's end: its last rows one by one
    constexpr int Q = G < U ? U / G : 1;                   // indices per lane: a batch of L * Q holds at least one step of every group
    for (int64_t base = b; base < e; base += L * Q) {
        const int cnt = (int)((e - base) < (int64_t)(L * Q) ? (e - base) : (int64_t)(L * Q));
        int mine[Q];
        float minew[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int tl = q * L + gi * G + t;
            const int64_t at = base + (tl < cnt ? tl : cnt - 1);
            mine[q] = idx[at];
            minew[q] = EV ? val[at] : 1.f;
        }
        auto step = [&](auto uc, int k) {                  // the group's rows k .. k + UC - 1 of the batch
            constexpr int UC = decltype(uc)::value;
            int64_t c[UC];
            float sc[UC];
            bool on[UC];
#pragma unroll
            for (int u = 0; u < UC; ++u) {
                const int pos = (k + u) * S + gi;
                on[u] = SINGLY || pos < cnt;
                // Q > 1: k is 0 and place u lies in register u / G (a place past the end reads a copy of the last index)
                const int q = Q > 1 ? u / G : 0;
                const int from = Q > 1 ? pos - q * L : on[u] ? pos : cnt - 1;
                c[u] = __shfl(mine[q], from, L);
                sc[u] = colscale ? colscale[c[u]] : 1.f;
                if (EV) sc[u] *= __shfl(minew[q], from, L);
                sc[u] = on[u] ? sc[u] : 0.f;
            }
            if constexpr (WIDE) {
                if (live[0]) {                             // F is a multiple of 8: both slabs are live or neither
                    uint4 r[UC];
#pragma unroll
                    for (int u = 0; u < UC; ++u) r[u] = *reinterpret_cast<const uint4*>(X + c[u] * ldx + 8 * t);
#pragma unroll
                    for (int u = 0; u < UC; ++u) {
                        if (!SINGLY) r[u] = on[u] ? r[u] : make_uint4(0u, 0u, 0u, 0u);
                        float4 lo, hi;
                        bf16x8_to_float4s(r[u], lo, hi);
                        axpy4(acc[0], sc[u], lo); axpy4(acc[1], sc[u], hi);
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if (!live[j]) continue;
                    float4 v[UC];
#pragma unroll
                    for (int u = 0; u < UC; ++u) v[u] = Vec4Load<XT>::ld(X + c[u] * ldx + colx[j]);
#pragma unroll
                    for (int u = 0; u < UC; ++u) {
                        if (!SINGLY) v[u] = make_float4(on[u] ? v[u].x : 0.f, on[u] ? v[u].y : 0.f, on[u] ? v[u].z : 0.f, on[u] ? v[u].w : 0.f);
                        axpy4(acc[j], sc[u], v[u]);        // x * 1 + acc rounds once, as x + acc does
                    }
                }
            }
        };
        int k = 0;
        if constexpr (SINGLY) {
            for (; k + U <= cnt; k += U) step(std::integral_constant<int, U>(), k);
            for (; k < cnt; ++k) step(std::integral_constant<int, 1>(), k);
        } else {
            for (; k * S < cnt; k += U) step(std::integral_constant<int, U>(), k);
        }
    }
}

struct SpmmEpilogue {
    int scale, self_term, relu, F;
    const float* addend;      // may alias Y
    int64_t ld_add;
    const float* bias;
    float* Y;
    int64_t ldy;
    const float* residual;    // added after the ReLU (residual layers); null otherwise
    int64_t ld_res;
    float* Y2;                // receives the activation before the residual is added; null otherwise
    int64_t ldy2;
    int64_t addend_rows;      // rows >= this have no addend
    const float* mask;        // keep where mask > 0 (after the ReLU); null otherwise
    int64_t ld_mask;
    const float* rowscale;    // a_i given explicitly; null: from `scale` and the row length
    const int64_t* n_rows_dev;       // when set: the real row count and the real addend_rows (device values;
    const int64_t* addend_rows_dev;  //           the launch and addend_rows above are upper bounds)
    int last_x;               // no vector of an X row starts past this column
    int tight;                // bit 0: last_x is not a whole number of vectors; bit 1: Y or the addend take no 16-byte vectors
};

template <typename XT>
__device__ __forceinline__ void finish_row(const SpmmEpilogue& ep, int64_t i, int64_t deg, int col, float4 r,
                                           const XT* __restrict__ X, int64_t ldx) {
    const float a = ep.rowscale ? ep.rowscale[i] : row_scale(ep.scale, deg, ep.self_term);
    if (ep.tight) {                                          // (uniform)
        if (ep.self_term) add4(r, Vec4Load<XT>::ld(X + i * ldx + imin(col, ep.last_x)));
        if (col > ep.last_x) {                               // the row's last vector was moved back: turn it into place
            const int by = col - ep.last_x;
            r = by == 1 ? make_float4(r.y, r.z, r.w, 0.f) : by == 2 ? make_float4(r.z, r.w, 0.f, 0.f) : make_float4(r.w, 0.f, 0.f, 0.f);
        }
        if (ep.tight & 2) {                                  // Y or the addend take no vectors
            const float o[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (col + q >= ep.F) break;
                float y = o[q] * a;
                if (ep.addend) y += ep.addend[i * ep.ld_add + col + q];
                if (ep.bias) y += ep.bias[col + q];
                if (ep.relu) y = y > 0.f ? y : 0.f;
                ep.Y[i * ep.ldy + col + q] = y;
            }
            return;
        }
    } else if (ep.self_term) {
        add4(r, Vec4Load<XT>::ld(X + i * ldx + col));
    }
    r.x *= a; r.y *= a; r.z *= a; r.w *= a;
    if (ep.addend && i < (ep.addend_rows_dev ? *ep.addend_rows_dev : ep.addend_rows)) add4(r, *reinterpret_cast<const float4*>(ep.addend + i * ep.ld_add + col));
    float o[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (col + q < ep.F) {
            if (ep.bias) o[q] += ep.bias[col + q];
            if (ep.relu) o[q] = o[q] > 0.f ? o[q] : 0.f;
        } else {
            o[q] = 0.f;           // pad columns stay zero
        }
    }
    if (ep.mask) {
        const float4 mk = *reinterpret_cast<const float4*>(ep.mask + i * ep.ld_mask + col);
        o[0] = mk.x > 0.f ? o[0] : 0.f; o[1] = mk.y > 0.f ? o[1] : 0.f;
        o[2] = mk.z > 0.f ? o[2] : 0.f; o[3] = mk.w > 0.f ? o[3] : 0.f;
    }
    if (ep.Y2) *reinterpret_cast<float4*>(ep.Y2 + i * ep.ldy2 + col) = make_float4(o[0], o[1], o[2], o[3]);
    if (ep.residual) {
        const float4 h = *reinterpret_cast<const float4*>(ep.residual + i * ep.ld_res + col);
        o[0] += h.x; o[1] += h.y; o[2] += h.z; o[3] += h.w;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (col + q >= ep.F) o[q] = 0.f;
    }
    *reinterpret_cast<float4*>(ep.Y + i * ep.ldy + col) = make_float4(o[0], o[1], o[2], o[3]);
}

// One workgroup per chunk of a long row -> one partial row.
template <typename XT, int G, int NJ, bool EV, bool WIDE = false>
__device__ __forceinline__ void chunk_body(int64_t cb, int64_t ce, const int32_t* __restrict__ idx,
                                           const float* __restrict__ val, int F, int last_x,
                                           const XT* __restrict__ X, int64_t ldx, const float* __restrict__ colscale,
                                           float* __restrict__ part_row, float* red) {
    constexpr int NG = 256 / G;
    constexpr int W = 4 * G * NJ;                 // padded row width held by a group
    const int t = threadIdx.x % G, gi = threadIdx.x / G;
    const int64_t per = (ce - cb + NG - 1) / NG;
    int64_t b = cb + gi * per, e = b + per;
    if (b > ce) b = ce;
    if (e > ce) e = ce;
    float4 acc[NJ];
    bool live[NJ];
    int colx[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        live[j] = slab_col<G, WIDE>(t, j) < F;
        colx[j] = imin(slab_col<G, WIDE>(t, j), last_x);
    }
    gather_rows<XT, G, 1, NJ, EV, WIDE>(idx, val, b, e, X, ldx, colscale, t, 0, live, colx, acc);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        *reinterpret_cast<float4*>(&red[gi * W + slab_col<G, WIDE>(t, j)]) = acc[j];
    __syncthreads();
    const int fpad = (F + 3) & ~3;
    for (int c = threadIdx.x; c < fpad; c += 256) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < NG; ++q) s += red[q * W + c];
        part_row[c] = s;
    }
}

// The first n_chunks workgroups each reduce one chunk of a long row to a partial row (they
// are the heavy ones, so they start first); the others take the rows of at most `long_thr`
// edges, one group per row.  One launch instead of two keeps the few chunk workgroups from
// running on an otherwise idle chip.
// S groups share a row (see spmm_share for the choice); their sums are added in a fixed butterfly.
template <typename XT, int G, int S, int NJ, bool EV, bool WIDE>
__device__ __forceinline__ void spmm_rows_kernel_body(unsigned gx, const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx,
                                                        const float* __restrict__ val, int64_t n_rows, int64_t long_thr,
                                                        const XT* __restrict__ X,
                                                        int64_t ldx, const float* __restrict__ colscale,
                                                        SpmmEpilogue ep, int n_chunks,
                                                        const int64_t* __restrict__ chunk_begin,
                                                        const int64_t* __restrict__ chunk_end,
                                                        float* __restrict__ partials, int64_t ld_part) {
    constexpr int ROWS = 256 / (G * S);
    __shared__ __attribute__((aligned(16))) float red[256 * 4 * NJ];
    if ((int)blockIdx.x < n_chunks) {              // uniform per workgroup
        chunk_body<XT, G, NJ, EV, WIDE>(chunk_begin[blockIdx.x], chunk_end[blockIdx.x], idx, val, ep.F, ep.last_x, X, ldx, colscale,
                              partials + (int64_t)blockIdx.x * ld_part, red);
        return;
    }
    const int t = threadIdx.x % G, gi = S == 1 ? 0 : threadIdx.x / G % S;
    const int64_t i = (int64_t)(blockIdx.x - n_chunks) * ROWS + threadIdx.x / (G * S);
    if (i >= (ep.n_rows_dev ? *ep.n_rows_dev : n_rows)) return;          // a row's lanes leave together (G * S divides 64)
    const int64_t b = ptr[i], e = ptr[i + 1];
    if (e - b > long_thr) return;     // its chunks are reduced above, the row is finished by the combine kernel
    float4 acc[NJ];
    bool live[NJ];
    int colx[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        live[j] = slab_col<G, WIDE>(t, j) < ep.F;
        colx[j] = imin(slab_col<G, WIDE>(t, j), ep.last_x);
    }
    gather_rows<XT, G, S, NJ, EV, WIDE>(idx, val, b, e, X, ldx, colscale, t, gi, live, colx, acc);
    if constexpr (S > 1) {
#pragma unroll
        for (int o = G; o < G * S; o <<= 1)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                acc[j].x += __shfl_xor(acc[j].x, o, 64); acc[j].y += __shfl_xor(acc[j].y, o, 64);
                acc[j].z += __shfl_xor(acc[j].z, o, 64); acc[j].w += __shfl_xor(acc[j].w, o, 64);
            }
        if (gi != 0) return;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        if (live[j]) finish_row<XT>(ep, i, e - b, slab_col<G, WIDE>(t, j), acc[j], X, ldx);
}
template <typename XT, int G, int S, int NJ, bool EV, bool WIDE = false>
__global__ __launch_bounds__(256) void spmm_rows_kernel(const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx,
                                                        const float* __restrict__ val, int64_t n_rows, int64_t long_thr,
                                                        const XT* __restrict__ X,
                                                        int64_t ldx, const float* __restrict__ colscale,
                                                        SpmmEpilogue ep, int n_chunks,
                                                        const int64_t* __restrict__ chunk_begin,
                                                        const int64_t* __restrict__ chunk_end,
                                                        float* __restrict__ partials, int64_t ld_part) {
    spmm_rows_kernel_body<XT, G, S, NJ, EV, WIDE>(gridDim.x, ptr, idx, val, n_rows, long_thr, X, ldx, colscale, ep, n_chunks, chunk_begin, chunk_end, partials, ld_part);
}
template <typename XT, int G, int S, int NJ, bool EV, bool WIDE = false>
struct spmm_rows_kernel_op {
    static constexpr int THREADS = 256, WGS = 1;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { spmm_rows_kernel_body<XT, G, S, NJ, EV, WIDE>(gx, a...); }
};

// One group per long row: partial rows added in chunk order, then the epilogue.
template <typename XT, int G, int NJ>
__device__ __forceinline__ void spmm_combine_kernel_body(unsigned gx, const int32_t* __restrict__ long_row,
                                                           const int32_t* __restrict__ long_first, int n_long,
                                                           const int64_t* __restrict__ ptr,
                                                           const float* __restrict__ partials, int64_t ld_part,
                                                           const XT* __restrict__ X, int64_t ldx, SpmmEpilogue ep) {
    constexpr int ROWS = 256 / G;
    const int t = threadIdx.x % G;
    const int j0 = blockIdx.x * ROWS + threadIdx.x / G;
    if (j0 >= n_long) return;
    const int64_t i = long_row[j0];
    if (i < 0) return;                // an unused slot of a schedule built to its capacity
    const int c0 = long_first[j0], c1 = long_first[j0 + 1];
    const int64_t deg = ptr[i + 1] - ptr[i];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = 4 * (t + G * j);
        if (col >= ep.F) continue;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        in_order(c0, c1, [&](int c) { return *reinterpret_cast<const float4*>(partials + (int64_t)c * ld_part + col); },
                 [&](const float4& v, bool on) { add4(acc, on ? v : make_float4(0.f, 0.f, 0.f, 0.f)); });
        finish_row<XT>(ep, i, deg, col, acc, X, ldx);
    }
}
template <typename XT, int G, int NJ>
__global__ __launch_bounds__(256) void spmm_combine_kernel(const int32_t* __restrict__ long_row,
                                                           const int32_t* __restrict__ long_first, int n_long,
                                                           const int64_t* __restrict__ ptr,
                                                           const float* __restrict__ partials, int64_t ld_part,
                                                           const XT* __restrict__ X, int64_t ldx, SpmmEpilogue ep) {
    spmm_combine_kernel_body<XT, G, NJ>(gridDim.x, long_row, long_first, n_long, ptr, partials, ld_part, X, ldx, ep);
}
template <typename XT, int G, int NJ>
struct spmm_combine_kernel_op {
    static constexpr int THREADS = 256, WGS = 1;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { spmm_combine_kernel_body<XT, G, NJ>(gx, a...); }
};

// ---- the source-sliced schedule of the long rows (slices.hip): one wavefront per task.
// A task is at most SLICE_TASK_MAX consecutive edges of one long row whose sources lie in one slice of the
// node ids.  The wavefront reads the task's indices with coalesced loads (SLICE_PIECE / 64 per lane), its 64 / G groups
// take consecutive runs of them (handed round with shuffles, up to four gathers in flight per group), the
// groups' sums are added across the wavefront in a fixed butterfly, and the first group writes the partial row.
// VW consecutive elements of a row as floats: the unit a lane owns (16 bytes of fp32, 8 or 16 bytes of bf16).
template <typename XT, int VW> struct LaneVec;
template <> struct LaneVec<float, 4> {
    static __device__ __forceinline__ void ld(const float* p, float (&f)[4]) {
        const float4 v = Vec4Load<float>::ld(p);
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
};
template <> struct LaneVec<__hip_bfloat16, 4> {
    static __device__ __forceinline__ void ld(const __hip_bfloat16* p, float (&f)[4]) {
        const u32x2_any r = *reinterpret_cast<const u32x2_any*>(p);
        f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xFFFF0000u);
        f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xFFFF0000u);
    }
};
template <> struct LaneVec<__hip_bfloat16, 8> {
    static __device__ __forceinline__ void ld(const __hip_bfloat16* p, float (&f)[8]) {
        const uint4 r = *reinterpret_cast<const uint4*>(p);
        f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xFFFF0000u);
        f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xFFFF0000u);
        f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xFFFF0000u);
        f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xFFFF0000u);
    }
};

// G lanes own a row, VW elements each (VW = 8 for bf16 rows that allow 16-byte loads: half the lanes per row,
// so twice the rows in flight per wavefront for the same registers), NJ slabs of G * VW columns.
// SHIFT32 (plain sums only: no edge values, no per-source scale): the rows of X start at multiples of 2^row_shift
// bytes and X is smaller than 4 GiB, so a row's address is a 32-bit shift and add beside the base (the generic
// 64-bit index x pitch product costs three quarter-rate multiplies per gather: a third of the loop's issue cycles),
// and a gathered row is added with one multiply-add per element (times 1, or 0 past the task's end).
template <typename XT, int G, int NJ, int VW, bool EV, bool CS, bool SHIFT32 = false>
__global__ __launch_bounds__(256) void spmm_tasks_kernel(const SliceTask* __restrict__ tasks, int64_t n_tasks, int64_t per_wave,
                                                         const int32_t* __restrict__ idx, const float* __restrict__ val, int F, int last_x,
                                                         const XT* __restrict__ X, int64_t ldx,
                                                         const float* __restrict__ colscale, float* __restrict__ partials,
                                                         int64_t ld_part, int row_shift) {
    static_assert(!SHIFT32 || (!EV && !CS), "the 32-bit addressing variant is built for plain sums");
    constexpr int IPL = SLICE_PIECE / 64;                 // indices of a task per lane
    static_assert(IPL * 64 == SLICE_PIECE && (IPL & (IPL - 1)) == 0, "a task's indices fill whole registers");
    constexpr int NG = 64 / G;
    constexpr int U = (G * VW >= 64 && NJ == 1) ? 8 : 4;   // gathers in flight per group (measured: 8 loses for narrower rows)
    const int lane = threadIdx.x & 63;
    const int t = lane % G, gi = lane / G;
    // wavefront w takes the tasks [w * per_wave, (w + 1) * per_wave): consecutive wavefronts walk the processing
    // order front to back (a launch holds at most 2^32 work-items, so one task per wavefront does not scale).
    // The loop is software-pipelined: while the gathers of task p are in flight, the indices of task p + 1 and the
    // record of task p + 2 are requested, so a task costs one memory round trip instead of three.
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t p0 = w * per_wave;
    const int64_t p_end = p0 + per_wave < n_tasks ? p0 + per_wave : n_tasks;
    if (p0 >= p_end) return;                               // uniform over the wavefront
    // Every load below is unconditional (an index past a task's end is clamped to its last edge and the gathered
    // row then dropped by a select): a conditional load becomes a branch with a wait behind it, and the gathers
    // of a task would no longer overlap.
    // A task is walked in passes of up to SLICE_PIECE edges; (begin, len) name a pass.
    auto load_indices = [&](int64_t begin, int len, int32_t (&ix)[IPL], float (&wx)[IPL]) {
        const int last = len > 0 ? len - 1 : 0;
#pragma unroll
        for (int q = 0; q < IPL; ++q) {
            const int64_t e = begin + (64 * q + lane < last ? 64 * q + lane : last);
            ix[q] = idx[e];
            if (EV) wx[q] = val[e];
        }
    };
    auto pass_len = [](const SliceTask& tk, int off) { return (int)tk.len - off < SLICE_PIECE ? (int)tk.len - off : SLICE_PIECE; };
    SliceTask cur = tasks[p0];
    SliceTask nxt = tasks[p0 + 1 < p_end ? p0 + 1 : p0];
    int32_t ix[IPL];
    float wx[IPL];
#pragma unroll
    for (int q = 0; q < IPL; ++q) wx[q] = 1.f;
    load_indices(cur.begin, pass_len(cur, 0), ix, wx);
    int col[NJ];                                           // first column the lane reads in slab j (a dead unit reads column 0)
    bool live[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        live[j] = VW * (t + G * j) < F;
        col[j] = live[j] ? (VW == 4 ? imin(VW * (t + G * j), last_x) : VW * t) : 0;
    }
    float acc[NJ][VW];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < VW; ++q) acc[j][q] = 0.f;
    int off = 0;                                           // edges of the current task already added
    for (int64_t p = p0; p < p_end;) {
        const int len = pass_len(cur, off);                // >= 1: this pass
        const bool last_pass = off + len == (int)cur.len;
        const int per = (len + NG - 1) / NG;               // the same in every lane
        const int first = gi * per;
        SliceTask nn = nxt;
        int32_t nix[IPL];
        float nwx[IPL];
#pragma unroll
        for (int q = 0; q < IPL; ++q) { nix[q] = 0; nwx[q] = 1.f; }
        for (int k0 = 0; k0 < per; k0 += U) {
            int64_t c[U];
            float sc[U];
            bool on[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int pos = first + k0 + u;
                on[u] = k0 + u < per && pos < len;
                const int src = pos & 63;
                int32_t ci = __shfl(ix[0], src, 64);
#pragma unroll
                for (int q = 1; q < IPL; ++q) {
                    const int32_t o = __shfl(ix[q], src, 64);
                    ci = (pos >> 6) == q ? o : ci;
                }
                c[u] = ci;                                 // a valid index of this task even where `on` is false
                sc[u] = 1.f;
                if (EV) {
                    float wi = __shfl(wx[0], src, 64);
#pragma unroll
                    for (int q = 1; q < IPL; ++q) {
                        const float o = __shfl(wx[q], src, 64);
                        wi = (pos >> 6) == q ? o : wi;
                    }
                    sc[u] = wi;
                }
                if (CS) sc[u] *= colscale[c[u]];
            }
            float v[NJ][U][VW];
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if constexpr (SHIFT32) {
                        const uint32_t off = ((uint32_t)c[u] << row_shift) + (uint32_t)(col[j] * (int)sizeof(XT));
                        const XT* const src = reinterpret_cast<const XT*>(reinterpret_cast<const char*>(X) + off);
                        LaneVec<XT, VW>::ld(src, v[j][u]);
                    } else {
                        LaneVec<XT, VW>::ld(X + c[u] * ldx + col[j], v[j][u]);
                    }
                }
            if (k0 == 0) {                                 // behind the first gathers: what the next pass and the task after next need
                __builtin_amdgcn_sched_barrier(0);
                if (last_pass) {
                    load_indices(nxt.begin, pass_len(nxt, 0), nix, nwx);
                    nn = tasks[p + 2 < p_end ? p + 2 : p];
                } else {
                    load_indices(cur.begin + off + len, pass_len(cur, off + len), nix, nwx);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int q = 0; q < VW; ++q) {
                        float x = v[j][u][q];
                        if constexpr (SHIFT32) {
                            acc[j][q] = fmaf(x, on[u] ? 1.f : 0.f, acc[j][q]);     // x * 1 + acc rounds once, as x + acc does
                        } else {
                            if (EV || CS) x *= sc[u];
                            acc[j][q] += on[u] ? x : 0.f;
                        }
                    }
        }
        if (last_pass) {                                   // uniform: the task's partial row
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int o = G; o < 64; o <<= 1)
#pragma unroll
                    for (int q = 0; q < VW; ++q) acc[j][q] += __shfl_xor(acc[j][q], o, 64);
                if (gi == 0 && live[j]) {
                    float* out = partials + (int64_t)cur.id * ld_part + VW * (t + G * j);
#pragma unroll
                    for (int q = 0; q < VW; q += 4)
                        *reinterpret_cast<float4*>(out + q) = make_float4(acc[j][q], acc[j][q + 1], acc[j][q + 2], acc[j][q + 3]);
                }
#pragma unroll
                for (int q = 0; q < VW; ++q) acc[j][q] = 0.f;
            }
            cur = nxt; nxt = nn;
            off = 0;
            ++p;
        } else {
            off += len;
        }
#pragma unroll
        for (int q = 0; q < IPL; ++q) { ix[q] = nix[q]; if (EV) wx[q] = nwx[q]; }
    }
}

// One wavefront per long row: group g adds the row's partial rows g, g + 64/G, ... in ascending order, the groups'
// sums are added in a fixed butterfly, then the epilogue.
template <typename XT, int G, int NJ>
__global__ __launch_bounds__(256) void spmm_combine_tasks_kernel(const int32_t* __restrict__ long_row,
                                                                 const int64_t* __restrict__ row_task, int n_long,
                                                                 const int64_t* __restrict__ ptr,
                                                                 const float* __restrict__ partials, int64_t ld_part,
                                                                 const XT* __restrict__ X, int64_t ldx, SpmmEpilogue ep) {
    constexpr int NG = 64 / G;
    const int lane = threadIdx.x & 63;
    const int j0 = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j0 >= n_long) return;
    const int64_t i = long_row[j0];
    if (i < 0) return;
    const int t = lane % G, gi = lane / G;
    const int64_t t0 = row_task[j0], t1 = row_task[j0 + 1];
    const int64_t deg = ptr[i + 1] - ptr[i];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = 4 * (t + G * j);
        const bool live = col < ep.F;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live) {
            int64_t c = t0 + gi;
            for (; c + 3 * NG < t1; c += 4 * NG) {          // four loads in flight, added in ascending order
                const float4 a0 = *reinterpret_cast<const float4*>(partials + c * ld_part + col);
                const float4 a1 = *reinterpret_cast<const float4*>(partials + (c + NG) * ld_part + col);
                const float4 a2 = *reinterpret_cast<const float4*>(partials + (c + 2 * NG) * ld_part + col);
                const float4 a3 = *reinterpret_cast<const float4*>(partials + (c + 3 * NG) * ld_part + col);
                add4(acc, a0); add4(acc, a1); add4(acc, a2); add4(acc, a3);
            }
            for (; c < t1; c += NG) add4(acc, *reinterpret_cast<const float4*>(partials + c * ld_part + col));
        }
#pragma unroll
        for (int o = G; o < 64; o <<= 1) {
            acc.x += __shfl_xor(acc.x, o, 64);
            acc.y += __shfl_xor(acc.y, o, 64);
            acc.z += __shfl_xor(acc.z, o, 64);
            acc.w += __shfl_xor(acc.w, o, 64);
        }
        if (gi == 0 && live) finish_row<XT>(ep, i, deg, col, acc, X, ldx);
    }
}

// ---- plain sums in slabs of columns: G lanes own an edge's part of a row, 16 bytes each (a slab: 64 columns of fp32 or 128 of bf16 with G =
// 16), and a launch walks the whole structure slab by slab, so that an L2 holds four times as many (quarter) rows of X at F = 256.
// The lanes of a group fetch the indices of SLAB_BATCH edges of its run and turn them into byte offsets; a lane's offset is handed to its
// group by DPP, which folds into the addition of the column (G = 8 needs two): no LDS, no 64-bit products.  X is read through a buffer
// descriptor: a place past the end of a run has an offset beyond it and reads as zeros, without a request to memory and without a select.
// What bounds them: the lines that miss the L2 (2^20 rows of 256 columns, 25 edges a row: 88 million, a quarter at 6 TB/s in each pass) and,
// below that, requests in flight.  Sum over the rows of a direction, us, before (spmm_rows_kernel, spmm_tasks_kernel) -> now:
//   2^20 rows, 25 edges, fp32: F = 16 292 -> 210, 32 446 -> 271, 64 679 -> 514, 128 1146 -> 996, 256 2314 -> 1927 (tasks 1240 -> 936, rows
//   1030 -> 950), 512 5099 -> 3747;  2^20 rows, 4 edges: F = 16 131 -> 74, 64 246 -> 183, 256 767 -> 714;  3e5 rows, 20 edges: F = 16 89 ->
//   73, 64 196 -> 165, 256 682 -> 553
//   bf16: 2^20 rows, 25 edges: F = 32 405 -> 271, 64 600 -> 368, 128 882 -> 679, 256 1467 -> 1289;  3e5 rows, 20 edges: F = 64 165 -> 100
// (Slabs of 32 columns for wide rows: 79 million lines, but 2350 us: a quarter of the bytes in flight for each index fetched.)
// Narrow rows are added up by batches (BY_BATCH).  R-MAT graphs, both directions, us, a chain per row / by batches: 1.5e5 rows, 3 edges: F = 16
// 49.5/44.3, F = 32 53.7/52.1, bf16 F = 64 76.8/71.1;  5e5 rows, 8 edges: 117/112, 133/133, 188/183 (all loads of a step are asked for before the
// first is waited for: with the additions among them F = 32 took 66 us).
constexpr int SLAB_BATCH = 16;
// (offsets are from a slab's first column: 2^22 rows of 1 KB, 4 GiB, leave room above the last row's)
constexpr uint32_t SLAB_NOWHERE = 0xFFFFFE00u;             // (a lane's bytes within the slab, at most 240, are added to it)
constexpr uint32_t SLAB_X_BYTES = 0xFFFFFE00u;             // a slab of X ends here at most

template <int G, int N> __device__ __forceinline__ uint32_t group_lane(uint32_t v) {      // lane N of the G lanes around this one
    static_assert(G == 4 || G == 8 || G == 16, "a quad, half a DPP row, a DPP row");
    if constexpr (G == 4) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, N * 0x55, 0xF, 0xF, false);        // quad_perm
    int r = __builtin_amdgcn_update_dpp(0, (int)v, 0x150 + N, 0xF, 0xF, false);            // row_newbcast
    if constexpr (G == 8) r = __builtin_amdgcn_update_dpp(r, (int)v, 0x158 + N, 0xF, 0xC, false);      // (banks 2 and 3: the upper half)
    return (uint32_t)r;
}
template <typename XT, int G> struct Slab {
    static constexpr int VW = 16 / (int)sizeof(XT);        // columns of a lane
    static constexpr int COLS = G * VW;                    // of a slab
    static constexpr int NG = 64 / G;                      // groups of a wavefront
    static constexpr int Q = SLAB_BATCH / G;               // offsets of a batch that a lane holds: edge q * G + t of the batch in place q
    __amdgpu_buffer_rsrc_t x;
    uint32_t pitch, colx;
    int t, col;                                            // lane of the group, its first column
    __device__ __forceinline__ Slab(const XT* X, uint32_t x_bytes, int64_t ldx, uint32_t slab, int F) {
        x = __builtin_amdgcn_make_buffer_rsrc(const_cast<XT*>(X) + (int64_t)slab * COLS, 0, (int)x_bytes, 0x00020000);
        pitch = (uint32_t)ldx * (uint32_t)sizeof(XT);
        t = (int)threadIdx.x % G;
        col = (int)slab * COLS + VW * t;
        colx = col < F ? 16u * (uint32_t)t : 0u;           // (a lane without columns reads what its first one does)
    }
    // Narrow rows are added up by batches: four rows first, those sums in turn, a batch's sum to acc.  So a row of 100 edges has the rounding
    // errors of four chains of 25 (the sums of narrow rows in the general kernel; one chain has 1.8 to 3 times as much).
    static constexpr bool BY_BATCH = G < 16;
    // acc (+)= the rows of the edges N0, N0 + 1, ... of a batch (by batches: = with the first of them).
    template <int N0, int... U> __device__ __forceinline__ void step(const uint32_t (&off)[Q], float (&acc)[VW], std::integer_sequence<int, U...>) const {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        constexpr int N = (int)sizeof...(U);
        static_assert(N % 4 == 0, "four at a time");
        u32x4 v[N];
        ((v[U] = __builtin_amdgcn_raw_buffer_load_b128(x, (int)(group_lane<G, (N0 + U) % G>(off[(N0 + U) / G]) + colx), 0, 0)), ...);
        __builtin_amdgcn_sched_barrier(0);                 // all of them in flight before the first is waited for
        auto column = [&](int u, int c) {                  // of edge u: column c of the lane's
            if constexpr (sizeof(XT) == 4) return __uint_as_float(v[u][c]);
            else return __uint_as_float(c % 2 ? v[u][c / 2] & 0xFFFF0000u : v[u][c / 2] << 16);
        };
        if constexpr (BY_BATCH) {
#pragma unroll
            for (int u = 0; u < N; u += 4)
#pragma unroll
                for (int c = 0; c < VW; ++c) {
                    const float four = (column(u, c) + column(u + 1, c)) + (column(u + 2, c) + column(u + 3, c));
                    acc[c] = N0 + u ? acc[c] + four : four;
                }
        } else {
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int c = 0; c < VW; ++c) acc[c] += column(u, c);
        }
    }
    template <int N0> __device__ __forceinline__ void steps(const uint32_t (&off)[Q], int cnt, float (&acc)[VW]) const {
        if (cnt > N0 + 4) step<N0>(off, acc, std::make_integer_sequence<int, 8>());
        else step<N0>(off, acc, std::make_integer_sequence<int, 4>());
    }
    // The first cnt edges of a batch (cnt: the same in every group; a group with fewer has offsets nowhere).
    __device__ __forceinline__ void gather(const uint32_t (&off)[Q], int cnt, float (&acc)[VW]) const {
        if constexpr (BY_BATCH) {
            float sum[VW];
            steps<0>(off, cnt, sum);
            if (cnt > 8) steps<8>(off, cnt, sum);
#pragma unroll
            for (int c = 0; c < VW; ++c) acc[c] += sum[c];
        } else {
            steps<0>(off, cnt, acc);
            if (cnt > 8) steps<8>(off, cnt, acc);
        }
    }
    // Indices of the edges k .. k + SLAB_BATCH - 1 of a run that ends at `end` (edge `some` exists and is read where there are none), and
    // the offsets of their rows.
    __device__ __forceinline__ void fetch(const int32_t* __restrict__ idx, int64_t some, uint32_t k, uint32_t end, int32_t (&ix)[Q]) const {
#pragma unroll
        for (int q = 0; q < Q; ++q) ix[q] = idx[some + (k + q * G + t < end ? (int64_t)(k + q * G + t) : 0)];
    }
    __device__ __forceinline__ void place(const int32_t (&ix)[Q], uint32_t k, uint32_t end, uint32_t (&off)[Q]) const {
#pragma unroll
        for (int q = 0; q < Q; ++q) off[q] = k + q * G + t < end ? (uint32_t)ix[q] * pitch : SLAB_NOWHERE;
    }
    __device__ __forceinline__ void store(float* row, const float (&acc)[VW]) const {      // a partial row
#pragma unroll
        for (int q = 0; q < VW; q += 4) *reinterpret_cast<float4*>(row + col + q) = make_float4(acc[q], acc[q + 1], acc[q + 2], acc[q + 3]);
    }
};

// The chunks of long rows (n_chunks workgroups of every slab: the groups take a run of the chunk each, their sums are added through
// LDS in ascending order) and the rows of at most long_thr edges.  A workgroup takes SLAB_ROWS consecutive rows, puts them in order of
// their lengths (longest first) and deals them to its wavefronts, a row a group, so that the groups of a wavefront end together.
// While a batch of a row is gathered, the indices of its next batch, or of the next row, are on their way.
constexpr int SLAB_ROWS = 256;
constexpr int64_t SLAB_MANY = (int64_t)1 << 17;
template <typename XT, int G>
__device__ __forceinline__ void spmm_slab_rows_kernel_body(unsigned gx, const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx, int64_t n_rows,
                                                           int64_t long_thr, const XT* __restrict__ X, int64_t ldx, uint32_t x_bytes,
                                                           const SpmmEpilogue& ep, uint32_t slab_blocks, int n_chunks,
                                                           const int64_t* __restrict__ chunk_begin, const int64_t* __restrict__ chunk_end,
                                                           float* __restrict__ partials, int64_t ld_part) {
    using S = Slab<XT, G>;
    constexpr int NG = S::NG, VW = S::VW, Q = S::Q;
    constexpr int BINS = SPMM_LONG_ROW + 2;                // lengths 0 .. SPMM_LONG_ROW, and above
    __shared__ union {
        float4 red[256 * VW / 4];
        struct {
            int64_t begin[SLAB_ROWS];
            uint32_t len[SLAB_ROWS], bin[BINS], wave_sum[4];
            uint8_t row[SLAB_ROWS];
        } o;
    } sh;
    const int tid = threadIdx.x;
    const uint32_t slab = blockIdx.x / slab_blocks, block = blockIdx.x - slab * slab_blocks;
    const S s(X, x_bytes, ldx, slab, ep.F);
    float acc[VW];
#pragma unroll
    for (int q = 0; q < VW; ++q) acc[q] = 0.f;
    uint32_t off[Q];
    int32_t ix[Q];
    if ((int)block < n_chunks) {
        const int64_t cb = chunk_begin[block];
        const uint32_t len = (uint32_t)(chunk_end[block] - cb), per = (len + 256 / G - 1) / (256 / G);
        const uint32_t run = (uint32_t)(tid / G) * per, end = run + per < len ? run + per : len;
        for (uint32_t k = 0; k < per; k += SLAB_BATCH) {
            s.fetch(idx, cb, run + k, end, ix);
            s.place(ix, run + k, end, off);
            s.gather(off, (int)(per - k), acc);
        }
#pragma unroll
        for (int q = 0; q < VW; q += 4) sh.red[tid * (VW / 4) + q / 4] = make_float4(acc[q], acc[q + 1], acc[q + 2], acc[q + 3]);
        __syncthreads();
        if (tid < G * (VW / 4) && (int)slab * S::COLS + 4 * tid < ep.F) {
            float4 sum = sh.red[tid];
            for (int g = 1; g < 256 / G; ++g) add4(sum, sh.red[g * (G * VW / 4) + tid]);
            *reinterpret_cast<float4*>(partials + (int64_t)block * ld_part + (int)slab * S::COLS + 4 * tid) = sum;
        }
        return;
    }
    const int64_t row0 = (int64_t)((int)block - n_chunks) * SLAB_ROWS;
    if (tid < BINS) sh.o.bin[tid] = 0;
    __syncthreads();
    int64_t b = 0, len = 0;
    bool mine = row0 + tid < n_rows;
    if (mine) {
        b = ptr[row0 + tid];
        len = ptr[row0 + tid + 1] - b;
        mine = len <= long_thr;
    }
    const int at_bin = BINS - 1 - (int)(len < BINS - 1 ? len : BINS - 1);
    const uint32_t rank = mine ? atomicAdd(&sh.o.bin[at_bin], 1u) : 0u;
    __syncthreads();
    uint32_t rows;
    const uint32_t first = block_scan<4>(tid < BINS ? sh.o.bin[tid] : 0u, sh.o.wave_sum, rows);
    if (tid < BINS) sh.o.bin[tid] = first;
    __syncthreads();
    if (mine) {
        const uint32_t at = sh.o.bin[at_bin] + rank;
        sh.o.begin[at] = b;
        sh.o.len[at] = (uint32_t)len;
        sh.o.row[at] = (uint8_t)tid;
    }
    __syncthreads();
    struct Rows { int64_t begin; uint32_t len, most; int row; };      // a group's row, and the longest of the wavefront's
    const int gi = (tid & 63) / G;
    auto take = [&](uint32_t q) {
        const uint32_t at = NG * q + gi;
        const bool on = at < rows;
        Rows r{on ? sh.o.begin[at] : 0, on ? sh.o.len[at] : 0u, 0u, on ? (int)sh.o.row[at] : -1};
        r.most = (uint32_t)__builtin_amdgcn_readlane((int)r.len, 0);
#pragma unroll
        for (int g = 1; g < NG; ++g) {                     // (lengths beyond the last bin are in no order)
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)r.len, G * g);
            r.most = o > r.most ? o : r.most;
        }
        return r;
    };
    // (a conditional load: a row without edges may begin past the last index)
    auto fetch = [&](const Rows& r, uint32_t k) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (k + q * G + s.t < r.len) ix[q] = idx[r.begin + k + q * G + s.t];
    };
    uint32_t q4 = (uint32_t)tid >> 6, k = 0;
    if (NG * q4 >= rows) return;
    Rows cur = take(q4);
#pragma unroll
    for (int q = 0; q < Q; ++q) ix[q] = 0;
    fetch(cur, 0);
    for (;;) {
        s.place(ix, k, cur.len, off);
        const bool last = k + SLAB_BATCH >= cur.most;
        Rows nxt = cur;
        uint32_t nk = k + SLAB_BATCH;
        if (last) {
            q4 += 4;
            nk = 0;
            nxt = take(q4);                                // (none: of no length)
        }
        fetch(nxt, nk);
        if (cur.most > k) s.gather(off, (int)(cur.most - k), acc);
        if (last) {
            if (cur.row >= 0) {
#pragma unroll
                for (int q = 0; q < VW; q += 4)
                    if (s.col + q < ep.F)
                        finish_row<XT>(ep, row0 + cur.row, (int64_t)cur.len, s.col + q, make_float4(acc[q], acc[q + 1], acc[q + 2], acc[q + 3]), X, ldx);
            }
#pragma unroll
            for (int q = 0; q < VW; ++q) acc[q] = 0.f;
            if (NG * q4 >= rows) return;
        }
        cur = nxt;
        k = nk;
    }
}
template <typename XT, int G> constexpr int SLAB_WGS = sizeof(XT) == 2 || G < 16 ? 5 : 6;       // (more registers spill)
template <typename XT, int G>
__global__ __launch_bounds__(256, (SLAB_WGS<XT, G>)) void spmm_slab_rows_kernel(const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx, int64_t n_rows,
                                                                int64_t long_thr, const XT* __restrict__ X, int64_t ldx, uint32_t x_bytes,
                                                                SpmmEpilogue ep, uint32_t slab_blocks, int n_chunks,
                                                                const int64_t* __restrict__ chunk_begin, const int64_t* __restrict__ chunk_end,
                                                                float* __restrict__ partials, int64_t ld_part) {
    spmm_slab_rows_kernel_body<XT, G>(gridDim.x, ptr, idx, n_rows, long_thr, X, ldx, x_bytes, ep, slab_blocks, n_chunks, chunk_begin, chunk_end, partials, ld_part);
}
template <typename XT, int G> struct spmm_slab_rows_kernel_op {
    static constexpr int THREADS = 256, WGS = SLAB_WGS<XT, G>;
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { spmm_slab_rows_kernel_body<XT, G>(gx, a...); }
};

// The tasks of the sliced schedule, one a wavefront: its groups take equal runs of the task's edges, two batches at a time, whose indices are
// asked for while the two before them are gathered.  (A wavefront that walks several tasks, consecutive or strided, with the next task's
// indices on their way, is slower the more it has: the wavefronts drift apart and the L2 holds more of X's slices at a time.)
template <typename XT, int G>
__global__ __launch_bounds__(256, 6) void spmm_slab_tasks_kernel(const SliceTask* __restrict__ tasks, int64_t n_tasks,
                                                                 const int32_t* __restrict__ idx, int F, const XT* __restrict__ X, int64_t ldx,
                                                                 uint32_t x_bytes, float* __restrict__ partials, int64_t ld_part,
                                                                 uint32_t slab_blocks) {
    using S = Slab<XT, G>;
    constexpr int NG = S::NG, VW = S::VW, Q = S::Q;
    const uint32_t slab = blockIdx.x / slab_blocks;
    const int64_t p = (int64_t)(blockIdx.x - slab * slab_blocks) * 4 + (threadIdx.x >> 6);
    if (p >= n_tasks) return;                              // uniform over the wavefront
    const S s(X, x_bytes, ldx, slab, F);
    const int gi = (threadIdx.x & 63) / G;
    const SliceTask tk = tasks[p];
    const uint32_t per = (tk.len + NG - 1) / NG;
    const uint32_t run = gi * per, end = run + per < tk.len ? run + per : tk.len;      // the group's edges of the task
    int32_t i0[Q], i1[Q];
    s.fetch(idx, tk.begin, run, end, i0);
    s.fetch(idx, tk.begin, run + SLAB_BATCH, end, i1);
    float acc[VW];
#pragma unroll
    for (int q = 0; q < VW; ++q) acc[q] = 0.f;
    for (uint32_t k = 0;;) {
        uint32_t o0[Q], o1[Q];
        s.place(i0, run + k, end, o0);
        s.place(i1, run + k + SLAB_BATCH, end, o1);
        const bool more = k + 2 * SLAB_BATCH < per;
        if (more) {
            s.fetch(idx, tk.begin, run + k + 2 * SLAB_BATCH, end, i0);
            s.fetch(idx, tk.begin, run + k + 3 * SLAB_BATCH, end, i1);
        }
        s.gather(o0, (int)(per - k), acc);
        if (per > k + SLAB_BATCH) s.gather(o1, (int)(per - k - SLAB_BATCH), acc);
        if (!more) break;
        k += 2 * SLAB_BATCH;
    }
#pragma unroll
    for (int o = G; o < 64; o <<= 1)
#pragma unroll
        for (int q = 0; q < VW; ++q) acc[q] += __shfl_xor(acc[q], o, 64);
    if (gi == 0 && s.col < F) s.store(partials + (int64_t)tk.id * ld_part, acc);
}

// Rows of fewer than four columns without room for one vector: one wavefront per row,
// one lane per column (handles rows of any length itself).
template <typename XT>
__global__ __launch_bounds__(256) void spmm_rows_scalar_kernel(
    const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx, int64_t n_rows, int F,
    const XT* __restrict__ X, int64_t ldx, int scale, int self_term, const float* __restrict__ colscale,
    const float* addend, int64_t ld_add, const float* __restrict__ bias, int relu,
    float* Y, int64_t ldy, const float* __restrict__ val, const float* __restrict__ rowscale,
    const int64_t* __restrict__ n_rows_dev /*when set: the real row count; n_rows sized the launch*/) {
    const int64_t i = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    if (i >= (n_rows_dev ? *n_rows_dev : n_rows)) return;
    const int t = threadIdx.x % 64;
    const int64_t b = ptr[i], e = ptr[i + 1];
    const float a = rowscale ? rowscale[i] : row_scale(scale, e - b, self_term);
    for (int col = t; col < F; col += 64) {
        float acc = 0.f;
        for (int64_t k = b; k < e; ++k)
            acc = fmaf((colscale ? colscale[idx[k]] : 1.f) * (val ? val[k] : 1.f), (float)X[(int64_t)idx[k] * ldx + col], acc);
        if (self_term) acc += (float)X[i * ldx + col];
        acc *= a;
        if (addend) acc += addend[i * ld_add + col];
        if (bias) acc += bias[col];
        if (relu) acc = acc > 0.f ? acc : 0.f;
        Y[i * ldy + col] = acc;
    }
}

// Whether a launch of n_chunks workgroups and of rows with so many lanes each holds fewer than 2^32 work-items, which is the limit.
static bool spmm_fits(int64_t n_rows, int64_t n_chunks, int lanes) { return (n_chunks + cdiv(n_rows, 256 / lanes)) * 256 < ((int64_t)1 << 32); }

// Groups that may share a row of G lanes' width: four, as far as a wavefront holds them.
constexpr int SPMM_GROUPS(int G) { return G >= 64 ? 1 : G == 32 ? 2 : 4; }
// Whether they do.  A lone group walks the longest unsplit row of a small graph while the chip waits, and a wavefront of many narrow
// groups waits for the longest of its rows; shared rows cost a butterfly each, and idle lanes where rows are short.  Against
// one group per row (us):
//   2500 rows, 3 edges a row (skewed): F = 8 18.2 -> 11.1, F = 47 17.2 -> 10.9;  2e4 rows, 15: F = 8 21.9 -> 11.1, F = 47 22.8 -> 16.0
//   1e6 rows, 25: F = 3 250 -> 227, F = 8 236 -> 209, F = 16 306 -> 266, F = 32 399 -> 376, but F = 47 601 -> 636
//   3e5 rows, 3.25: F = 8 35 -> 28, F = 16 44 -> 40, but F = 32 52 -> 60, F = 47 63 -> 94, F = 100 91 -> 108
//   1e5 rows, 14: F = 100 78 -> 75, F = 47 58 -> 56 (uniform degrees: 45 -> 49), bf16 F = 128 73 -> 75
// (before: at F = 8 these were 30, 36, 354 and 56 us.)
// n_chunks: workgroups that the launch holds besides those of its rows.
bool spmm_share(int64_t n_rows, int64_t nnz, int64_t n_chunks, int G, int S) {
    if (!spmm_fits(n_rows, n_chunks, G * S)) return false;
    const int64_t waves = n_rows * G / 64;                 // with one group per row
    if (G <= 2 || waves <= 2048 || (G <= 4 && nnz >= 2 * n_rows)) return true;
    return nnz >= 8 * n_rows && (G <= 8 || waves <= (G == 32 ? 65536 : 8192));
}

template <typename XT, int G, int NJ>
static void launch_one(const SpmmArgs& a, const SpmmEpilogue& ep, hipStream_t st) {
    constexpr int ROWS = 256 / G;
    const LongRows* lr = a.long_rows;
    const bool split = lr && lr->n_long > 0;
    const bool sliced = split && lr->n_tasks > 0;
    const int64_t thr = split ? (int64_t)SPMM_LONG_ROW : INT64_MAX;
    const int n_chunks = split && !sliced ? lr->n_chunks : 0;
    const int64_t ld_part = round_up(a.F, 4);
    bool tasks_done = false, rows_done = false;
    constexpr int VW = 16 / (int)sizeof(XT), LANES = G * NJ * 4 / VW;      // lanes of a whole row, 16 bytes each
    if constexpr (LANES >= 4) {
        constexpr int SG = LANES < 16 ? LANES : 16;
        const int64_t slabs = cdiv(a.F, SG * VW);
        const int64_t x_rows = a.n_src > 0 ? a.n_src : a.n_rows;
        const int64_t x_bytes = ((x_rows - 1) * a.ldx + std::min<int64_t>(round_up(a.F, VW), SG * VW)) * (int64_t)sizeof(XT);      // of a slab
        const bool units = VW == 4 || (a.F % VW == 0 && a.ldx % VW == 0 && (uintptr_t)a.X % 16 == 0);
        // several slabs: of whole lines, and at most a quarter of them without columns (20 edges a row, 3e5 rows, fp32, us of rows / slabs:
        // F = 96 260/225, 160 412/364, 224 612/494, but 72 260/274 and lines cut by slabs: 112 308/312, 120 352/378, 172 530/573)
        const bool whole = slabs == 1 || ((a.ldx * (int64_t)sizeof(XT)) % 128 == 0 && (uintptr_t)a.X % 128 == 0 && slabs * SG * VW * 3 <= (int64_t)a.F * 4);
        // (rows of few edges with more than Y to read or write beside them are done a whole row at a time: 3.25 edges, F = 256, mask and
        // addend: 255 us, in slabs 278; without them 190 and 187)
        const bool sums = slabs == 1 || a.nnz >= 8 * a.n_rows || (!a.mask && !a.addend && !a.residual && !a.Y2);
        if (!a.val && !a.colscale && !ep.tight && !a.n_rows_dev && units && whole && sums && x_bytes <= (int64_t)SLAB_X_BYTES) {
            const int64_t task_blocks = sliced ? cdiv(lr->n_tasks, 4) : 0, row_blocks = n_chunks + cdiv(a.n_rows, SLAB_ROWS);
            if (sliced && slabs * task_blocks < ((int64_t)1 << 24)) {          // (fewer than 2^32 work-items)
                GRP_LARGE_LAUNCH((spmm_slab_tasks_kernel<XT, SG>), dim3((unsigned)(slabs * task_blocks)), dim3(256), 0, st, (const SliceTask*)lr->tasks,
                                 lr->n_tasks, a.idx, a.F, (const XT*)a.X, a.ldx, (uint32_t)x_bytes, a.partials, ld_part, (uint32_t)task_blocks);
                tasks_done = true;
            }
            // SLAB_MANY rows: below, the workgroups of SLAB_ROWS rows leave the GPU idle (1.5e4 .. 1e5 rows, 15 edges a row: 33 against 18 us at
            // F = 64 and 2e4 rows, 64 and 50 at 4e4, 65 and 64 at 1e5, 81 and 83 at 1.5e5)
            // Dealing rows by length pays where their lengths differ (long rows, as far as the host knows them, hold a sixteenth of the edges)
            // or where they are long; short rows of like lengths are done faster a whole row at a time, but for those of four lanes.  Rows / slabs,
            // both directions, 3e5 rows, us.  Skewed (R-MAT), 5 edges a row: F = 32 130/78, 128 233/208, 256 445/434; uniform: F = 32 74/79, 64
            // 128/141, 256 484/551, 12 edges: 145/150, 273/286, 1095/1120, 40 edges (2.6e5 rows, one direction): 175/159, 366/366; F = 16: 3 edges
            // 60/47, 5 edges 66/66, 8 edges 83/91; bf16, F = 128: 174/188, 12 edges 298/325, 40 edges 384/384.
            const bool uneven = split && 16 * ((int64_t)lr->n_long * SPMM_LONG_ROW + (int64_t)(lr->n_chunks - lr->n_long) * SPMM_CHUNK) >= a.nnz;
            const bool deal = uneven || a.nnz >= 32 * a.n_rows || (SG == 4 && a.nnz <= 5 * a.n_rows);
            if (deal && a.n_rows >= SLAB_MANY && slabs * row_blocks < ((int64_t)1 << 24)) {
                launch(spmm_slab_rows_kernel<XT, SG>, spmm_slab_rows_kernel_op<XT, SG>(), dim3((unsigned)(slabs * row_blocks)), st, a.ptr, a.idx,
                       a.n_rows, thr, (const XT*)a.X, a.ldx, (uint32_t)x_bytes, ep, (uint32_t)row_blocks, n_chunks,
                       n_chunks ? lr->chunk_begin : nullptr, n_chunks ? lr->chunk_end : nullptr, a.partials, ld_part);
                rows_done = true;
            }
        }
    }
    if (sliced && !tasks_done) {                           // the long rows' tasks, slice by slice
        // at most 2^19 workgroups of four wavefronts: a wavefront that walks a dozen consecutive tasks keeps its
        // pipeline of index and record prefetches full (2^21 / 2^19 / 2^17 workgroups on the 2^32-edge share: bf16
        // launch 44.3 / 42.9 / 42.4 ms, fp32 F = 16 launch 34.7 / 34.7 / 35.6 ms)
        const int64_t per_wave = cdiv(lr->n_tasks, (int64_t)4 << 19);
        const dim3 tgrid((unsigned)cdiv(lr->n_tasks, 4 * per_wave));
        // Plain sums over rows that start at multiples of a power of two inside less than 4 GiB: 32-bit addressing; not for the one or two
        // lanes of a bf16 row of 8 or 16 columns (2^20 rows, 1e8 edges, forward and transposed, us with / without: 1711 / 1346 at 8,
        // 1578 / 1577 at 16; no difference for fp32 of 72 columns).
        int row_shift = -1;
        {
            const int64_t pitch_bytes = a.ldx * (int64_t)sizeof(XT);
            const int64_t x_rows = a.n_src > 0 ? a.n_src : a.n_rows;
            if (!a.val && !a.colscale && pitch_bytes > 0 && (pitch_bytes & (pitch_bytes - 1)) == 0 &&
                x_rows * pitch_bytes <= ((int64_t)1 << 32)) {
                row_shift = 0;
                while (((int64_t)1 << row_shift) < pitch_bytes) ++row_shift;
            }
        }
        auto go = [&](auto kernel) {
            GRP_LARGE_LAUNCH(kernel, tgrid, dim3(256), 0, st, (const SliceTask*)lr->tasks, lr->n_tasks, per_wave, a.idx, a.val, a.F, ep.last_x,
                               (const XT*)a.X, a.ldx, a.colscale, a.partials, ld_part, row_shift);
        };
        // bf16 rows of whole 16-byte units: eight elements per lane, half the lanes per row
        constexpr bool bf16 = std::is_same<XT, __hip_bfloat16>::value;
        const bool wide = bf16 && G >= 2 && NJ == 1 && a.F % 8 == 0 && a.ldx % 8 == 0 && ((uintptr_t)a.X % 16) == 0;
        if constexpr (bf16 && G >= 2 && NJ == 1) {
            if (wide) {
                if (a.val && a.colscale) go(spmm_tasks_kernel<XT, G / 2, 1, 8, true, true>);
                else if (a.val) go(spmm_tasks_kernel<XT, G / 2, 1, 8, true, false>);
                else if (a.colscale) go(spmm_tasks_kernel<XT, G / 2, 1, 8, false, true>);
                else if (LANES >= 4 && row_shift >= 0) {
                    if constexpr (LANES >= 4) go(spmm_tasks_kernel<XT, G / 2, 1, 8, false, false, true>);
                } else go(spmm_tasks_kernel<XT, G / 2, 1, 8, false, false>);
            }
        }
        if (!wide) {
            if (a.val && a.colscale) go(spmm_tasks_kernel<XT, G, NJ, 4, true, true>);
            else if (a.val) go(spmm_tasks_kernel<XT, G, NJ, 4, true, false>);
            else if (a.colscale) go(spmm_tasks_kernel<XT, G, NJ, 4, false, true>);
            else if (row_shift >= 0) go(spmm_tasks_kernel<XT, G, NJ, 4, false, false, true>);
            else go(spmm_tasks_kernel<XT, G, NJ, 4, false, false>);
        }
    }
    auto rows = [&](auto kernel, auto op, int lanes) {     // lanes: of a row
        launch(kernel, op, dim3((unsigned)(n_chunks + cdiv(a.n_rows, 256 / lanes))), st, a.ptr, a.idx, a.val, a.n_rows, thr, (const XT*)a.X, a.ldx,
               a.colscale, ep, n_chunks, n_chunks ? lr->chunk_begin : nullptr, n_chunks ? lr->chunk_end : nullptr, a.partials, ld_part);
    };
    auto rows_val = [&](auto kernel, int lanes) {          // with edge values
        launch_alone(kernel, dim3((unsigned)(n_chunks + cdiv(a.n_rows, 256 / lanes))), dim3(256), 0, st, a.ptr, a.idx, a.val, a.n_rows, thr,
                         (const XT*)a.X, a.ldx, a.colscale, ep, n_chunks, n_chunks ? lr->chunk_begin : nullptr, n_chunks ? lr->chunk_end : nullptr,
                         a.partials, ld_part);
    };
    if constexpr (std::is_same<XT, __hip_bfloat16>::value && G >= 2 && NJ == 1) {
        // bf16 rows of whole 16-byte units: eight columns per lane, half the lanes per row (twice the rows per wavefront)
        if (!rows_done && a.F % 8 == 0 && a.ldx % 8 == 0 && ((uintptr_t)a.X % 16) == 0 && !a.self_term) {
            constexpr int GW = G / 2, S = SPMM_GROUPS(GW);
            if (S > 1 && spmm_share(a.n_rows, a.nnz, n_chunks, GW, S)) {
                if (a.val) rows_val(spmm_rows_kernel<XT, GW, S, 2, true, true>, GW * S);
                else rows(spmm_rows_kernel<XT, GW, S, 2, false, true>, spmm_rows_kernel_op<XT, GW, S, 2, false, true>(), GW * S);
            } else if (a.val) rows_val(spmm_rows_kernel<XT, GW, 1, 2, true, true>, GW);
            else rows(spmm_rows_kernel<XT, GW, 1, 2, false, true>, spmm_rows_kernel_op<XT, GW, 1, 2, false, true>(), GW);
            rows_done = true;
        }
    }
    if (!rows_done) {
        constexpr int S = SPMM_GROUPS(G);
        if (S > 1 && spmm_share(a.n_rows, a.nnz, n_chunks, G, S)) {
            if (a.val) rows_val(spmm_rows_kernel<XT, G, S, NJ, true>, G * S);
            else rows(spmm_rows_kernel<XT, G, S, NJ, false>, spmm_rows_kernel_op<XT, G, S, NJ, false>(), G * S);
        } else if (a.val) rows_val(spmm_rows_kernel<XT, G, 1, NJ, true>, G);
        else rows(spmm_rows_kernel<XT, G, 1, NJ, false>, spmm_rows_kernel_op<XT, G, 1, NJ, false>(), G);
    }
    if (sliced) {
        GRP_LARGE_LAUNCH((spmm_combine_tasks_kernel<XT, G, NJ>), dim3((unsigned)cdiv(lr->n_long, 4)), dim3(256), 0, st,
                           lr->long_row, (const int64_t*)lr->row_task, lr->n_long, a.ptr, (const float*)a.partials, ld_part,
                           (const XT*)a.X, a.ldx, ep);
    } else if (split) {
        launch(spmm_combine_kernel<XT, G, NJ>, spmm_combine_kernel_op<XT, G, NJ>(), dim3((unsigned)cdiv(lr->n_long, ROWS)), st,
                           lr->long_row, lr->long_first, lr->n_long, a.ptr, (const float*)a.partials, ld_part,
                           (const XT*)a.X, a.ldx, ep);
    }
}

template <typename XT>
static grp_status dispatch(const SpmmArgs& a, const SpmmEpilogue& ep, hipStream_t st) {
    const int f4 = (a.F + 3) / 4;
    {       // a launch holds fewer than 2^32 work-items: a row per group of f4 lanes (rounded up to a power of two)
        int g = 1;
        while (g < f4 && g < 64) g <<= 1;
        const LongRows* lr = a.long_rows;
        const int64_t chunks = lr && lr->n_long > 0 && lr->n_tasks == 0 ? lr->n_chunks : 0;
        if (!spmm_fits(a.n_rows, chunks, g))
            return fail(GRP_EUNSUPPORTED, "spmm: %lld rows of %d columns exceed one launch", (long long)a.n_rows, a.F);
    }
    if (f4 <= 1) launch_one<XT, 1, 1>(a, ep, st);
    else if (f4 <= 2) launch_one<XT, 2, 1>(a, ep, st);
    else if (f4 <= 4) launch_one<XT, 4, 1>(a, ep, st);
    else if (f4 <= 8) launch_one<XT, 8, 1>(a, ep, st);
    else if (f4 <= 16) launch_one<XT, 16, 1>(a, ep, st);
    else if (f4 <= 32) launch_one<XT, 32, 1>(a, ep, st);
    else if (f4 <= 64) launch_one<XT, 64, 1>(a, ep, st);
    else if (f4 <= 128) launch_one<XT, 64, 2>(a, ep, st);
    else if (f4 <= 256) launch_one<XT, 64, 4>(a, ep, st);
    else return fail(GRP_EUNSUPPORTED, "spmm: F = %d exceeds 1024", a.F);
    return GRP_OK;
}

size_t spmm_partials_bytes(const LongRows* lr, int32_t F) {
    if (!lr || lr->n_long == 0) return 0;
    const int64_t slots = lr->n_tasks > 0 ? lr->n_tasks : (int64_t)lr->n_chunks;      // one partial row per task or chunk
    return (size_t)slots * round_up(F, 4) * sizeof(float);
}

grp_status launch_spmm(const SpmmArgs& a, hipStream_t st) {
    if (a.n_rows == 0) return GRP_OK;
    if (a.n_rows < 0 || a.F <= 0 || !a.ptr || !a.X || !a.Y)
        return fail(GRP_EINVAL, "spmm: bad arguments");
    const int elem = a.x_bf16 ? 2 : 4;
    const int64_t fpad = round_up(a.F, 4);
    // X rows of any pitch and alignment are read as vectors; only a row of fewer than four columns packed without padding is not.
    // (Rows of whole vectors that are also aligned keep the last vector where it is and may read pad columns.)
    const bool roomy = a.ldx >= fpad && a.ldx % 4 == 0 && ((uintptr_t)a.X % (4 * elem)) == 0;
    const bool vec_out = a.ldy >= fpad && a.ldy % 4 == 0 && ((uintptr_t)a.Y % 16) == 0 &&
                         (!a.addend || (a.ld_add % 4 == 0 && a.ld_add >= fpad && ((uintptr_t)a.addend % 16) == 0));
    const bool plain = !a.residual && !a.Y2 && !a.mask && a.addend_rows <= 0 && !a.addend_rows_dev;
    const bool vec_ok = (roomy || a.F >= 4) && (vec_out || plain);
    // compulsory traffic: the index stream, the row pointers, every source row once, every
    // output row once (+ addend rows)
    const int64_t n_src = a.n_src > 0 ? a.n_src : a.n_rows;
    const double bytes = 4.0 * a.nnz + 8.0 * (a.n_rows + 1) + (double)elem * a.F * n_src +
                         4.0 * a.F * a.n_rows * (1.0 + (a.addend ? 1.0 : 0.0) + (a.mask ? 1.0 : 0.0)) +
                         (a.colscale ? 4.0 * n_src : 0.0) + (a.val ? 4.0 * a.nnz : 0.0);
    prof_detail("[rows=%lld,F=%d,nnz=%lld]", (long long)a.n_rows, a.F, (long long)a.nnz);
    ProfScope ps(a.x_bf16 ? "spmm_rows_bf16" : "spmm_rows_f32", st, 2.0 * a.nnz * a.F, bytes);
    if (vec_ok) {
        if (a.long_rows && a.long_rows->n_long > 0 && (!a.partials || ((uintptr_t)a.partials % 16) != 0))
            return fail(GRP_EINVAL, "spmm: partition has long rows but no scratch for their partial sums");
        if (a.residual && (a.ld_res % 4 != 0 || a.ld_res < fpad || (uintptr_t)a.residual % 16 != 0))
            return fail(GRP_EINVAL, "spmm: residual operand must be 16-byte aligned with a pitch multiple of 4");
        if (a.Y2 && (a.ldy2 % 4 != 0 || a.ldy2 < fpad || (uintptr_t)a.Y2 % 16 != 0))
            return fail(GRP_EINVAL, "spmm: second output must be 16-byte aligned with a pitch multiple of 4");
        if (a.mask && (a.ld_mask % 4 != 0 || a.ld_mask < fpad || (uintptr_t)a.mask % 16 != 0))
            return fail(GRP_EINVAL, "spmm: mask must be 16-byte aligned with a pitch multiple of 4");
        SpmmEpilogue ep{a.scale, a.self_term, a.relu, a.F, a.addend, a.ld_add, a.bias, a.Y, a.ldy,
                        a.residual, a.ld_res, a.Y2, a.ldy2, a.addend_rows > 0 ? a.addend_rows : a.n_rows, a.mask, a.ld_mask,
                        a.rowscale, a.n_rows_dev, a.addend_rows_dev, (int)(roomy ? fpad : a.F) - 4, (roomy ? 0 : 1) | (vec_out ? 0 : 2)};
        GRP_TRY(a.x_bf16 ? dispatch<__hip_bfloat16>(a, ep, st) : dispatch<float>(a, ep, st));
    } else {
        if (!plain)
            return fail(GRP_EUNSUPPORTED, "spmm: this epilogue needs 16-byte friendly operands");
        const int64_t blocks = cdiv(a.n_rows, 4);
        if (a.x_bf16)
            launch_alone((spmm_rows_scalar_kernel<__hip_bfloat16>), dim3((unsigned)blocks), dim3(256), 0, st,
                               a.ptr, a.idx, a.n_rows, a.F, (const __hip_bfloat16*)a.X, a.ldx, a.scale,
                               a.self_term, a.colscale, a.addend, a.ld_add, a.bias, a.relu, a.Y, a.ldy, a.val, a.rowscale, a.n_rows_dev);
        else
            launch_alone((spmm_rows_scalar_kernel<float>), dim3((unsigned)blocks), dim3(256), 0, st, a.ptr,
                               a.idx, a.n_rows, a.F, (const float*)a.X, a.ldx, a.scale, a.self_term, a.colscale, a.addend,
                               a.ld_add, a.bias, a.relu, a.Y, a.ldy, a.val, a.rowscale, a.n_rows_dev);
    }
    GRP_LAUNCH_CHECK();
    return GRP_OK;
}

}  // namespace grp

namespace grp {

static grp_status spmm_args_from_call(const grp_partition_t* part, int32_t transposed, int32_t scale, int32_t self_term, int32_t F,
                                      const void* X, int64_t ldx, int32_t x_dtype, float* Y, int64_t ldy, const char* who,
                                      SpmmArgs* out) {
    if (!part || !X || !Y) return fail(GRP_EINVAL, "%s: null argument", who);
    if (F <= 0 || F > 1024 || ldx < F || ldy < F) return fail(GRP_EINVAL, "%s: bad F / pitch", who);
    if (scale < GRP_SCALE_NONE || scale > GRP_SCALE_RSQRT) return fail(GRP_EINVAL, "%s: bad scale", who);
    if (x_dtype != GRP_DTYPE_FP32 && x_dtype != GRP_DTYPE_BF16) return fail(GRP_EINVAL, "%s: bad dtype", who);
    SpmmArgs a;
    a.ptr = transposed ? part->colptr : part->rowptr;
    a.idx = transposed ? part->row : part->col;
    a.long_rows = transposed ? &part->csc_long : &part->csr_long;
    a.n_rows = part->n;
    a.nnz = part->nnz;
    a.F = F;
    a.X = X;
    a.ldx = ldx;
    a.x_bf16 = x_dtype == GRP_DTYPE_BF16;
    a.scale = scale;
    a.self_term = self_term ? 1 : 0;
    a.Y = Y;
    a.ldy = ldy;
    *out = a;
    return GRP_OK;
}

// The partial sums of split rows for callers that cannot allocate: one array per GPU, reserved when the
// library is loaded and kept until the process ends.  The array's name is only a host-side stand-in;
// its device address is looked up once per device and cached.
constexpr size_t SPMM_STATIC_SCRATCH_BYTES = (size_t)32 << 20;
static __device__ __align__(256) unsigned char g_spmm_scratch[SPMM_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static void* g_spmm_scratch_ptr[MAX_DEVICES] = {nullptr};
static std::mutex g_spmm_scratch_mu;

static grp_status spmm_static_scratch(void** out) {
    int dev = 0;
    GRP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(GRP_EUNSUPPORTED, "device index %d is outside [0, %d)", dev, MAX_DEVICES);
    std::lock_guard<std::mutex> lk(g_spmm_scratch_mu);
    if (!g_spmm_scratch_ptr[dev]) {
        void* p = nullptr;
        GRP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(g_spmm_scratch)));      // the copy of the array on the current device
        g_spmm_scratch_ptr[dev] = p;
    }
    *out = g_spmm_scratch_ptr[dev];
    return GRP_OK;
}

}  // namespace grp

extern "C" grp_status grp_spmm_workspace_bytes(const grp_partition_t* part, int32_t transposed, int32_t F, size_t* bytes) {
    if (!part || !bytes) return grp::fail(GRP_EINVAL, "grp_spmm_workspace_bytes: null argument");
    if (F <= 0 || F > 1024) return grp::fail(GRP_EINVAL, "grp_spmm_workspace_bytes: bad F");
    *bytes = grp::spmm_partials_bytes(transposed ? &part->csc_long : &part->csr_long, F);
    return GRP_OK;
}

extern "C" grp_status grp_spmm(const grp_partition_t* part, int32_t transposed, int32_t scale,
                               int32_t self_term, int32_t F, const void* X, int64_t ldx, int32_t x_dtype,
                               float* Y, int64_t ldy, void* workspace, size_t workspace_bytes, void* stream) {
    grp::SpmmArgs a;
    GRP_TRY(grp::spmm_args_from_call(part, transposed, scale, self_term, F, X, ldx, x_dtype, Y, ldy, "grp_spmm", &a));
    const size_t need = grp::spmm_partials_bytes(a.long_rows, F);
    if (need > 0 && (!workspace || workspace_bytes < need))
        return grp::fail(GRP_EWORKSPACE, "grp_spmm: workspace of %zu bytes, %zu needed", workspace_bytes, need);
    if (need > 0 && ((uintptr_t)workspace % 16) != 0) return grp::fail(GRP_EINVAL, "grp_spmm: workspace must be 16-byte aligned");
    a.partials = need ? (float*)workspace : nullptr;
    return grp::launch_spmm(a, (hipStream_t)stream);
}

extern "C" grp_status grp_spmm_static(const grp_partition_t* part, int32_t transposed, int32_t scale,
                                      int32_t self_term, int32_t F, const void* X, int64_t ldx, int32_t x_dtype,
                                      float* Y, int64_t ldy, void* stream) {
    grp::SpmmArgs a;
    GRP_TRY(grp::spmm_args_from_call(part, transposed, scale, self_term, F, X, ldx, x_dtype, Y, ldy, "grp_spmm_static", &a));
    const size_t need = grp::spmm_partials_bytes(a.long_rows, F);
    if (need > grp::SPMM_STATIC_SCRATCH_BYTES)
        return grp::fail(GRP_EWORKSPACE, "grp_spmm_static: the split rows of this partition need %zu bytes of partial sums at F = %d, "
                         "the built-in scratch holds %zu; use grp_spmm with a workspace", need, F, grp::SPMM_STATIC_SCRATCH_BYTES);
    void* scratch = nullptr;
    if (need > 0) GRP_TRY(grp::spmm_static_scratch(&scratch));
    a.partials = (float*)scratch;
    return grp::launch_spmm(a, (hipStream_t)stream);
}
