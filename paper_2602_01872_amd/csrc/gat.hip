// Graph attention layers (one head) for gfx950: attention-weighted neighbour aggregation and its
// reverse pass, around the same MFMA GEMMs as the other models.
//
//   t_u = W^T h_u,  p_u = a_src . t_u,  q_v = a_dst . t_v,
//   e_uv = LeakyReLU_0.2(p_u + q_v) over the in-edges u -> v and the self term u = v,
//   alpha = softmax_u(e_uv),  out_v = sum_u alpha_uv t_u + b,  h'_v = ReLU(out_v) (hidden layers).
//
// Layout.  p and q are two more outputs of the layer's linear map, p = h . (W a_src) and
// q = h . (W a_dst), so the GEMM computes  T_ext = H [W | 0 | W a_src | W a_dst | 0 0]  with the
// two scores at the 16-byte aligned column ld(F); the reverse pass hands the GEMMs
// dT_ext = [dT | 0 | dp | dq | 0 0] in the same layout, and the gradients of W, a_src, a_dst
// follow from dW_ext = H^T dT_ext by the chain rule of the two extra columns.
//
// No per-edge state is kept: alpha_uv is recomputed from four per-node scalars (p_u, q_v, the
// row maximum m_v and the row sum Z_v).  The reverse pass walks the CSR (rows = destinations, for dq
// and what an edge needs of its destination) and then, with that, the CSC (rows = sources, for dT and dp),
// each row summing in its stored edge order: no floating-point atomics, bit-reproducible.
//
// Mapping as in the SpMM: a group of G lanes owns a row, lane t owns columns 4*(t + G*j); rows
// longer than SPMM_LONG_ROW edges are walked in the partition's chunks by whole workgroups.
#include "common.h"

#include <algorithm>

namespace grp {

constexpr float GAT_SLOPE = 0.2f;

__device__ __forceinline__ float leaky(float x) { return x > 0.f ? x : GAT_SLOPE * x; }
__device__ __forceinline__ float leaky_d(float x) { return x > 0.f ? 1.f : GAT_SLOPE; }

template <int G>
__device__ __forceinline__ float group_sum(float x) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, G);
    return x;
}
template <int G>
__device__ __forceinline__ float group_max(float x) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, G));
    return x;
}
// A group's number in the workgroup, and what its lane k holds.  A group of a whole wavefront has both in scalar registers: a row's
// bounds, its scalars and the addresses of the rows it gathers take no vector registers then, of which the walks have few
// to spare (3e5 rows of 256 columns, 3.25 edges a row, us of FWD / DST / SRC: 291/229/315, registers 54/62/68 -> 276/225/282, 36/54/52).
template <int G>
__device__ __forceinline__ int group_id() {
    const int g = (int)threadIdx.x / G;
    return G == 64 ? __builtin_amdgcn_readfirstlane(g) : g;
}
template <int G>
__device__ __forceinline__ int held_by(int x, int k) {
    return G == 64 ? __builtin_amdgcn_readlane(x, k) : __shfl(x, k, G);
}
template <int G>
__device__ __forceinline__ float held_by(float x, int k) { return __int_as_float(held_by<G>(__float_as_int(x), k)); }
__device__ __forceinline__ float dot4(const float4& a, const float4& b) {
    return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
}
__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// pq[v] = (p_v, q_v) from the two score columns of T_ext (compact copy: stays in L2).
__global__ __launch_bounds__(256) void gat_extract_pq_kernel(const float* __restrict__ Tx, int64_t ldx, int col_p, int64_t n,
                                                             float2* __restrict__ pq) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < n) pq[v] = make_float2(Tx[v * ldx + col_p], Tx[v * ldx + col_p + 1]);
}

// Row statistics of the attention softmax: rowstat[v] = (m_v, Z_v) = (max_u e_uv, sum_u exp(e_uv - m_v)),
// self term included.  Scalars only (p and q sit in L2).  The first n_long workgroups each take one
// row longer than long_thr edges with all their threads (partial results combined through LDS in a
// fixed order): the launch lasts as long as the longest row, a chain of gathers.  The others give G lanes to a row and skip the long ones.
// G: 4 up to 16 edges a row on average (four gathers a lane), else 16.
constexpr int GAT_STATS_THREADS = 1024;
template <int G>
__global__ __launch_bounds__(GAT_STATS_THREADS) void gat_stats_kernel(const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx,
                                                        int64_t n, const float2* __restrict__ pq,
                                                        float2* __restrict__ rowstat, const int32_t* __restrict__ long_row,
                                                        int n_long, int64_t long_thr) {
    constexpr int T = GAT_STATS_THREADS, WAVES = T / 64;
    if ((int)blockIdx.x < n_long) {
        __shared__ float red[WAVES];
        const int64_t v = long_row[blockIdx.x];
        const int64_t b = ptr[v], e = ptr[v + 1];
        const float2 pqv = pq[v];
        const float es = leaky(pqv.x + pqv.y);
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        auto score = [&](int64_t k) { return k < e ? leaky(pq[idx[k]].x + pqv.y) : -INFINITY; };
        float mx = es;
        for (int64_t k = b + tid; k < e; k += 4 * T) {
            const float s0 = score(k), s1 = score(k + T), s2 = score(k + 2 * T), s3 = score(k + 3 * T);
            mx = fmaxf(fmaxf(mx, fmaxf(s0, s1)), fmaxf(s2, s3));
        }
        mx = group_max<64>(mx);
        if (lane == 0) red[wave] = mx;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES; ++w) mx = fmaxf(mx, red[w]);
        __syncthreads();
        float sum = 0.f;
        for (int64_t k = b + tid; k < e; k += 4 * T) {
            const float s0 = score(k), s1 = score(k + T), s2 = score(k + 2 * T), s3 = score(k + 3 * T);
            sum += __expf(s0 - mx); sum += __expf(s1 - mx); sum += __expf(s2 - mx); sum += __expf(s3 - mx);
        }
        sum = group_sum<64>(sum);
        if (lane == 0) red[wave] = sum;
        __syncthreads();
        if (tid == 0) {
            float all = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; w += 4) all += (red[w] + red[w + 1]) + (red[w + 2] + red[w + 3]);
            rowstat[v] = make_float2(mx, all + __expf(es - mx));
        }
        return;
    }
    const int t = threadIdx.x % G;
    const int64_t v = ((int64_t)blockIdx.x - n_long) * (T / G) + threadIdx.x / G;
    if (v >= n) return;               // whole groups leave together
    const int64_t b = ptr[v], e = ptr[v + 1];
    if (e - b > long_thr) return;     // done by one of the first workgroups
    const float2 pqv = pq[v];
    const float es = leaky(pqv.x + pqv.y);
    // four independent index -> score gathers per lane and trip
    auto score = [&](int64_t k) { return k < e ? leaky(pq[idx[k]].x + pqv.y) : -INFINITY; };
    const float f0 = score(b + t), f1 = score(b + t + G), f2 = score(b + t + 2 * G), f3 = score(b + t + 3 * G);      // the first trip's are kept
    float mx = fmaxf(fmaxf(fmaxf(es, f0), fmaxf(f1, f2)), f3);
    for (int64_t k = b + 4 * G + t; k < e; k += 4 * G) {
        const float s0 = score(k), s1 = score(k + G), s2 = score(k + 2 * G), s3 = score(k + 3 * G);
        mx = fmaxf(fmaxf(mx, fmaxf(s0, s1)), fmaxf(s2, s3));
    }
    mx = group_max<G>(mx);
    float sum = (__expf(f0 - mx) + __expf(f1 - mx)) + (__expf(f2 - mx) + __expf(f3 - mx));
    for (int64_t k = b + 4 * G + t; k < e; k += 4 * G) {
        const float s0 = score(k), s1 = score(k + G), s2 = score(k + 2 * G), s3 = score(k + 3 * G);
        sum += (__expf(s0 - mx) + __expf(s1 - mx)) + (__expf(s2 - mx) + __expf(s3 - mx));
    }
    sum = group_sum<G>(sum) + __expf(es - mx);
    if (t == 0) rowstat[v] = make_float2(mx, sum);
}

// The three edge walks share one skeleton.  A walk visits the edges of a row (of the CSR for
// FWD and DST, of the CSC for SRC) and accumulates a feature row `acc` and a scalar `scal`:
//   FWD  acc += alpha_uv T[u,:]                                           (row v, edges u -> v)
//   DST  scal += alpha_uv (dOut_v . T[u,:] - c_v) LeakyReLU'(pre_uv)      (row v; acc unused)
//        (the slope LeakyReLU' here less that of the self edge, so that only some of the edges are looked at: see gat_walk_edges)
//   SRC  acc += alpha_uv dOut[v,:];  scal += alpha_uv (T_u . dOut[v,:] - c_v) LeakyReLU'(pre_uv)   (row u, edges u -> v)
// Short rows are walked by one group of G lanes.  Rows longer than `long_thr` edges use the
// partition's split schedule: the first workgroups of the launch each walk one chunk (their
// 256/G groups take contiguous slices, summed through LDS in a fixed order) into a partial
// row; a second kernel adds a row's partials in chunk order and finishes it.
enum { GAT_FWD = 0, GAT_DST = 1, GAT_SRC = 2 };

struct GatWalk {
    const int64_t* ptr;
    const int32_t* idx;
    int64_t n;
    int F;
    const float* Tx;  int64_t ldx;
    const float2* pq;
    float2* rowstat;                     // (m_v, Z_v); FWD: Z_v negated where out_v is not finite before the ReLU, which hides it; DST: read
    const float* bias;
    int relu;
    float* Hout;      int64_t ldh;       // FWD: output; DST: the layer's stored output
    float hout_scale;                    // DST: out_v = hout_scale * Hout[v,:] where dOut is non-zero (undoes dropout)
    const float* dOut; int64_t ldd;
    float4* dst;                         // (q_v, m_v, 1 / Z_v, c_v), what an edge needs of its destination: DST: written; SRC: read
    float* dq;                           // without the self edge's term.  DST: written; SRC: read
    float* colsum;                       // DST: [workgroups of rows x F] partial column sums of dOut
    float* dTx;                          // SRC: output rows [dT | 0 | dp | dq | 0 0]
    int64_t long_thr;
    int n_chunks;
    const int64_t* chunk_begin;
    const int64_t* chunk_end;
    float* partials;  int64_t ld_part;   // [n_chunks x ld_part]: F columns, the scalar at column ld(F)
};

template <int G, int NJ>
struct GatRow {                          // per-row constants held by every lane of the group
    float4 vec[NJ];                      // DST: dOut[v,:]; SRC: T[u,:]
    float p;
    float q, mx, inv, c;                 // (SRC: not held)
    bool all;                            // DST: edges that add zero are walked too
};

template <int PASS, int G, int NJ>
__device__ __forceinline__ void gat_row_setup(const GatWalk& A, int64_t r, int t, const bool (&live)[NJ], GatRow<G, NJ>& R) {
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    R.p = A.pq[r].x;
    if (PASS == GAT_SRC) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) R.vec[j] = live[j] ? ld4(A.Tx + r * A.ldx + 4 * (t + G * j)) : zero;
        return;
    }
    const float2 st = A.rowstat[r];
    R.q = A.pq[r].y;
    R.mx = st.x; R.inv = 1.f / fabsf(st.y);
    R.c = 0.f;
    if (PASS == GAT_DST) {
        float cpart = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            R.vec[j] = zero;
            if (!live[j]) continue;
            const int col = 4 * (t + G * j);
            R.vec[j] = ld4(A.dOut + r * A.ldd + col);
            const float4 h = ld4(A.Hout + r * A.ldh + col);
            float bb[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) bb[q] = col + q < A.F ? A.bias[col + q] : 0.f;
            const float hs = A.hout_scale;
            cpart += R.vec[j].x * (h.x * hs - bb[0]) + R.vec[j].y * (h.y * hs - bb[1]) + R.vec[j].z * (h.z * hs - bb[2]) +
                     R.vec[j].w * (h.w * hs - bb[3]);
        }
        R.c = group_sum<G>(cpart);        // c_v = dOut_v . (out_v - b) = sum_u alpha_uv (dOut_v . t_u)
        R.all = st.y < 0.f || !(fabsf(R.c) < INFINITY);
    }
}

template <int PASS, int G, int NJ>
__device__ __forceinline__ void gat_walk_edges(const GatWalk& A, const GatRow<G, NJ>& R, int64_t b, int64_t e, int first, int t,
                                               const bool (&live)[NJ], float4 (&acc)[NJ], float& scal) {
    // DST adds up alpha_uv (dOut_v . t_u - c_v) LeakyReLU'(pre_uv) over a row.  Without the last factor that sum is zero, so the
    // self edge's slope is taken off every factor: what is left are the edges on the other side of the kink, instead of
    // terms of both signs that cancel to rounding noise (the self edge itself then adds nothing).  The others add nothing and their rows
    // of T are not fetched, but where c_v or one of the t_u is not finite: 0 times that is not zero.  (Where both are, a product dOut_v . t_u that
    // overflows counts only for the edges across the kink.)  3e5 rows of 256 columns, 3.25
    // skewed edges a row, the bias gradient's column sums included: 308 + 45 -> 225 us.
    const float slope0 = PASS == GAT_DST ? leaky_d(R.p + R.q) : 0.f;
    for (int64_t base = b; base < e; base += G) {
        const int cnt = (int)(e - base < G ? e - base : G);
        int mine = 0;
        float mya = 0.f, mw = 0.f, mc = PASS == GAT_SRC ? 0.f : R.c;              // alpha, alpha * LeakyReLU', c of the edge's destination
        if (t < cnt) {
            mine = PASS == GAT_DST && base == b ? first : A.idx[base + t];      // (asked for before the row itself)
            float pre, mx, inv;
            if (PASS == GAT_SRC) {
                const float4 to = A.dst[mine];
                pre = R.p + to.x; mx = to.y; inv = to.z; mc = to.w;
            } else {
                pre = A.pq[mine].x + R.q; mx = R.mx; inv = R.inv;
            }
            mya = __expf(leaky(pre) - mx) * inv;
            mw = mya * (leaky_d(pre) - slope0);
        }
        if constexpr (PASS == GAT_DST) {
            unsigned long long who = __ballot(t < cnt && (R.all || mw != 0.f));      // (NaN is not 0)
            if (G < 64) who = (who >> ((threadIdx.x & 63) / G * G)) & ((1ull << (G & 63)) - 1ull);
            while (who) {                                  // the edges that are walked, two at a time
                const int k0 = __ffsll(who) - 1;
                who &= who - 1;
                const bool two = who != 0;
                const int k1 = two ? __ffsll(who) - 1 : k0;
                who &= who - 1;
                const int64_t c0 = held_by<G>(mine, k0), c1 = held_by<G>(mine, k1);
                float d0 = 0.f, d1 = 0.f;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if (!live[j]) continue;
                    const float4 v0 = ld4(A.Tx + c0 * A.ldx + 4 * (t + G * j)), v1 = ld4(A.Tx + c1 * A.ldx + 4 * (t + G * j));
                    d0 += dot4(R.vec[j], v0); d1 += dot4(R.vec[j], v1);
                }
                d0 = group_sum<G>(d0); d1 = group_sum<G>(d1);
                scal += held_by<G>(mw, k0) * (d0 - R.c);
                const float w1 = held_by<G>(mw, k1);
                if (two) scal += w1 * (d1 - R.c);
            }
            continue;
        }
        for (int k = 0; k < cnt; k += 4) {
            const bool p1 = k + 1 < cnt, p2 = k + 2 < cnt, p3 = k + 3 < cnt;
            const int k1 = p1 ? k + 1 : k, k2 = p2 ? k + 2 : k, k3 = p3 ? k + 3 : k;
            const int64_t c0 = held_by<G>(mine, k), c1 = held_by<G>(mine, k1), c2 = held_by<G>(mine, k2), c3 = held_by<G>(mine, k3);
            const float a0 = held_by<G>(mya, k), a1 = p1 ? held_by<G>(mya, k1) : 0.f;
            const float a2 = p2 ? held_by<G>(mya, k2) : 0.f, a3 = p3 ? held_by<G>(mya, k3) : 0.f;
            float d0 = 0.f, d1 = 0.f, d2 = 0.f, d3 = 0.f;
            const float* base_ptr = PASS == GAT_SRC ? A.dOut : A.Tx;
            const int64_t ld = PASS == GAT_SRC ? A.ldd : A.ldx;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (!live[j]) continue;
                const int col = 4 * (t + G * j);
                const float4 v0 = ld4(base_ptr + c0 * ld + col), v1 = ld4(base_ptr + c1 * ld + col);
                const float4 v2 = ld4(base_ptr + c2 * ld + col), v3 = ld4(base_ptr + c3 * ld + col);
                {
                    acc[j].x += a0 * v0.x; acc[j].y += a0 * v0.y; acc[j].z += a0 * v0.z; acc[j].w += a0 * v0.w;
                    acc[j].x += a1 * v1.x; acc[j].y += a1 * v1.y; acc[j].z += a1 * v1.z; acc[j].w += a1 * v1.w;
                    acc[j].x += a2 * v2.x; acc[j].y += a2 * v2.y; acc[j].z += a2 * v2.z; acc[j].w += a2 * v2.w;
                    acc[j].x += a3 * v3.x; acc[j].y += a3 * v3.y; acc[j].z += a3 * v3.z; acc[j].w += a3 * v3.w;
                }
                if (PASS != GAT_FWD) {
                    d0 += dot4(R.vec[j], v0); d1 += dot4(R.vec[j], v1); d2 += dot4(R.vec[j], v2); d3 += dot4(R.vec[j], v3);
                }
            }
            if (PASS != GAT_FWD) {
                d0 = group_sum<G>(d0); d1 = group_sum<G>(d1); d2 = group_sum<G>(d2); d3 = group_sum<G>(d3);
                scal += held_by<G>(mw, k) * (d0 - held_by<G>(mc, k));
                const float w1 = held_by<G>(mw, k1), w2 = held_by<G>(mw, k2), w3 = held_by<G>(mw, k3);
                const float e1 = held_by<G>(mc, k1), e2 = held_by<G>(mc, k2), e3 = held_by<G>(mc, k3);
                if (p1) scal += w1 * (d1 - e1);
                if (p2) scal += w2 * (d2 - e2);
                if (p3) scal += w3 * (d3 - e3);
            }
        }
    }
}

// Adds the self term and writes the row's results.
template <int PASS, int G, int NJ>
__device__ __forceinline__ void gat_row_finish(const GatWalk& A, const GatRow<G, NJ>& R, int64_t r, int t,
                                               const bool (&live)[NJ], float4 (&acc)[NJ], float scal) {
    if (PASS == GAT_FWD) {
        const float as = __expf(leaky(R.p + R.q) - R.mx) * R.inv;
        bool odd = false;                 // one of the t_u is not finite (a weight of zero does not hide it)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (!live[j]) continue;
            const int col = 4 * (t + G * j);
            const float4 tv = ld4(A.Tx + r * A.ldx + col);
            float o[4] = {acc[j].x + as * tv.x, acc[j].y + as * tv.y, acc[j].z + as * tv.z, acc[j].w + as * tv.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                odd = odd || !(fabsf(o[q]) < INFINITY);
                if (col + q < A.F) {
                    o[q] += A.bias[col + q];
                    if (A.relu) o[q] = o[q] > 0.f ? o[q] : 0.f;
                } else {
                    o[q] = 0.f;       // pad columns stay zero
                }
            }
            *reinterpret_cast<float4*>(A.Hout + r * A.ldh + col) = make_float4(o[0], o[1], o[2], o[3]);
        }
        if (odd) A.rowstat[r].y = -fabsf(A.rowstat[r].y);      // (every lane that sees one writes the same)
    } else if (PASS == GAT_DST) {
        if (t == 0) {
            A.dst[r] = make_float4(R.q, R.mx, R.inv, R.c);
            A.dq[r] = scal;
        }
    } else {
        const float4 to = A.dst[r];
        const float pre = R.p + to.x, as = __expf(leaky(pre) - to.y) * to.z;
        float own = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (!live[j]) continue;
            const int col = 4 * (t + G * j);
            const float4 d = ld4(A.dOut + r * A.ldd + col);
            own += dot4(R.vec[j], d);
            float o[4] = {acc[j].x + as * d.x, acc[j].y + as * d.y, acc[j].z + as * d.z, acc[j].w + as * d.w};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (col + q >= A.F) o[q] = 0.f;
            *reinterpret_cast<float4*>(A.dTx + r * A.ldx + col) = make_float4(o[0], o[1], o[2], o[3]);
        }
        own = as * (group_sum<G>(own) - to.w) * leaky_d(pre);      // the self edge's score gradient
        if (t == 0)
            *reinterpret_cast<float4*>(A.dTx + r * A.ldx + ((A.F + 3) & ~3)) = make_float4(scal + own, A.dq[r], 0.f, 0.f);
    }
}

template <int PASS, int G, int NJ>
__global__ __launch_bounds__(256) void gat_walk_kernel(GatWalk A) {
    constexpr int ROWS = 256 / G;
    constexpr int W = 4 * G * NJ;                 // padded row width held by a group
    __shared__ __attribute__((aligned(16))) float red[ROWS * (W + 4)];
    __shared__ int64_t chunk_row;
    const int t = threadIdx.x % G, gi = group_id<G>();
    bool live[NJ];
    float4 acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        live[j] = 4 * (t + G * j) < A.F;
        acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    GatRow<G, NJ> R;
    float scal = 0.f;
    if ((int)blockIdx.x < A.n_chunks) {           // uniform per workgroup: one chunk of a long row
        const int64_t cb = A.chunk_begin[blockIdx.x], ce = A.chunk_end[blockIdx.x];
        if (threadIdx.x == 0) {                   // the row that owns edge cb: last r with ptr[r] <= cb
            int64_t lo = 0, hi = A.n;
            while (hi - lo > 1) {
                const int64_t mid = (lo + hi) >> 1;
                if (A.ptr[mid] <= cb) lo = mid; else hi = mid;
            }
            chunk_row = lo;
        }
        __syncthreads();
        const int64_t r = chunk_row;
        const int64_t per = (ce - cb + ROWS - 1) / ROWS;
        int64_t b = cb + gi * per, e = b + per;
        if (b > ce) b = ce;
        if (e > ce) e = ce;
        const int first = PASS == GAT_DST && b + t < e ? A.idx[b + t] : 0;
        gat_row_setup<PASS, G, NJ>(A, r, t, live, R);
        gat_walk_edges<PASS, G, NJ>(A, R, b, e, first, t, live, acc, scal);
#pragma unroll
        for (int j = 0; j < NJ; ++j) *reinterpret_cast<float4*>(&red[gi * (W + 4) + 4 * (t + G * j)]) = acc[j];
        if (t == 0) red[gi * (W + 4) + W] = scal;
        __syncthreads();
        float* prow = A.partials + (int64_t)blockIdx.x * A.ld_part;
        const int fpad = (A.F + 3) & ~3;
        for (int c = threadIdx.x; c <= fpad; c += 256) {
            const int cc = c < fpad ? c : W;      // the last one is the scalar
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < ROWS; ++q) s += red[q * (W + 4) + cc];
            prow[c] = s;
        }
        return;
    }
    if constexpr (PASS == GAT_DST) {
        // several rows a group: its column sums of dOut, which it reads anyway, stay in registers until the last
        const int block = (int)blockIdx.x - A.n_chunks, blocks = (int)gridDim.x - A.n_chunks;
        float4 csum[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) csum[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        // (Asking for the next row while the edges of one are walked took 14 more registers and 46 us more.)
        for (int64_t r = (int64_t)block * ROWS + gi; r < A.n; r += (int64_t)blocks * ROWS) {
            const int64_t b = A.ptr[r], e = A.ptr[r + 1];
            const int first = b + t < e ? A.idx[b + t] : 0;
            gat_row_setup<PASS, G, NJ>(A, r, t, live, R);
#pragma unroll
            for (int j = 0; j < NJ; ++j) { csum[j].x += R.vec[j].x; csum[j].y += R.vec[j].y; csum[j].z += R.vec[j].z; csum[j].w += R.vec[j].w; }
            if (e - b > A.long_thr) continue;     // walked in chunks above, finished by the combine kernel
            scal = 0.f;
            gat_walk_edges<PASS, G, NJ>(A, R, b, e, first, t, live, acc, scal);
            gat_row_finish<PASS, G, NJ>(A, R, r, t, live, acc, scal);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) *reinterpret_cast<float4*>(&red[gi * (W + 4) + 4 * (t + G * j)]) = csum[j];
        __syncthreads();
        for (int c = threadIdx.x; c < A.F; c += 256) {
            float sum = 0.f;
#pragma unroll
            for (int q = 0; q < ROWS; ++q) sum += red[q * (W + 4) + c];
            A.colsum[(int64_t)block * A.F + c] = sum;
        }
    } else {
        const int64_t r = (int64_t)(blockIdx.x - A.n_chunks) * ROWS + gi;
        if (r >= A.n) return;                         // whole groups leave together
        const int64_t b = A.ptr[r], e = A.ptr[r + 1];
        if (e - b > A.long_thr) return;               // walked in chunks above, finished by the combine kernel
        gat_row_setup<PASS, G, NJ>(A, r, t, live, R);
        gat_walk_edges<PASS, G, NJ>(A, R, b, e, 0, t, live, acc, scal);
        gat_row_finish<PASS, G, NJ>(A, R, r, t, live, acc, scal);
    }
}

// Workgroups of rows of a DST walk: as many as run at a time (each leaves a partial row of column sums).
constexpr int GAT_DST_BLOCKS = 2048;

template <int PASS, int G, int NJ>
__global__ __launch_bounds__(256) void gat_combine_kernel(GatWalk A, const int32_t* __restrict__ long_row,
                                                          const int32_t* __restrict__ long_first, int n_long) {
    constexpr int ROWS = 256 / G;
    const int t = threadIdx.x % G;
    const int j0 = blockIdx.x * ROWS + group_id<G>();
    if (j0 >= n_long) return;
    const int64_t r = long_row[j0];
    const int c0 = long_first[j0], c1 = long_first[j0 + 1];
    bool live[NJ];
    float4 acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        live[j] = 4 * (t + G * j) < A.F;
        acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    GatRow<G, NJ> R;
    float scal = 0.f;
    gat_row_setup<PASS, G, NJ>(A, r, t, live, R);
    const int fpad = (A.F + 3) & ~3;
    struct Part { float4 v[NJ]; float s; };
    in_order(c0, c1,
             [&](int c) {
                 const float* prow = A.partials + (int64_t)c * A.ld_part;
                 Part p;
#pragma unroll
                 for (int j = 0; j < NJ; ++j) p.v[j] = ld4(prow + (live[j] ? 4 * (t + G * j) : 0));
                 p.s = prow[fpad];
                 return p;
             },
             [&](const Part& p, bool on) {
#pragma unroll
                 for (int j = 0; j < NJ; ++j) {
                     const bool is = on && live[j];
                     acc[j].x += is ? p.v[j].x : 0.f; acc[j].y += is ? p.v[j].y : 0.f;
                     acc[j].z += is ? p.v[j].z : 0.f; acc[j].w += is ? p.v[j].w : 0.f;
                 }
                 scal += on ? p.s : 0.f;
             });
    gat_row_finish<PASS, G, NJ>(A, R, r, t, live, acc, scal);
}

// Packed weights of one layer: Wp[Fin x ldx] = wp_scale [W | 0 | W a_src | W a_dst | 0 0] (rows of the
// product dT_ext -> dH; wp_scale = 1 / (1 - rate) when the layer's input went through dropout) and the
// unscaled transpose Wt[ldx x ld(Fin)] (rows of the product H -> T_ext).
// The first workgroups multiply W by the attention vectors, a row a wavefront (one thread a row: 15 us at 256 x 256).
__global__ __launch_bounds__(256) void gat_pack_kernel(const float* __restrict__ W, const float* __restrict__ a_s,
                                                       const float* __restrict__ a_d, int fin, int fout, int fin_pad, int ldx,
                                                       float wp_scale, float* __restrict__ Wp, float* __restrict__ Wt) {
    const int cp = (fout + 3) & ~3, score_blocks = (fin_pad + 3) / 4;
    auto put = [&](int i, int c, float val) {
        if (i < fin) Wp[(int64_t)i * ldx + c] = val * wp_scale;
        Wt[(int64_t)c * fin_pad + i] = val;
    };
    if ((int)blockIdx.x < score_blocks) {
        const int i = 4 * blockIdx.x + (threadIdx.x >> 6), lane = threadIdx.x & 63;
        if (i >= fin_pad) return;
        float s = 0.f, d = 0.f;
        for (int j = lane; i < fin && j < fout; j += 64) {
            const float w = W[(int64_t)i * fout + j];
            s = fmaf(w, a_s[j], s);
            d = fmaf(w, a_d[j], d);
        }
        s = group_sum<64>(s);
        d = group_sum<64>(d);
        if (lane < 2) put(i, cp + lane, lane ? d : s);
        return;
    }
    const int64_t e = (int64_t)(blockIdx.x - score_blocks) * 256 + threadIdx.x;
    if (e >= (int64_t)fin_pad * ldx) return;
    const int i = (int)(e / ldx), c = (int)(e % ldx);
    if (c == cp || c == cp + 1) return;
    put(i, c, i < fin && c < fout ? W[(int64_t)i * fout + c] : 0.f);
}

// Gradients of W, a_src, a_dst from dWx = H^T dT_ext [Fin x ldx]:
//   dW = dWx[:, :F] + dWx[:, cp] a_src^T + dWx[:, cp+1] a_dst^T,  da_src = W^T dWx[:, cp],  da_dst = W^T dWx[:, cp+1].
// (The bias gradient comes along from where the step's sums left it.)
__global__ __launch_bounds__(256) void gat_param_grad_kernel(const float* __restrict__ dWx, const float* __restrict__ dbias, int ldx, const float* __restrict__ W,
                                                             const float* __restrict__ a_s, const float* __restrict__ a_d,
                                                             int fin, int fout, float* __restrict__ gW,
                                                             float* __restrict__ ga_s, float* __restrict__ ga_d, float* __restrict__ gb) {
    // workgroup j < fout: column j of dW and the two attention-vector gradients of index j
    __shared__ float sm[8];
    const int cp = (fout + 3) & ~3;
    const int j = blockIdx.x;
    float s = 0.f, d = 0.f;
    const float asj = a_s[j], adj = a_d[j];
    for (int i = threadIdx.x; i < fin; i += 256) {
        const float ds = dWx[(int64_t)i * ldx + cp], dd = dWx[(int64_t)i * ldx + cp + 1];
        const float w = W[(int64_t)i * fout + j];
        gW[(int64_t)i * fout + j] = dWx[(int64_t)i * ldx + j] + ds * asj + dd * adj;
        s = fmaf(w, ds, s);
        d = fmaf(w, dd, d);
    }
    for (int o = 32; o > 0; o >>= 1) { s += __shfl_down(s, o, 64); d += __shfl_down(d, o, 64); }
    if ((threadIdx.x & 63) == 0) { sm[threadIdx.x >> 6] = s; sm[4 + (threadIdx.x >> 6)] = d; }
    __syncthreads();
    if (threadIdx.x == 0) {
        ga_s[j] = (sm[0] + sm[1]) + (sm[2] + sm[3]);
        ga_d[j] = (sm[4] + sm[5]) + (sm[6] + sm[7]);
        gb[j] = dbias[j];
    }
}

// ------------------------------------------------------------------ launchers
struct GatLayer {
    int fin, fout;
    int64_t ldx, ldh, ldin_pad;      // ld(Fout) + 4; ld(Fout); ld(Fin)
    int64_t off_w, off_as, off_ad, off_b;
    float *Wp, *Wt, *Tx, *Hout;
    float2 *pq, *rowstat;
    // what the step's sums (StepSums) read and write
    float *dWx, *dbias, *colsum;
    void* tn_ws;
    size_t tn_ws_bytes;
};

struct GatPlan {
    std::vector<GatLayer> L;
    float *dZa, *dZb, *dTx, *dq, *partials;
    char* base;
    float4* dst;
    void* stats_ws;
    size_t total;
    unsigned char* planes = nullptr;   // the weights of the product at hand, split (GemmNNArgs::planes)
    size_t planes_bytes = 0;
};

static inline int64_t ldp4(int64_t f) { return round_up(f, 4); }

static GatPlan gat_plan(const grp_partition_t* part, const grp_model_desc* m, void* ws, size_t ws_bytes) {
    GatPlan p;
    Bump b(ws, ws_bytes);
    const int64_t n = part->n;
    const int k = m->n_layers;
    p.L.resize(k);
    int64_t off = 0, ldmax = 4, ldxmax = 8;
    size_t pl_bytes = 0;
    p.base = (char*)ws;
    for (int l = 0; l < k; ++l) {          // first: within reach of 32-bit numbers of floats
        GatLayer& L = p.L[l];
        L.fin = m->dims[l]; L.fout = m->dims[l + 1];
        L.ldh = ldp4(L.fout); L.ldx = L.ldh + 4; L.ldin_pad = ldp4(L.fin);
        L.dWx = b.take<float>((size_t)L.fin * L.ldx);
        L.dbias = b.take<float>((size_t)L.fout);
        L.colsum = b.take<float>((size_t)GAT_DST_BLOCKS * L.ldx);
        L.tn_ws_bytes = gemm_tn_workspace_bytes(n, L.fin, (int32_t)L.ldx);
        L.tn_ws = b.take<char>(L.tn_ws_bytes);
    }
    for (int l = 0; l < k; ++l) {
        GatLayer& L = p.L[l];
        L.off_w = off; off += (int64_t)L.fin * L.fout;
        L.off_as = off; off += L.fout;
        L.off_ad = off; off += L.fout;
        L.off_b = off; off += L.fout;
        L.Wp = b.take<float>((size_t)L.ldin_pad * L.ldx);
        L.Wt = b.take<float>((size_t)L.ldx * L.ldin_pad);
        L.Tx = b.take<float>((size_t)n * L.ldx);
        L.Hout = b.take<float>((size_t)n * L.ldh);
        L.pq = b.take<float2>((size_t)n);
        L.rowstat = b.take<float2>((size_t)n);
        if (L.ldh > ldmax) ldmax = L.ldh;
        if (L.ldx > ldxmax) ldxmax = L.ldx;
        pl_bytes = std::max({pl_bytes, gemm_planes_bytes(n, (int32_t)L.ldx, L.fin), gemm_planes_bytes(n, L.fin, (int32_t)L.ldx)});
    }
    p.dZa = b.take<float>((size_t)n * ldmax);
    p.dZb = b.take<float>((size_t)n * ldmax);
    p.dTx = b.take<float>((size_t)n * ldxmax);
    p.dst = b.take<float4>((size_t)n);
    p.dq = b.take<float>((size_t)n);
    const int64_t chunks_cap = part->csr_long.n_chunks > part->csc_long.n_chunks ? part->csr_long.n_chunks : part->csc_long.n_chunks;
    p.partials = b.take<float>((size_t)chunks_cap * ldxmax);
    if (pl_bytes > 0) p.planes = b.take<unsigned char>(pl_bytes);
    p.planes_bytes = pl_bytes;
    p.stats_ws = b.take<char>(stats_workspace_bytes(n));
    p.total = b.total();
    return p;
}

size_t gat_step_workspace_bytes(const grp_partition_t* part, const grp_model_desc* m) {
    return gat_plan(part, m, nullptr, 0).total;
}

void gat_step_activation(const grp_partition_t* part, const grp_model_desc* m, void* ws, size_t ws_bytes, int layer,
                         const float** out, int64_t* ld) {
    const GatPlan p = gat_plan(part, m, ws, ws_bytes);
    *out = p.L[layer].Hout;
    *ld = p.L[layer].ldh;
}

template <int PASS, int G, int NJ>
static void gat_walk_one(const GatWalk& A, const LongRows* lr, StepSums* sums, float* dbias, hipStream_t st) {
    constexpr int ROWS = 256 / G;
    const int64_t blocks = PASS == GAT_DST ? std::min<int64_t>(cdiv(A.n, ROWS), GAT_DST_BLOCKS) : cdiv(A.n, ROWS);
    hipLaunchKernelGGL((gat_walk_kernel<PASS, G, NJ>), dim3((unsigned)(A.n_chunks + blocks)), dim3(256), 0, st, A);
    if (PASS == GAT_DST) sums->add(SUM_COLUMNS, A.colsum, (int32_t)blocks, 0, A.F, 0, dbias, nullptr, nullptr, A.F);
    if (A.n_chunks > 0)
        hipLaunchKernelGGL((gat_combine_kernel<PASS, G, NJ>), dim3((unsigned)cdiv(lr->n_long, ROWS)), dim3(256), 0, st, A,
                           (const int32_t*)lr->long_row, (const int32_t*)lr->long_first, lr->n_long);
}

template <int PASS>
static grp_status launch_gat_walk(GatWalk A, const LongRows* lr, float* partials, hipStream_t st, StepSums* sums = nullptr, float* dbias = nullptr /*DST: column sums of dOut*/) {
    const bool split = lr && lr->n_long > 0;
    A.long_thr = split ? (int64_t)SPMM_LONG_ROW : INT64_MAX;
    A.n_chunks = split ? lr->n_chunks : 0;
    A.chunk_begin = split ? lr->chunk_begin : nullptr;
    A.chunk_end = split ? lr->chunk_end : nullptr;
    A.partials = partials;
    A.ld_part = round_up(A.F, 4) + 4;
    const int f4 = (A.F + 3) / 4;
    if (f4 <= 1) gat_walk_one<PASS, 1, 1>(A, lr, sums, dbias, st);
    else if (f4 <= 2) gat_walk_one<PASS, 2, 1>(A, lr, sums, dbias, st);
    else if (f4 <= 4) gat_walk_one<PASS, 4, 1>(A, lr, sums, dbias, st);
    else if (f4 <= 8) gat_walk_one<PASS, 8, 1>(A, lr, sums, dbias, st);
    else if (f4 <= 16) gat_walk_one<PASS, 16, 1>(A, lr, sums, dbias, st);
    else if (f4 <= 32) gat_walk_one<PASS, 32, 1>(A, lr, sums, dbias, st);
    else if (f4 <= 64) gat_walk_one<PASS, 64, 1>(A, lr, sums, dbias, st);
    else if (f4 <= 128) gat_walk_one<PASS, 64, 2>(A, lr, sums, dbias, st);
    else gat_walk_one<PASS, 64, 4>(A, lr, sums, dbias, st);
    GRP_LAUNCH_CHECK();
    return GRP_OK;
}

grp_status gat_step(const grp_partition_t* g, const grp_model_desc* m, const grp_step_opts* o, const void* X,
                    const int32_t* labels, const uint8_t* mask, const float* theta, void* ws, size_t ws_bytes,
                    hipStream_t st, float* grad, grp_step_stats* stats) {
    GatPlan p = gat_plan(g, m, ws, ws_bytes);
    const int64_t n = g->n;
    const int k = m->n_layers;
    StepPrelude pre;
    StatsIn& si = pre.stats;
    si.n_loss = n; si.mask = mask; si.d_local = g->d_local_in; si.d_global = g->d_global_in; si.nnz_const = g->nnz; si.scratch = p.stats_ws;
    GRP_TRY(launch_prelude(pre, st));
    if (n == 0) {                                       // nothing to train on: zero gradient
        int64_t P = 0;
        for (int l = 0; l < k; ++l) P += (int64_t)m->dims[l] * m->dims[l + 1] + 3 * m->dims[l + 1];
        GRP_TRY(launch_fill_zero(grad, (size_t)P * sizeof(float), st));      // a kernel, so the step can be captured in a graph
        return launch_softmax_xent(si, m->dims[k], nullptr, 4, labels, o->estimator == GRP_EST_NODE_LEVEL, nullptr, p.dZa, 4, stats, st);
    }
    const DropoutPlan drop = dropout_plan(o);
    // ---------------- packed weights
    for (int l = 0; l < k; ++l) {
        const GatLayer& L = p.L[l];
        ProfScope ps("gat_pack_weights", st);
        hipLaunchKernelGGL(gat_pack_kernel, dim3((unsigned)(cdiv(L.ldin_pad, 4) + cdiv((int64_t)L.ldin_pad * L.ldx, 256))), dim3(256), 0, st,
                           theta + L.off_w, theta + L.off_as, theta + L.off_ad, L.fin, L.fout, (int)L.ldin_pad, (int)L.ldx,
                           l > 0 ? drop.scale : 1.f, L.Wp, L.Wt);
        GRP_LAUNCH_CHECK();
    }
    // ---------------- forward
    const void* H = X;
    int64_t ldh = m->dims[0];
    int h_bf16 = m->feat_dtype == GRP_DTYPE_BF16;
    for (int l = 0; l < k; ++l) {
        const GatLayer& L = p.L[l];
        GemmNNArgs a;          // T_ext = H [W | 0 | W a_src | W a_dst | 0 0]
        a.planes = p.planes; a.planes_bytes = p.planes_bytes;
        a.M = n; a.N = (int)L.ldx; a.K = L.fin; a.A = H; a.lda = ldh; a.a_bf16 = h_bf16; a.Bt = L.Wt; a.ldbt = L.ldin_pad;
        a.C = L.Tx; a.ldc = L.ldx;
        GRP_TRY(launch_gemm_nn(a, st));
        {
            ProfScope ps("gat_forward", st, 2.0 * g->nnz * L.fout, 4.0 * g->nnz + 8.0 * L.fout * n);
            hipLaunchKernelGGL(gat_extract_pq_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, L.Tx, L.ldx, (int)L.ldh, n, L.pq);
            const bool few = g->nnz <= 16 * n;
            const dim3 grid((unsigned)(cdiv(n, GAT_STATS_THREADS / (few ? 4 : 16)) + g->csr_long.n_long));
            hipLaunchKernelGGL(few ? gat_stats_kernel<4> : gat_stats_kernel<16>, grid, dim3(GAT_STATS_THREADS), 0, st, g->rowptr, g->col, n,
                               (const float2*)L.pq, L.rowstat, g->csr_long.long_row, g->csr_long.n_long, (int64_t)SPMM_LONG_ROW);
            GRP_LAUNCH_CHECK();
            GatWalk A{};
            A.ptr = g->rowptr; A.idx = g->col; A.n = n; A.F = L.fout; A.Tx = L.Tx; A.ldx = L.ldx; A.pq = L.pq;
            A.rowstat = L.rowstat; A.bias = theta + L.off_b; A.relu = l < k - 1 ? 1 : 0; A.Hout = L.Hout; A.ldh = L.ldh;
            GRP_TRY(launch_gat_walk<GAT_FWD>(A, &g->csr_long, p.partials, st));
        }
        if (l < k - 1) GRP_TRY(launch_dropout(drop, l, g->l2g, n, L.fout, L.Hout, L.ldh, nullptr, 0, nullptr, 0, st));
        H = L.Hout; ldh = L.ldh; h_bf16 = 0;
    }
    // ---------------- loss
    const int C = m->dims[k];
    float* dZ = p.dZa;
    float* dZ_other = p.dZb;
    StepSums sums(p.base, (float*)p.base);
    GRP_TRY(launch_softmax_xent(si, C, p.L[k - 1].Hout, ldp4(C), labels, o->estimator == GRP_EST_NODE_LEVEL, nullptr, dZ, ldp4(C), stats, st, &sums));
    // ---------------- backward
    for (int l = k - 1; l >= 0; --l) {
        const GatLayer& L = p.L[l];
        const void* Hin = l == 0 ? X : (const void*)p.L[l - 1].Hout;
        const int64_t ldin = l == 0 ? m->dims[0] : p.L[l - 1].ldh;
        const int in_bf16 = l == 0 && m->feat_dtype == GRP_DTYPE_BF16;
        {
            ProfScope ps("gat_backward", st, 6.0 * g->nnz * L.fout, 8.0 * g->nnz + 16.0 * L.fout * n);
            GatWalk A{};
            A.ptr = g->rowptr; A.idx = g->col; A.n = n; A.F = L.fout; A.Tx = L.Tx; A.ldx = L.ldx; A.pq = L.pq;
            A.rowstat = L.rowstat; A.bias = theta + L.off_b; A.Hout = L.Hout; A.ldh = L.ldh; A.dOut = dZ; A.ldd = L.ldh;
            A.dst = p.dst; A.dq = p.dq; A.dTx = p.dTx; A.colsum = L.colsum;
            A.hout_scale = (drop.on && l < k - 1) ? 1.0f - o->dropout_rate : 1.f;
            GRP_TRY(launch_gat_walk<GAT_DST>(A, &g->csr_long, p.partials, st, &sums, L.dbias));
            A.ptr = g->colptr; A.idx = g->row;
            GRP_TRY(launch_gat_walk<GAT_SRC>(A, &g->csc_long, p.partials, st));
        }
        GemmTNArgs t;          // dW_ext = H_in^T dT_ext
        t.M = n; t.K = L.fin; t.N = (int)L.ldx; t.A = Hin; t.lda = ldin; t.a_bf16 = in_bf16; t.B = p.dTx; t.ldb = L.ldx;
        t.C = L.dWx; t.ldc = L.ldx; t.workspace = L.tn_ws; t.workspace_bytes = L.tn_ws_bytes; t.sums = &sums;
        GRP_TRY(launch_gemm_tn(t, st));
        if (l > 0) {
            GemmNNArgs c;      // dZ_prev = (H_in > 0) * (dT_ext W_ext^T)
            c.planes = p.planes; c.planes_bytes = p.planes_bytes;
            c.M = n; c.N = L.fin; c.K = (int)L.ldx; c.A = p.dTx; c.lda = L.ldx; c.Bt = L.Wp; c.ldbt = L.ldx;
            c.mask = p.L[l - 1].Hout; c.ld_mask = p.L[l - 1].ldh;
            c.C = dZ_other; c.ldc = p.L[l - 1].ldh; c.zero_pad_to = (int)p.L[l - 1].ldh;
            GRP_TRY(launch_gemm_nn(c, st));
        }
        float* sw = dZ; dZ = dZ_other; dZ_other = sw;
    }
    GRP_TRY(launch_step_sums(sums, st));
    for (const GatLayer& L : p.L) {
        ProfScope ps("gat_param_grad", st);
        hipLaunchKernelGGL(gat_param_grad_kernel, dim3((unsigned)L.fout), dim3(256), 0, st, (const float*)L.dWx, (const float*)L.dbias,
                               (int)L.ldx, theta + L.off_w, theta + L.off_as, theta + L.off_ad, L.fin, L.fout,
                               grad + L.off_w, grad + L.off_as, grad + L.off_ad, grad + L.off_b);
        GRP_LAUNCH_CHECK();
    }
    return GRP_OK;
}

}  // namespace grp
