// Dense feature transforms on the gfx950 matrix cores, in fp32 precision.
//
//   gemm_nn:  C[M x N] = epilogue(A[M x K] B[K x N] + A2[M x K2] B2[K2 x N])   (X W, dY W^T)
//   gemm_tn:  C[K x N] = A[M x K]^T B[M x N]                                   (X^T dY)
//
// M is the number of nodes (10^5..10^7); K and N are layer widths (<= a few hundred), so
// both products are tall-and-skinny: a workgroup owns a 128-row slab of nodes (nn) or a
// slice of the node dimension (tn, partial sums reduced afterwards in a fixed order, so
// the result does not depend on scheduling).
//
// Arithmetic.  The bf16 matrix instructions run at 16 times the rate of the fp32 ones, and an fp32 number is
// exactly the sum of three bf16 numbers: x = hi + mid + lo, hi = bf16(x), mid = bf16(x - hi) and lo = x - hi - mid, which
// has at most 7 significant bits (both differences are exact).  A product of two fp32 numbers is then nine bf16 products, each
// exact in fp32; all are computed but lo.lo, which is below 2^-34 of |a||b|.  An operand stored in bf16 is its own
// hi: three products, none left out.  The split is done by the thread that stages an element (5.5 instructions per element).
//   What the matrix unit does to a sum (measured on single instructions): it adds eight products and the accumulator at a time and rounds
// to nearest, but first cuts the products at 2^-24 of the largest one's power of two, towards zero, and their sum or the accumulator, whichever
// is smaller, towards minus infinity: a smaller accumulator at the same place, the sum 8 bits below a larger accumulator's last bit.
// So nothing is accumulated over k in the matrix unit: a 32-deep k-tile starts from zero, hi.hi in one accumulator and the
// seven small products, smallest first, in another (its cuts are 2^-8 of a last bit), and the two are added to each other and to the
// running sum in fp32.  A sum of one term is rounded once, a long one once per 32 terms.
//   Error against fp64, rms of the result, fp32 instructions -> here, normal deviates: K = 1 2.53e-8 -> 2.53e-8, K = 4 4.1e-8 -> 2.7e-8,
// K = 32 1.0e-7 -> 3.9e-8, K = 256 2.9e-7 -> 6.8e-8, K = 1024 5.7e-7 -> 1.1e-7; X^T dY over 10^6 rows, uniform operands 7.8e-8 -> 5.7e-8;
// mean relative error against equal weights of 1/3 up to 9e-9 -> 1.5e-9.  (Six products in one chain over all of k, as these kernels
// first had it: K = 1 4.3e-8, 10^6 uniform rows 3.3e-6, equal weights 2e-8.)
//   Operands below 2^-110 in size lose what lies below 2^-133, the smallest bf16.
//
// Loads and arithmetic overlap the same way everywhere: the next k-tile is requested from HBM into raw registers before
// the current one is multiplied and is only touched (split, masked, written to LDS) afterwards; addresses are clamped into the
// operand instead of branching.  The layouts are described at the kernels.  Products whose operands are not 16-byte
// friendly, or whose B is not given transposed, take gemm_nn_kernel, which uses the fp32 instructions.
#include "common.h"
#include "step_sums.h"

#include <algorithm>

#include <type_traits>

namespace grp {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BK = 32;      // k-tile depth
// Resident workgroups per CU that the kernels are built for: three of 168 registers, but two where the partial sums of a tile would
// not fit beside the rest and were spilled (NT, 128 columns with B split in the kernel: K = N = 256 over 3e5 rows 380 us with three,
// 338 with two; TN with two 32 x 32 tiles per wavefront: K = 256, N = 47 129 and 112 us, with four: 1127 and 323).
// Four of 128 where 64 columns of an fp32 product take hardly more (130 if left alone): steps on graphs of few edges, us with three and four: GCN 128-48-40
// over 1e5 rows 199 and 195, SAGE 100-64-64-47 over 3e5 910 and 903, GCN 256-64-64 over 2^20 2019 and 2014; 2e4 rows and fewer the same.
constexpr int nt_wgs(int TN, bool pre, bool lean = false) { return TN >= 8 && !pre ? 2 : TN == 4 && pre && lean ? 4 : 3; }
constexpr int tn_wgs(int tiles) { return tiles > 1 ? 2 : 3; }
constexpr int NT_PRE_SLABS = 512;      // products over fewer slabs of 128 rows whose B is not ready split it in the kernel (a launch for the planes costs 3 us)
constexpr int NXCD = 8;     // L2 domains; consecutive workgroup ids go round them

template <typename T> __device__ __forceinline__ float to_f(T v);
template <> __device__ __forceinline__ float to_f<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f<__hip_bfloat16>(__hip_bfloat16 v) { return __bfloat162float(v); }

// Four consecutive elements as raw bits (fp32: 16 bytes, bf16: 8 bytes in .x/.y).
template <typename T, bool ANY = false /* at any element boundary */>
__device__ __forceinline__ uint4 ldg_raw4(const T* __restrict__ p) {
    if constexpr (sizeof(T) == 4) {
        using V = typename std::conditional<ANY, u32x4_any, u32x4_al>::type;
        const V r = *reinterpret_cast<const V*>(p);
        return make_uint4(r.x, r.y, r.z, r.w);
    } else {
        using V = typename std::conditional<ANY, u32x2_any, u32x2_al>::type;
        const V r = *reinterpret_cast<const V*>(p);
        return make_uint4(r.x, r.y, 0u, 0u);
    }
}
__device__ __forceinline__ void unpack4(const uint4& r, bool bf16, float o[4]) {
    if (bf16) {
        o[0] = __uint_as_float(r.x << 16);
        o[1] = __uint_as_float(r.x & 0xFFFF0000u);
        o[2] = __uint_as_float(r.y << 16);
        o[3] = __uint_as_float(r.y & 0xFFFF0000u);
    } else {
        o[0] = __uint_as_float(r.x); o[1] = __uint_as_float(r.y);
        o[2] = __uint_as_float(r.z); o[3] = __uint_as_float(r.w);
    }
}

// Slow, always-safe element loads (rows of fewer than four columns without padding, B not given transposed).
template <typename T>
__device__ __forceinline__ uint4 ldg_safe4(const T* __restrict__ row, bool row_ok, int k, int K) {
    float o[4] = {0.f, 0.f, 0.f, 0.f};
    if (row_ok) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (k + q < K) o[q] = to_f<T>(row[k + q]);
    }
    return make_uint4(__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3]));
}

__device__ __forceinline__ int64_t lmin(int64_t a, int64_t b) { return a < b ? a : b; }

// ------------------------------------------------------------------------------- fp32 as three bf16 planes
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void split8(const float (&v)[8], uint4& hi, uint4& mid, uint4& lo) {
    split2(v[0], v[1], hi.x, mid.x, lo.x);
    split2(v[2], v[3], hi.y, mid.y, lo.y);
    split2(v[4], v[5], hi.z, mid.z, lo.z);
    split2(v[6], v[7], hi.w, mid.w, lo.w);
}
// Eight k values of one row into the three planes of a tile; `at` is their place in the first.
template <int PLANE>
__device__ __forceinline__ void put_split8(unsigned char* at, const float (&v)[8]) {
    uint4 hi, mid, lo;
    split8(v, hi, mid, lo);
    *reinterpret_cast<uint4*>(at) = hi;
    *reinterpret_cast<uint4*>(at + PLANE) = mid;
    *reinterpret_cast<uint4*>(at + 2 * PLANE) = lo;
}

__device__ __forceinline__ floatx4 mfma16(bf16x8 a, bf16x8 b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// Keeps the additions to an accumulator where they are written: left alone, the compiler moves them behind the tile's last
// barrier, and holds (and spills) the partial sums of every output tile until then.
template <typename V> __device__ __forceinline__ void pin(V& v) { asm volatile("" : "+v"(v)); }

// One 32-deep step of a wavefront's TM x TN block of 32x32 tiles.  as / bs + c0: this lane's eight of the first 16 k of its first
// tile row in the first plane; its eight of the other 16 k lie at c0 ^ 32.  sign: +1 or -1, of the tile.  MAYBE_ONE and one: A is a single
// plane (an operand stored in bf16).
template <int TM, int TN, int PLANE_A, int PLANE_B, bool MAYBE_ONE>
__device__ __forceinline__ void mma32(const unsigned char* as, const unsigned char* bs, int c0, bool one, float sign, floatx16 (&acc)[TM][TN]) {
    auto mul = [](bf16x8 a, bf16x8 b, floatx16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        bf16x8 a[3][2];
        auto get_a = [&](int p) {
#pragma unroll
            for (int h = 0; h < 2; ++h) a[p][h] = *reinterpret_cast<const bf16x8*>(as + (c0 ^ (32 * h)) + p * PLANE_A + i * 32 * 64);
        };
        get_a(0);
        if (!MAYBE_ONE || !one) { get_a(1); get_a(2); }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            bf16x8 b[3][2];
#pragma unroll
            for (int p = 2; p >= 0; --p)
#pragma unroll
                for (int h = 0; h < 2; ++h) b[p][h] = *reinterpret_cast<const bf16x8*>(bs + (c0 ^ (32 * h)) + p * PLANE_B + j * 32 * 64);
            floatx16 t;
#pragma unroll
            for (int r = 0; r < 16; ++r) t[r] = 0.f;
            auto both = [&](int pa, int pb) {
#pragma unroll
                for (int h = 0; h < 2; ++h) t = mul(a[pa][h], b[pb][h], t);
            };
            if (!MAYBE_ONE || !one) {                     // small products first
                both(1, 2);
                both(2, 1);
                both(0, 2);
                both(2, 0);
                both(1, 1);
                both(0, 1);
                both(1, 0);
            } else {
                both(0, 2);
                both(0, 1);
            }
            floatx16 top;
#pragma unroll
            for (int r = 0; r < 16; ++r) top[r] = 0.f;
#pragma unroll
            for (int h = 0; h < 2; ++h) top = mul(a[0][h], b[0][h], top);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = fmaf(t[r] + top[r], sign, acc[i][j][r]);
            pin(acc[i][j]);
        }
    }
}

// One BKT-deep step of the wavefront's TM x TN block from k-major LDS tiles.  The operands of
// the next k-pair are read from LDS before the matrix instructions of the current one are
// issued, so the LDS latency hides behind them.
template <int TM, int TN, int PA, int PB, int BKT>
__device__ __forceinline__ void mma_step(const float* __restrict__ As, const float* __restrict__ Bs, int a_off,
                                         int b_off, floatx16 (&acc)[TM][TN]) {
    const int lane = threadIdx.x & 63;
    const int li = lane & 31, lk = lane >> 5;
    const float* ap = As + lk * PA + a_off + li;
    const float* bp = Bs + lk * PB + b_off + li;
    float a[2][TM], b[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) a[0][i] = ap[32 * i];
#pragma unroll
    for (int j = 0; j < TN; ++j) b[0][j] = bp[32 * j];
#pragma unroll
    for (int k = 0; k < BKT; k += 2) {
        const int cur = (k >> 1) & 1, nxt = cur ^ 1;
        if (k + 2 < BKT) {
#pragma unroll
            for (int i = 0; i < TM; ++i) a[nxt][i] = ap[(k + 2) * PA + 32 * i];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[nxt][j] = bp[(k + 2) * PB + 32 * j];
        }
        __builtin_amdgcn_sched_barrier(0);    // keep the next operands' LDS reads ahead of these MFMAs
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][i], b[cur][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Epilogue shared by the nn kernels: (+ addend) (+ bias) -> C_raw; (* rowscale) (ReLU) (mask) -> C.
// When every operand allows 16-byte accesses the accumulators go through LDS, 32 tile rows
// per wavefront row at a time, so that addend / mask are read and the results written as
// whole 16-byte vectors along rows (one 512-byte run per 32 lanes).  `lds` must hold
// WM*32*(BN+4) floats and must no longer be read by the main loop.
template <bool VEC, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void nn_epilogue(const GemmNNArgs& g, floatx16 (&acc)[TM][TN], float* lds, int64_t m0, int n0,
                                            int n_store) {
    constexpr int BN = WN * TN * 32;
    constexpr int PC = BN + 4;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WN, wn = wave % WN;
    const int li = lane & 31, lk = lane >> 5;
    // Epilogue.  When every operand allows 16-byte accesses the accumulators go through LDS,
    // 32 tile rows per wavefront row at a time, so that bias / addend / mask are read and the
    // results written as whole 16-byte vectors along rows (one 512-byte run per 32 lanes).
    const bool vec_epi = VEC && (n_store % 4 == 0) && g.ldc % 4 == 0 && ((uintptr_t)g.C % 16) == 0 &&
                         (!g.addend || (g.ld_add % 4 == 0 && ((uintptr_t)g.addend % 16) == 0)) &&
                         (!g.mask || (g.ld_mask % 4 == 0 && ((uintptr_t)g.mask % 16) == 0)) &&
                         (!g.C_raw || (g.ld_raw % 4 == 0 && ((uintptr_t)g.C_raw % 16) == 0));
    const int bias_n = g.bias_n > 0 ? g.bias_n : g.N - g.bias_col0;
    const int rs_cols = g.rowscale_cols > 0 ? g.rowscale_cols : g.N;   // a multiple of 4 when set
    if (vec_epi) {
        float* Cs = lds;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (i > 0) __syncthreads();               // the previous pass has been read out
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    Cs[(wm * 32 + 8 * (r / 4) + 4 * lk + (r % 4)) * PC + (wn * TN + j) * 32 + li] = acc[i][j][r];
            __syncthreads();
            constexpr int C4 = BN / 4;                // 16-byte columns per tile row
            for (int f = tid; f < WM * 32 * C4; f += 256) {
                const int lr = f / C4, c4 = f % C4;
                const int col = n0 + 4 * c4;
                const int64_t m = m0 + ((lr >> 5) * TM + i) * 32 + (lr & 31);
                if (m >= g.M || col >= n_store) continue;
                const float4 a4 = *reinterpret_cast<const float4*>(&Cs[lr * PC + 4 * c4]);
                float v[4] = {a4.x, a4.y, a4.z, a4.w};
                if (g.addend) {
                    const float4 t = *reinterpret_cast<const float4*>(g.addend + m * g.ld_add + col);
                    v[0] += t.x; v[1] += t.y; v[2] += t.z; v[3] += t.w;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int cb = col + q - g.bias_col0;
                    if (col + q < g.N) { if (g.bias && cb >= 0 && cb < bias_n) v[q] += g.bias[cb]; }
                    else v[q] = 0.f;
                }
                if (g.C_raw) *reinterpret_cast<float4*>(g.C_raw + m * g.ld_raw + col) = make_float4(v[0], v[1], v[2], v[3]);
                const float rs = (g.rowscale && col < rs_cols) ? g.rowscale[m] : 1.f;
                float4 mk = make_float4(1.f, 1.f, 1.f, 1.f);
                if (g.mask) mk = *reinterpret_cast<const float4*>(g.mask + m * g.ld_mask + col);
                const float mv[4] = {mk.x, mk.y, mk.z, mk.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float t = v[q] * rs;
                    if (g.relu) t = t > 0.f ? t : 0.f;
                    if (g.mask) t = mv[q] > 0.f ? t : 0.f;
                    v[q] = col + q < g.N ? t : 0.f;
                }
                *reinterpret_cast<float4*>(g.C + m * g.ldc + col) = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + (wn * TN + j) * 32 + li;
            if (col >= n_store) continue;
            const int cb = col - g.bias_col0;
            const float bv = (g.bias && col < g.N && cb >= 0 && cb < bias_n) ? g.bias[cb] : 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t m = m0 + (wm * TM + i) * 32 + 8 * (r / 4) + 4 * lk + (r % 4);
                if (m >= g.M) continue;
                float v = 0.f;
                if (col < g.N) {
                    v = acc[i][j][r] + bv;
                    if (g.addend) v += g.addend[m * g.ld_add + col];
                }
                if (g.C_raw) g.C_raw[m * g.ld_raw + col] = v;
                if (col < g.N) {
                    if (g.rowscale && col < rs_cols) v *= g.rowscale[m];
                    if (g.relu) v = v > 0.f ? v : 0.f;
                    if (g.mask) v = g.mask[m * g.ld_mask + col] > 0.f ? v : 0.f;
                }
                g.C[m * g.ldc + col] = v;
            }
        }
}

// ------------------------------------------------------------------------------- NN
template <typename AT, bool VEC, int WM, int WN, int TM, int TN, int BK, int NBUF>
__global__ __launch_bounds__(256) void gemm_nn_kernel(GemmNNArgs g) {
    if (g.M_dev) {                                    // the launch was sized by upper bounds
        g.M = *g.M_dev;
        if (g.a_valid_rows_dev) g.a_valid_rows = *g.a_valid_rows_dev;
    }
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    constexpr int PA = BM + 2, PB = BN + 4;          // PA = 2 mod 8 spreads the transposing writes
    constexpr int A_REPS = BM * BK / 4 / 256;        // 4-element loads per thread for the A tile
    constexpr int B_REPS = (BN * BK / 4 + 255) / 256;
    constexpr bool A_BF16 = sizeof(AT) == 2;
    static_assert(BM * BK / 4 % 256 == 0, "A tile must fill the workgroup");
    constexpr int PC = BN + 4;                        // pitch of the staged output tile
    constexpr int A_FLOATS = ((BK * PA + 3) / 4) * 4; // keeps the B tiles 16-byte aligned
    constexpr int MAIN_FLOATS = NBUF * (A_FLOATS + BK * PB);
    constexpr int EPI_FLOATS = WM * 32 * PC;
    constexpr int LDS_FLOATS = MAIN_FLOATS > EPI_FLOATS ? MAIN_FLOATS : EPI_FLOATS;
    __shared__ __attribute__((aligned(16))) float lds[LDS_FLOATS];
    float* const As0 = lds;
    float* const Bs0 = lds + NBUF * A_FLOATS;

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WN, wn = wave % WN;
    const int n_store = g.zero_pad_to > g.N ? g.zero_pad_to : g.N;
    const int n_tiles = (n_store + BN - 1) / BN;
    // Workgroup ids go round the NXCD L2 domains; the column tiles of one row slab get ids
    // that differ by NXCD, so they run on the same domain and the slab's second read hits L2.
    const int64_t hq = blockIdx.x / NXCD;
    const int64_t slab = (hq / n_tiles) * NXCD + blockIdx.x % NXCD;
    const int64_t m0 = slab * BM;
    const int n0 = (int)(hq % n_tiles) * BN;
    if (m0 >= g.M) return;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const int nk1 = (g.K + BK - 1) / BK;
    const int nk2 = (g.K2 + BK - 1) / BK;
    const int nk = nk1 + nk2;
    const int npad = (g.N + 3) & ~3;

    uint4 ra[A_REPS], rb[B_REPS];

    // rows of the first product's A: optional indirection and a limit on the valid rows
    const int64_t a_valid = g.a_valid_rows > 0 ? g.a_valid_rows : g.M;
    int64_t arow[A_REPS];
#pragma unroll
    for (int r = 0; r < A_REPS; ++r) {
        const int64_t gm = lmin(m0 + (tid + 256 * r) / (BK / 4), a_valid - 1);
        arow[r] = g.a_rows ? (int64_t)g.a_rows[gm] : gm;
    }

    auto fetch = [&](int kt) {
        const bool second = kt >= nk1;
        const int k0 = (second ? kt - nk1 : kt) * BK;
        const int Kc = second ? g.K2 : g.K;
        const int kpad = (Kc + 3) & ~3;
        const float* Bp = second ? g.B2 : g.B;
        const int64_t ldb = second ? g.ldb2 : g.ldb;
#pragma unroll
        for (int r = 0; r < A_REPS; ++r) {
            const int f = tid + 256 * r;                 // 4-element slot in the BM x BK tile
            const int m = f / (BK / 4), kq = f % (BK / 4);
            if constexpr (VEC) {
                const int64_t gm = lmin(m0 + m, g.M - 1);
                const int kk = imin(k0 + 4 * kq, kpad - 4);
                ra[r] = second ? ldg_raw4<float>(g.A2 + gm * g.lda2 + kk)
                               : ldg_raw4<AT>((const AT*)g.A + arow[r] * g.lda + kk);
            } else {
                const int64_t gm = m0 + m;
                const bool ok2 = gm < g.M, ok1 = gm < a_valid;
                ra[r] = second ? ldg_safe4<float>(g.A2 + (ok2 ? gm : 0) * g.lda2, ok2, k0 + 4 * kq, Kc)
                               : ldg_safe4<AT>((const AT*)g.A + arow[r] * g.lda, ok1, k0 + 4 * kq, Kc);
            }
        }
#pragma unroll
        for (int r = 0; r < B_REPS; ++r) {
            const int f = tid + 256 * r;
            const int k = f / (BN / 4), nq = f % (BN / 4);
            if (BN * BK / 4 % 256 != 0 && f >= BN * BK / 4) { rb[r] = make_uint4(0u, 0u, 0u, 0u); continue; }
            if constexpr (VEC) {
                const int kb = imin(k0 + k, Kc - 1);
                const int nc = imin(n0 + 4 * nq, npad - 4);
                rb[r] = ldg_raw4<float>(Bp + (int64_t)kb * ldb + nc);
            } else if (g.Bt) {                           // B given transposed: element (k, n) is Bt[n][k]
                const float* Btp = second ? g.Bt2 : g.Bt;
                const int64_t ldbt = second ? g.ldbt2 : g.ldbt;
                float o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = n0 + 4 * nq + q;
                    o[q] = (k0 + k < Kc && n < g.N) ? Btp[(int64_t)n * ldbt + k0 + k] : 0.f;
                }
                rb[r] = make_uint4(__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3]));
            } else {
                const bool ok = k0 + k < Kc;
                rb[r] = ldg_safe4<float>(Bp + (int64_t)(ok ? k0 + k : 0) * ldb, ok, n0 + 4 * nq, g.N);
            }
        }
    };
    auto stage = [&](int kt) {
        const bool second = kt >= nk1;
        const int k0 = (second ? kt - nk1 : kt) * BK;
        const int Kc = second ? g.K2 : g.K;
        float* As = As0 + (NBUF == 1 ? 0 : (kt & 1)) * A_FLOATS;
        float* Bs = Bs0 + (NBUF == 1 ? 0 : (kt & 1)) * (BK * PB);
#pragma unroll
        for (int r = 0; r < A_REPS; ++r) {
            const int f = tid + 256 * r;
            const int m = f / (BK / 4), kq = f % (BK / 4);
            float v[4];
            unpack4(ra[r], VEC && A_BF16 && !second, v);
            const bool row_ok = m0 + m < (second ? g.M : a_valid);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                As[(4 * kq + q) * PA + m] = (!VEC || (row_ok && k0 + 4 * kq + q < Kc)) ? v[q] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < B_REPS; ++r) {
            const int f = tid + 256 * r;
            const int k = f / (BN / 4), nq = f % (BN / 4);
            if (BN * BK / 4 % 256 != 0 && f >= BN * BK / 4) continue;
            float v[4];
            unpack4(rb[r], false, v);
            const bool k_ok = k0 + k < Kc;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (VEC && !(k_ok && n0 + 4 * nq + q < g.N)) v[q] = 0.f;
            *reinterpret_cast<float4*>(&Bs[k * PB + 4 * nq]) = make_float4(v[0], v[1], v[2], v[3]);
        }
    };

    fetch(0);
    stage(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) fetch(kt + 1);
        mma_step<TM, TN, PA, PB, BK>(As0 + (NBUF == 1 ? 0 : (kt & 1)) * A_FLOATS,
                                     Bs0 + (NBUF == 1 ? 0 : (kt & 1)) * (BK * PB), wm * TM * 32, wn * TN * 32, acc);
        if (NBUF == 1) __syncthreads();
        if (kt + 1 < nk) stage(kt + 1);
        __syncthreads();
    }

    nn_epilogue<VEC, WM, WN, TM, TN>(g, acc, lds, m0, n0, n_store);
}

// ------------------------------------------------------------------------------- NT (fast path of nn)
// Same product as gemm_nn with B supplied transposed (Bt[N x K], k contiguous), which is how
// the step keeps its weight matrices.
//
// A wavefront owns 16*TM rows of C and all BN = 16*TN columns of the workgroup's tile.  Its rows of A go from memory to
// its registers and are split there: no other wavefront needs them, so they never pass through LDS.  Only B does (three
// planes, double-buffered, one barrier per 32-deep k-tile).  v_mfma_f32_16x16x32_bf16 is used with B as its first operand:
// lane l supplies eight k of column n = l%16 of the tile (B) and of row m = l%16 (A), and its four accumulator registers
// are C[m = l%16][n = 4*(l/16) .. +3], so that results leave as 16-byte vectors along rows and the epilogue reads its operands the
// same way, without LDS.  Which eight k a lane takes is free as long as both operands agree: lane group q = l/16 takes
// the four from 4*q and the four from 16 + 4*q, so that one load instruction covers 64 consecutive bytes of a row.
// LDS rows hold 32 k (64 bytes, 4 places of 16); group q of row r sits at place q ^ ((r >> 1) & 3): the reads of eight
// consecutive rows fall in distinct banks.
// Loads use a uniform base that advances along k plus 32-bit per-thread offsets fixed before the loop; rows past the end of
// an operand are clamped to its last row (their products are not stored); only the last, ragged k-tile of a product
// is masked.
// IRREG selects the variant with gathered (a_rows), limited (a_valid_rows) or tightly packed (a_tight) A rows.
// PRE: B comes as planes (g.ready: of a step's weights by the launch that re-packs them, else split_b_kernel below) whose 1 KB runs are copied from memory to LDS without passing
// through registers.  The loop is bound by issue: matrix and vector instructions of a SIMD's wavefronts add up (N = 512, K = 256: per
// k-tile 128 of the former of 16 cycles and 350 of the latter of 4, 2048 + 1400 cycles; 3360 measured), and the split of B, which
// every slab of 128 rows does again otherwise, would add to the latter and to the registers.  With and without, in us: the four 128-wide
// products of a SAGE step on 3e5 rows 1652 and 1997, those of a residual GCN-8 step on 2^20 rows 14.1 and 16.5 ms, a bf16 one over
// 8.4e6 rows (K = 64 + 64) 2.74 and 3.30 ms.  Products of few rows, whose every workgroup would split all of B for 64 rows: K = 256 + 256, N = 172 ..
// 256 over 1e3 .. 1e4 rows 15.0 -> 13.2, gathered bf16 K = 128 + 128 over 2e4 37 -> 35, K = 130 over 1e5 a ragged step 612 -> 594.
// One element of the product, added up in plain fp32 along k (up to the first NaN: a diverged step has them everywhere).
template <typename AT>
__device__ __forceinline__ float nt_plain(const GemmNNArgs& g, int64_t m, int n) {
    const bool zero = g.a_valid_rows > 0 && m >= g.a_valid_rows;       // (such rows of the first A read as zero)
    const AT* const a = (const AT*)g.A + (zero ? 0 : (g.a_rows ? (int64_t)g.a_rows[m] : m) * g.lda);
    const float* const b = g.Bt + (int64_t)n * g.ldbt;
    float s = 0.f;
    for (int k = 0; k < g.K && !isnan(s); ++k) s = fmaf(zero ? 0.f : to_f<AT>(a[k]), b[k], s);
    const float* const a2 = g.A2 + m * g.lda2;
    const float* const b2 = g.Bt2 + (int64_t)n * g.ldbt2;
    for (int k = 0; k < g.K2 && !isnan(s); ++k) s = fmaf(a2[k], b2[k], s);
    return s;
}

template <typename AT, int TM, int TN, bool IRREG, bool PRE>
__device__ __forceinline__ void gemm_nt_kernel_body(unsigned gx, GemmNNArgs g) {
    if (g.M_dev) {                                    // the launch was sized by upper bounds
        g.M = *g.M_dev;
        if (g.a_valid_rows_dev) g.a_valid_rows = *g.a_valid_rows_dev;
    }
    constexpr int BM = 4 * TM * 16, BN = TN * 16;
    constexpr int PLANE = BN * 64;
    constexpr int B_REPS = (BN + 63) / 64;            // a pass of the workgroup covers 64 rows of Bt
    constexpr bool A_BF16 = sizeof(AT) == 2;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * 3 * PLANE];

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int li = lane & 15, lq = lane >> 4;
    const int n_store = g.zero_pad_to > g.N ? g.zero_pad_to : g.N;
    const int n_tiles = (n_store + BN - 1) / BN;
    // Workgroup ids go round the NXCD L2 domains; the column tiles of one row slab get ids
    // that differ by NXCD, so they run on the same domain and the slab's second read hits L2.
    const int64_t hq = blockIdx.x / NXCD;
    const int64_t slab = (hq / n_tiles) * NXCD + blockIdx.x % NXCD;
    const int64_t m0 = slab * BM;
    const int n0 = (int)(hq % n_tiles) * BN;
    if (m0 >= g.M) return;

    floatx4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // Offsets of this lane's A rows (its first four k included).  Regular variant: 32-bit offsets from the slab's
    // first row; irregular variant: 64-bit offsets from the operand base.
    const int rows_here = (int)lmin((int64_t)BM, g.M - m0);
    using aoff_t = typename std::conditional<IRREG, int64_t, uint32_t>::type;
    aoff_t aoff[TM];
    uint32_t aoff2[TM];
    bool a_zero[TM];
    // Rows of A without room for a whole last group are read up to their last element instead: that group is read a_turn
    // elements early and turned into place before it is masked.  (The base is moved back and the offsets forward by as much:
    // the early group may start before the k-tile, and an unsigned offset from the tile's start could not say so.)
    const int a_turn = IRREG && g.a_tight ? -g.K & 3 : 0;
    const AT* a_base = (const AT*)g.A - a_turn;
    if (!IRREG) a_base += m0 * g.lda;
    const float* const a2_base = g.A2 + m0 * g.lda2;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int lr = imin(wave * 16 * TM + 16 * i + li, rows_here - 1);
        if (IRREG) {
            const int64_t a_valid = g.a_valid_rows > 0 ? g.a_valid_rows : g.M;
            const int64_t r1 = lmin(m0 + lr, a_valid - 1);
            aoff[i] = (aoff_t)((g.a_rows ? (int64_t)g.a_rows[r1] : r1) * g.lda + 4 * lq + a_turn);
            a_zero[i] = m0 + lr >= a_valid;
        } else {
            aoff[i] = (aoff_t)((uint32_t)lr * (uint32_t)g.lda + 4 * lq);
            a_zero[i] = false;
        }
        aoff2[i] = (uint32_t)lr * (uint32_t)g.lda2 + 4 * lq;
    }
    // This thread's part of the B tile: k group tq of rows trow, trow + 64.
    const int tq = tid & 3, trow = tid >> 2;
    uint32_t boff[B_REPS], boff2[B_REPS];
#pragma unroll
    for (int r = 0; r < B_REPS; ++r) {
        const uint32_t nc = imin(n0 + trow + 64 * r, g.N - 1);
        boff[r] = nc * (uint32_t)g.ldbt + 4 * tq;
        boff2[r] = nc * (uint32_t)g.ldbt2 + 4 * tq;
    }
    const int nk1 = (g.K + BK - 1) / BK;
    const int nk = nk1 + (g.K2 + BK - 1) / BK;
    uint4 ra[TM][2], rb[B_REPS][2];

    // a ragged last tile reads the operand's last four-element group again (masked afterwards); in A that group may lie a_turn
    // elements early (below)
    auto clamp = [&](int k0, int Kc, int q, int turn, int& d0, int& d1) {
        d0 = 0; d1 = 16;
        if (k0 + BK > Kc) {
            const int last = ((Kc + 3) & ~3) - 4 - turn - k0 - 4 * q;
            d0 = imin(0, last);
            d1 = imin(16, last);
        }
    };
    // PRE: tile kt of B into its half of the LDS; a wavefront's copy is 64 consecutive units of 16 bytes on both sides
    const uint32_t lds_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
    const int swave = __builtin_amdgcn_readfirstlane(wave);
    auto copy_b = [&](int kt) {
        constexpr int RUNS = 3 * BN / 16, PER_PLANE = BN / 16;
        const unsigned char* const tile = (kt < nk1 ? g.ready : g.ready2) + (int64_t)(kt < nk1 ? kt : kt - nk1) * 3 * g.ready_rows * 64;
#pragma unroll
        for (int r = 0; r < (RUNS + 3) / 4; ++r) {
            const int c = swave + 4 * r;
            if (RUNS % 4 != 0 && c >= RUNS) break;
            const unsigned char* const from = tile + ((int64_t)(c / PER_PLANE) * g.ready_rows + n0 + 16 * (c % PER_PLANE)) * 64;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(lds_at + (kt & 1) * 3 * PLANE + c * 1024), "v"(lane * 16), "s"(from) : "memory", "m0");
        }
    };
    auto fetch = [&](int kt) {
        const bool second = kt >= nk1;
        const int k0 = (second ? kt - nk1 : kt) * BK;
        const int Kc = second ? g.K2 : g.K;
        int d0, d1, e0, e1;
        clamp(k0, Kc, lq, second ? 0 : a_turn, d0, d1);
        if (!PRE) clamp(k0, Kc, tq, 0, e0, e1);
        if (second) {
            const float* pa = a2_base + k0;
            const float* pb = g.Bt2 + k0;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                ra[i][0] = ldg_raw4<float>(pa + (aoff2[i] + d0));
                ra[i][1] = ldg_raw4<float>(pa + (aoff2[i] + d1));
            }
#pragma unroll
            for (int r = 0; !PRE && r < B_REPS; ++r) {
                rb[r][0] = ldg_raw4<float>(pb + (boff2[r] + e0));
                rb[r][1] = ldg_raw4<float>(pb + (boff2[r] + e1));
            }
        } else {
            const AT* pa = a_base + k0;
            const float* pb = g.Bt + k0;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                ra[i][0] = ldg_raw4<AT, IRREG>(pa + (aoff[i] + d0));
                ra[i][1] = ldg_raw4<AT, IRREG>(pa + (aoff[i] + d1));
            }
#pragma unroll
            for (int r = 0; !PRE && r < B_REPS; ++r) {
                rb[r][0] = ldg_raw4<float>(pb + (boff[r] + e0));
                rb[r][1] = ldg_raw4<float>(pb + (boff[r] + e1));
            }
        }
    };
    // eight values of k group q as floats, zero where the k does not exist
    auto floats = [&](const uint4 (&r)[2], int left /*k values of the tile that exist*/, int q, int turn, float (&v)[8]) {
        unpack4(r[0], false, *reinterpret_cast<float(*)[4]>(&v[0]));
        unpack4(r[1], false, *reinterpret_cast<float(*)[4]>(&v[4]));
        if (left < BK) {
            if (turn) {                               // (uniform) only the group that `left` cuts is kept in part
                const int at = left & ~3;             // its first k within the tile
#pragma unroll
                for (int h = 0; h < 8; h += 4) {
                    if (4 * q + (h ? 16 : 0) != at) continue;
                    const float x = v[h + 1], y = v[h + 2], z = v[h + 3];
                    v[h] = turn == 1 ? x : turn == 2 ? y : z;
                    v[h + 1] = turn == 1 ? y : z;
                    v[h + 2] = z;
                }
            }
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = 4 * q + (t & 3) + (t >= 4 ? 16 : 0) < left ? v[t] : 0.f;
        }
    };
    auto left_of = [&](int kt) { return kt >= nk1 ? g.K2 - (kt - nk1) * BK : g.K - kt * BK; };
    unsigned char* const bput = lds + 64 * trow + 16 * (tq ^ ((trow >> 1) & 3));
    auto stage_b = [&](int kt) {
        const int left = left_of(kt);
#pragma unroll
        for (int r = 0; r < B_REPS; ++r) {
            float v[8];
            floats(rb[r], left, tq, 0, v);
            if (BN % 64 == 0 || trow + 64 * r < BN) put_split8<PLANE>(bput + (kt & 1) * 3 * PLANE + 64 * 64 * r, v);
        }
    };
    // What the matrix unit cuts off has always the same sign.  It is nothing beside the rounding of one result, but a bias gradient adds
    // up the results of 10^5..10^7 rows: every other 16 rows are multiplied as -A, and their sums subtracted.
    auto odd_rows = [&](int i) { return ((wave * TM + i) & 1) != 0; };
    const float turned = (wave & 1) ? -1.f : 1.f;     // (TM = 1)
    bf16x8 a[TM][3];
    auto split_a = [&](int kt) {
        const int left = left_of(kt);
        const bool second = kt >= nk1;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const bool zero = IRREG && !second && a_zero[i];
            if (A_BF16 && !second) {
                uint4 w = make_uint4(ra[i][0].x, ra[i][0].y, ra[i][1].x, ra[i][1].y);
                if (left < BK && a_turn) {            // two packed pairs: shifted as one 64-bit word
                    auto turned = [&](uint32_t lo, uint32_t hi) { return (((uint64_t)hi << 32) | lo) >> (16 * a_turn); };
                    const uint64_t t0 = turned(w.x, w.y), t1 = turned(w.z, w.w);
                    if (4 * lq == (left & ~3)) { w.x = (uint32_t)t0; w.y = (uint32_t)(t0 >> 32); }
                    if (4 * lq + 16 == (left & ~3)) { w.z = (uint32_t)t1; w.w = (uint32_t)(t1 >> 32); }
                }
                if (left < BK || zero) {
                    const int have = zero ? -64 : left - 4 * lq;
                    auto keep = [&](uint32_t x, int q) { return have >= q + 2 ? x : have == q + 1 ? x & 0xFFFFu : 0u; };
                    w = make_uint4(keep(w.x, 0), keep(w.y, 2), keep(w.z, 16), keep(w.w, 18));
                }
                if (odd_rows(i)) w = make_uint4(w.x ^ 0x80008000u, w.y ^ 0x80008000u, w.z ^ 0x80008000u, w.w ^ 0x80008000u);
                a[i][0] = a[i][1] = a[i][2] = __builtin_bit_cast(bf16x8, w);
            } else {
                float v[8];
                floats(ra[i], left, lq, second ? 0 : a_turn, v);
                if (zero) {
#pragma unroll
                    for (int t = 0; t < 8; ++t) v[t] = 0.f;
                }
                if (TM % 2 != 0) {
                    const uint32_t sign = (uint32_t)(wave & 1) << 31;
#pragma unroll
                    for (int t = 0; t < 8; ++t) v[t] = __uint_as_float(__float_as_uint(v[t]) ^ sign);
                } else if (odd_rows(i)) {
#pragma unroll
                    for (int t = 0; t < 8; ++t) v[t] = -v[t];
                }
                uint4 hi, mid, lo;
                split8(v, hi, mid, lo);
                a[i][0] = __builtin_bit_cast(bf16x8, hi);
                a[i][1] = __builtin_bit_cast(bf16x8, mid);
                a[i][2] = __builtin_bit_cast(bf16x8, lo);
            }
        }
    };
    const unsigned char* const bget = lds + 64 * li + 16 * (lq ^ ((li >> 1) & 3));
    auto mma = [&](int kt) {
        const unsigned char* const bp = bget + (kt & 1) * 3 * PLANE;
        const bool one = A_BF16 && kt < nk1;
        // A wavefront of two row tiles multiplies a column tile at a time: two chains of dependent instructions.  Of one row tile it takes
        // all its column tiles together, since such products run with one wavefront per SIMD, that waits for its chains alone: what bounds
        // them is the instructions of an iteration (64 rows, N = 64: a k-tile 1.02 -> 0.91 us, most of it the one sign per wavefront that
        // took both branches before; requesting k-tiles further ahead changed nothing).
        constexpr int J = TM == 1 ? TN : 1;
        bf16x8 b[J == 1 ? 2 : 1][J][3];
        auto get = [&](int j0) {
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    b[J == 1 ? j0 & 1 : 0][j][p] = *reinterpret_cast<const bf16x8*>(bp + p * PLANE + (j0 + j) * 16 * 64);
        };
        get(0);
#pragma unroll
        for (int j0 = 0; j0 < TN; j0 += J) {
            if (j0 + J < TN) get(j0 + J);             // a column tile ahead: the LDS latency hides behind the products
            __builtin_amdgcn_sched_barrier(0);
            auto& bj = b[J == 1 ? j0 & 1 : 0];
            floatx4 t[TM][J], top[TM][J];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < J; ++j) t[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            auto mul = [&](int pb, int pa) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < J; ++j) t[i][j] = mfma16(bj[j][pb], a[i][pa], t[i][j]);
            };
            if (!one) {                               // small products first
                mul(2, 1);
                mul(1, 2);
                mul(2, 0);
                mul(0, 2);
                mul(1, 1);
                mul(1, 0);
                mul(0, 1);
            } else {
                mul(2, 0);
                mul(1, 0);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < J; ++j) top[i][j] = mfma16(bj[j][0], a[i][0], floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const floatx4 sum = t[i][j] + top[i][j];
                    if (TM % 2 == 0) acc[i][j0 + j] = odd_rows(i) ? acc[i][j0 + j] - sum : acc[i][j0 + j] + sum;
                    else {                            // (not known when compiled; a sum times +1 or -1 is added with one rounding as well)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[i][j0 + j][q] = fmaf(sum[q], turned, acc[i][j0 + j][q]);
                    }
                    pin(acc[i][j0 + j]);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    fetch(0);
    if constexpr (PRE) {
        copy_b(0);
        for (int kt = 0; kt < nk; ++kt) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wavefront's part of tile kt is in LDS (and its rows of A here)
            split_a(kt);
            if (kt + 1 < nk) fetch(kt + 1);
            __syncthreads();                          // so is everybody's; everybody is done with tile kt - 1
            if (kt + 1 < nk) copy_b(kt + 1);
            mma(kt);
        }
    } else {
        stage_b(0);
        for (int kt = 0; kt < nk; ++kt) {
            split_a(kt);
            if (kt + 1 < nk) fetch(kt + 1);
            __syncthreads();                          // tile kt is written; everybody is done with tile kt - 1
            mma(kt);
            if (kt + 1 < nk) stage_b(kt + 1);
        }
    }

    // An infinity has no planes (x - hi is NaN), and a sum of planes may pass the largest float where the sum of the
    // products does not.  Both show as results that are not finite: those are added up again in plain fp32.
    float odd[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) odd[q] = fmaf(acc[i][j][q], 0.f, odd[q]);
    if (!((odd[0] + odd[1]) + (odd[2] + odd[3]) == 0.f)) {
#pragma unroll 1
        for (int e = 0; e < TM * TN * 4; ++e) {
            const int m_at = wave * 16 * TM + 16 * (e / (4 * TN)) + li, n_at = n0 + 16 * (e / 4 % TN) + 4 * lq + e % 4;
            auto each = [&](auto f) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[i][j][q] = f((i * TN + j) * 4 + q, acc[i][j][q]);
            };
            float v = 0.f;
            each([&](int at, float x) { v = at == e ? x : v; return x; });
            if (isfinite(v) || m_at >= rows_here || n_at >= g.N) continue;
            v = nt_plain<AT>(g, m0 + m_at, n_at);
            each([&](int at, float x) { return at == e ? v : x; });
        }
    }

    // ---- epilogue: (+ addend) (+ bias) -> C_raw; (* rowscale) (ReLU) (mask) -> C
    const int bias_n = g.bias_n > 0 ? g.bias_n : g.N - g.bias_col0;
    const int rs_cols = g.rowscale_cols > 0 ? g.rowscale_cols : g.N;
    const bool vec = n_store % 4 == 0 && g.ldc % 4 == 0 && ((uintptr_t)g.C % 16) == 0 &&
                     (!g.addend || (g.ld_add % 4 == 0 && ((uintptr_t)g.addend % 16) == 0)) &&
                     (!g.mask || (g.ld_mask % 4 == 0 && ((uintptr_t)g.mask % 16) == 0)) &&
                     (!g.C_raw || (g.ld_raw % 4 == 0 && ((uintptr_t)g.C_raw % 16) == 0));
    // columns [n0, n0 + BN) all exist and lie on one side of the bias' and the row scale's ranges
    const bool bias_in = g.bias && n0 >= g.bias_col0 && n0 + BN <= g.bias_col0 + bias_n && g.bias_col0 % 4 == 0 && ((uintptr_t)g.bias % 16) == 0;
    const bool bias_out = !g.bias || n0 + BN <= g.bias_col0 || n0 >= g.bias_col0 + bias_n;
    const bool rs_in = g.rowscale && n0 + BN <= rs_cols;
    const bool rs_out = !g.rowscale || n0 >= rs_cols;
    const bool lean = vec && n0 + BN <= g.N && (bias_in || bias_out) && (rs_in || rs_out);
    constexpr bool COLS = PRE && !IRREG && !A_BF16;
    const bool cols = COLS && g.col_part;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int lr = wave * 16 * TM + 16 * i + li;
        if (lr >= rows_here) {
#pragma unroll
            for (int j = 0; COLS && j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            continue;
        }
        const int64_t m = m0 + lr;
        const float cm = cols ? g.col_mul[m] : 0.f;
        const int nl = n0 + 4 * lq;
        const float rs = g.rowscale ? g.rowscale[m] : 1.f;
        float* const Cr = g.C + m * g.ldc + nl;
        if (lean) {
            const float s = rs_in ? rs : 1.f;
            float4 av[TN], mv[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                av[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                mv[j] = make_float4(1.f, 1.f, 1.f, 1.f);
                if (g.addend) av[j] = *reinterpret_cast<const float4*>(g.addend + m * g.ld_add + nl + 16 * j);
                if (g.mask) mv[j] = *reinterpret_cast<const float4*>(g.mask + m * g.ld_mask + nl + 16 * j);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                float4 v = make_float4(acc[i][j][0] + av[j].x, acc[i][j][1] + av[j].y, acc[i][j][2] + av[j].z, acc[i][j][3] + av[j].w);
                if (bias_in) {
                    const float4 b4 = *reinterpret_cast<const float4*>(g.bias + (nl - g.bias_col0) + 16 * j);
                    v.x += b4.x; v.y += b4.y; v.z += b4.z; v.w += b4.w;
                }
                if (g.C_raw) *reinterpret_cast<float4*>(g.C_raw + m * g.ld_raw + nl + 16 * j) = v;
                v.x *= s; v.y *= s; v.z *= s; v.w *= s;
                if (g.relu) {
                    v.x = v.x > 0.f ? v.x : 0.f; v.y = v.y > 0.f ? v.y : 0.f;
                    v.z = v.z > 0.f ? v.z : 0.f; v.w = v.w > 0.f ? v.w : 0.f;
                }
                v.x = mv[j].x > 0.f ? v.x : 0.f; v.y = mv[j].y > 0.f ? v.y : 0.f;
                v.z = mv[j].z > 0.f ? v.z : 0.f; v.w = mv[j].w > 0.f ? v.w : 0.f;
                *reinterpret_cast<float4*>(Cr + 16 * j) = v;
                if (COLS) acc[i][j] = floatx4{v.x * cm, v.y * cm, v.z * cm, v.w * cm};
            }
            continue;
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int nb = nl + 16 * j;
            float v[4], raw[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = nb + q, cb = n - g.bias_col0;
                float t = acc[i][j][q];
                if (n < g.N) {
                    if (g.addend) t += g.addend[m * g.ld_add + n];
                    if (g.bias && cb >= 0 && cb < bias_n) t += g.bias[cb];
                    raw[q] = t;
                    if (n < rs_cols) t *= rs;
                    if (g.relu) t = t > 0.f ? t : 0.f;
                    if (g.mask) t = g.mask[m * g.ld_mask + n] > 0.f ? t : 0.f;
                } else {
                    t = 0.f;
                    raw[q] = 0.f;
                }
                v[q] = t;
                if (COLS) acc[i][j][q] = t * cm;
            }
            if (vec) {
                if (nb >= n_store) continue;
                if (g.C_raw) *reinterpret_cast<float4*>(g.C_raw + m * g.ld_raw + nb) = make_float4(raw[0], raw[1], raw[2], raw[3]);
                *reinterpret_cast<float4*>(Cr + 16 * j) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (nb + q >= n_store) break;
                    if (g.C_raw) g.C_raw[m * g.ld_raw + nb + q] = raw[q];
                    Cr[16 * j + q] = v[q];
                }
            }
        }
    }
    // Column sums: over the 16 rows of the lanes' DPP row, then over the wavefronts.  (A pass of its own over C took 199 us over 2^20 rows of
    // 256, and a launch of 4.6 where the rows are few.)
    if constexpr (COLS) {
        if (!cols) return;
        __syncthreads();                              // everybody is done with the tiles of B
        float* const red = reinterpret_cast<float*>(lds);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float x = acc[0][j][q];
#pragma unroll
                for (int i = 1; i < TM; ++i) x += acc[i][j][q];
                auto turn = [](float y, auto ctrl) { return y + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), decltype(ctrl)::value, 0xF, 0xF, false)); };
                x = turn(x, std::integral_constant<int, 0x128>());      // row_ror 8, 4, 2, 1
                x = turn(x, std::integral_constant<int, 0x124>());
                x = turn(x, std::integral_constant<int, 0x122>());
                x = turn(x, std::integral_constant<int, 0x121>());
                (q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w) = x;
            }
            if (li == 0) *reinterpret_cast<float4*>(red + wave * BN + 16 * j + 4 * lq) = v;
        }
        __syncthreads();
        if (tid < BN && n0 + tid < g.N) g.col_part[slab * g.N + n0 + tid] = (red[tid] + red[BN + tid]) + (red[2 * BN + tid] + red[3 * BN + tid]);
    }
}
template <typename AT, int TM, int TN, bool IRREG, bool PRE = false>
__global__ __launch_bounds__(256, nt_wgs(TN, PRE, !IRREG && sizeof(AT) == 4)) void gemm_nt_kernel(GemmNNArgs g) {
    gemm_nt_kernel_body<AT, TM, TN, IRREG, PRE>(gridDim.x, g);
}
template <typename AT, int TM, int TN, bool IRREG, bool PRE = false>
struct gemm_nt_kernel_op {
    static constexpr int THREADS = 256, WGS = nt_wgs(TN, PRE, !IRREG && sizeof(AT) == 4);
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { gemm_nt_kernel_body<AT, TM, TN, IRREG, PRE>(gx, a...); }
};

// Bt as planes (bt_planes_at).
__global__ __launch_bounds__(256) void split_b_kernel(const float* __restrict__ Bt, int64_t ldbt, int K, const float* __restrict__ Bt2,
                                                      int64_t ldbt2, int K2, int N, int n_all, unsigned char* __restrict__ planes) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int nk1 = (K + BK - 1) / BK, nk = nk1 + (K2 + BK - 1) / BK;
    if (e >= nk * n_all * 4) return;
    const int q = e & 3, n = (e >> 2) % n_all, kt = (e >> 2) / n_all;
    const bool second = kt >= nk1;
    const int k0 = (second ? kt - nk1 : kt) * BK + 4 * q, Kc = second ? K2 : K;
    const float* const row = second ? Bt2 + (int64_t)n * ldbt2 : Bt + (int64_t)n * ldbt;
    float v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int k = k0 + (t & 3) + (t >= 4 ? 16 : 0);
        v[t] = n < N && k < Kc ? row[k] : 0.f;
    }
    uint4 part[3];
    split8(v, part[0], part[1], part[2]);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(planes + bt_planes_at(kt * BK + 4 * q, n, p, n_all)) = part[p];
}

size_t gemm_planes_bytes(int64_t M, int32_t N, int32_t K) {
    if (cdiv(M, 128) < NT_PRE_SLABS) return 0;
    return (size_t)(cdiv(K, BK) + 1) * 3 * round_up(N, 128) * 64;      // (two products round their k up one by one)
}

// Output tiles of an NT product: 128 rows by 128, 96, 64 or 32 columns, whichever covers the columns with the least to spare, or 64 x 64.
struct NtPlan {
    int tile_m, tile_n;
    int n_all;               // columns that the tiles cover
    size_t planes_need;
    bool pre;                // B is read as planes: a.ready, or made once in a.planes
    bool large;              // launched by itself
};
static NtPlan nt_plan(const GemmNNArgs& a, int n_eff) {
    NtPlan p;
    p.tile_m = 128;
    p.tile_n = n_eff > 96 ? 128 : n_eff > 64 ? 96 : n_eff > 32 ? 64 : 32;
    // A product whose 128-row tiles would leave half the chip idle (mini-batch blocks) is cut into
    // 64 x 64 tiles instead: four times the workgroups, each a quarter of the work.
    // (an upper bound of M that the device will cut down counts half: sampled blocks fill about that much)
    const int64_t m_plan = a.M_dev ? (a.M + 1) / 2 : a.M;
    const int64_t wide_tiles = cdiv(m_plan, 128) * cdiv(n_eff, p.tile_n);
    // A product with almost no reduction (K + K2 <= 64) is its epilogue: eight resident 64 x 64 workgroups per CU overlap their loads
    // and stores better than three wide ones (K = 32, N = 128 over 3e5 rows: 41 against 46 us; N = 100, 200: 47 against 70, 81 against 119),
    // until the wide ones, with half the splits of A and no column to spare, come in large numbers (K = 64, N = 128 over
    // 2e6 rows: 460 against 421 us, masked over 8.4e6 2.55 against 2.26 ms; N = 256 over 1e6 459 against 419 us), or waste the least
    // (N = 96 over 3e5 rows 43 against 34 us).
    const bool short_k = a.K + a.K2 <= 64 && !(n_eff % p.tile_n == 0 && (p.tile_n == 96 || (p.tile_n == 128 && wide_tiles >= 4096)));
    if (n_eff > 32 && (wide_tiles < 384 || short_k)) p.tile_m = p.tile_n = 64;
    // (W + the attention columns: 260 columns are three tiles of 96 with 28 to spare, of 128 with 124)
    else if (n_eff > 128 && round_up(n_eff, 96) < round_up(n_eff, 128)) p.tile_n = 96;
    // Both k tilings and the padding fit what gemm_planes_bytes reserved for this N and K + K2.
    p.n_all = (int)cdiv(n_eff, p.tile_n) * p.tile_n;
    p.planes_need = (size_t)(cdiv(a.K, BK) + cdiv(a.K2, BK)) * 3 * p.n_all * 64;
    p.large = cdiv(m_plan, 128) >= NT_PRE_SLABS;
    p.pre = a.ready || (p.tile_m == 128 && p.tile_n >= 64 && a.planes && p.large && p.planes_need <= a.planes_bytes);
    return p;
}

// The fp32 kernel's tiles (measured at M = 3e5): 128 x 128 output tiles at three workgroups per CU beat 128 x 256 at one; a 32-deep
// single-buffered k-tile is best for long reductions, a 16-deep double-buffered one wastes less on short or ragged K.
template <typename AT, bool VEC>
static void nn_pick(const GemmNNArgs& a, hipStream_t st) {
    const int n_eff = a.zero_pad_to > a.N ? a.zero_pad_to : a.N;
    const bool short_k = a.K <= 128 || (a.K2 > 0 && a.K2 <= 128);
    const int64_t slabs = round_up(cdiv(a.M, 128), NXCD);
    if (n_eff > 64) {
        const unsigned blocks = (unsigned)(slabs * cdiv(n_eff, 128));
        if (short_k) launch_alone((gemm_nn_kernel<AT, VEC, 2, 2, 2, 2, 16, 2>), dim3(blocks), dim3(256), 0, st, a);
        else launch_alone((gemm_nn_kernel<AT, VEC, 2, 2, 2, 2, 32, 1>), dim3(blocks), dim3(256), 0, st, a);
    } else if (n_eff > 32) {
        launch_alone((gemm_nn_kernel<AT, VEC, 4, 1, 1, 2, 32, 1>), dim3((unsigned)slabs), dim3(256), 0, st, a);
    } else {
        launch_alone((gemm_nn_kernel<AT, VEC, 4, 1, 1, 1, 32, 1>), dim3((unsigned)slabs), dim3(256), 0, st, a);
    }
}

grp_status launch_gemm_nn(const GemmNNArgs& a, hipStream_t st) {
    if (a.M == 0 || a.N == 0) return GRP_OK;
    if (a.M < 0 || a.N < 0 || a.K <= 0 || !a.A || (!a.B && !a.Bt) || !a.C) return fail(GRP_EINVAL, "gemm_nn: bad arguments");
    if (a.K2 > 0 && (!a.A2 || (!a.B2 && !a.Bt2) || a.lda2 % 4 != 0 || a.lda2 < round_up(a.K2, 4) || (uintptr_t)a.A2 % 16 != 0))
        return fail(GRP_EINVAL, "gemm_nn: second operand must be 16-byte aligned with a pitch multiple of 4");
    const int elem = a.a_bf16 ? 2 : 4;
    const bool veca = a.lda % 4 == 0 && a.lda >= round_up(a.K, 4) && (uintptr_t)a.A % (4 * elem) == 0;
    const bool vecb = a.B && a.ldb % 4 == 0 && a.ldb >= round_up(a.N, 4) && (uintptr_t)a.B % 16 == 0 &&
                      (a.K2 == 0 || (a.ldb2 % 4 == 0 && a.ldb2 >= round_up(a.N, 4) && (uintptr_t)a.B2 % 16 == 0));
    const double nn_flops = 2.0 * a.M * a.N * ((double)a.K + a.K2);
    const double nn_bytes = (double)a.M * a.K * elem + 4.0 * a.M * a.K2 + 4.0 * a.N * ((double)a.K + a.K2) +
                            4.0 * a.M * a.N * (1.0 + (a.addend ? 1.0 : 0.0) + (a.mask ? 1.0 : 0.0));
    prof_detail("[M=%lld,N=%d,K=%d+%d%s%s%s]", (long long)a.M, a.N, a.K, a.K2, a.addend ? ",add" : "", a.mask ? ",mask" : "",
                a.rowscale ? ",rs" : "");
    if (a.Bt) {
        // 32-bit element offsets inside a slab and inside Bt
        const bool small = a.lda < (1 << 23) && a.lda2 < (1 << 23) && (int64_t)a.N * a.ldbt < (1ll << 31) &&
                           (int64_t)a.N * a.ldbt2 < (1ll << 31);
        const bool ok = small && (veca || a.K >= 4) && a.ldbt % 4 == 0 && a.ldbt >= round_up(a.K, 4) && (uintptr_t)a.Bt % 16 == 0 &&
                        (a.K2 == 0 || (a.Bt2 && a.ldbt2 % 4 == 0 && a.ldbt2 >= round_up(a.K2, 4) && (uintptr_t)a.Bt2 % 16 == 0));
        const int n_eff = a.zero_pad_to > a.N ? a.zero_pad_to : a.N;
        const NtPlan p = nt_plan(a, n_eff);
        // One profiling name per tile shape and element type of the kernels, and per place where B is split, as in a kernel trace (a
        // product with planes includes the launch that makes them).
        char pname[64];
        snprintf(pname, sizeof pname, "gemm_%s_%s_%dx%d%s", ok ? "nt" : "nn", a.a_bf16 ? "bf16a" : "f32", ok ? p.tile_m : 128,
                 ok ? p.tile_n : n_eff > 64 ? 128 : n_eff > 32 ? 64 : 32, ok && p.pre ? "_planes" : "");
        ProfScope ps(pname, st, nn_flops, nn_bytes);
        if (!ok) {                                       // slow, always-safe kernel
            if (a.col_part) return fail(GRP_EUNSUPPORTED, "gemm_nn: column sums of such a product");
            if (a.a_bf16) nn_pick<__hip_bfloat16, false>(a, st); else nn_pick<float, false>(a, st);
            GRP_LAUNCH_CHECK();
            return GRP_OK;
        }
        GemmNNArgs t = a;
        t.a_tight = veca ? 0 : 1;
        const bool irreg = t.a_tight || a.a_rows != nullptr || a.a_valid_rows_dev != nullptr || (a.a_valid_rows > 0 && a.a_valid_rows < a.M);
        if (a.col_part) {
            if (irreg || a.a_bf16 || !p.pre || a.M_dev) return fail(GRP_EUNSUPPORTED, "gemm_nn: column sums of such a product");
            a.sums->add(SUM_COLUMNS, a.col_part, (int32_t)cdiv(a.M, p.tile_m), 0, a.N, 0, a.col_out, nullptr, nullptr, a.N);
        }
        const int64_t slabs = round_up(cdiv(a.M, p.tile_m), NXCD);
        const unsigned blocks = (unsigned)(slabs * cdiv(n_eff, p.tile_n));
        if (p.pre && !a.ready) {
            GRP_LARGE_LAUNCH(split_b_kernel, dim3((unsigned)cdiv((int64_t)p.planes_need / 48, 256)), dim3(256), 0, st, a.Bt, a.ldbt, a.K, a.Bt2,
                               a.ldbt2, a.K2, a.N, p.n_all, a.planes);
            t.ready = a.planes;
            t.ready2 = a.planes + (int64_t)cdiv(a.K, BK) * 3 * p.n_all * 64;
            t.ready_rows = p.n_all;
        }
        // (the products of a step have their planes ready: only those launches are merged)
#define GRP_NT_LAUNCH3(AT, TM_, TN_, IRR)                                                                                  \
    do {                                                                                                                   \
        if (p.pre && p.large) GRP_LARGE_LAUNCH((gemm_nt_kernel<AT, TM_, TN_, IRR, true>), dim3(blocks), dim3(256), 0, st, t); \
        else if (p.pre) launch(gemm_nt_kernel<AT, TM_, TN_, IRR, true>, gemm_nt_kernel_op<AT, TM_, TN_, IRR, true>(), dim3(blocks), st, t); \
        else launch_alone((gemm_nt_kernel<AT, TM_, TN_, IRR, false>), dim3(blocks), dim3(256), 0, st, t);                    \
    } while (0)
#define GRP_NT_LAUNCH2(AT, TM_, TN_)                                                                                       \
    do {                                                                                                                   \
        if (irreg) GRP_NT_LAUNCH3(AT, TM_, TN_, true); else GRP_NT_LAUNCH3(AT, TM_, TN_, false);                           \
    } while (0)
#define GRP_NT_LAUNCH(TM_, TN_)                                                                                            \
    do {                                                                                                                   \
        if (a.a_bf16) GRP_NT_LAUNCH2(__hip_bfloat16, TM_, TN_); else GRP_NT_LAUNCH2(float, TM_, TN_);                      \
    } while (0)
        if (p.tile_m == 64) GRP_NT_LAUNCH(1, 4);
        else if (p.tile_n == 128) GRP_NT_LAUNCH(2, 8);
        else if (p.tile_n == 96) GRP_NT_LAUNCH(2, 6);
        else if (p.tile_n == 64) GRP_NT_LAUNCH(2, 4);
        else GRP_NT_LAUNCH(2, 2);
#undef GRP_NT_LAUNCH3
#undef GRP_NT_LAUNCH2
#undef GRP_NT_LAUNCH
        GRP_LAUNCH_CHECK();
        return GRP_OK;
    }
    ProfScope ps(a.a_bf16 ? "gemm_nn_bf16a" : "gemm_nn_f32", st, nn_flops, nn_bytes);
    if (a.a_bf16) {
        if (veca && vecb) nn_pick<__hip_bfloat16, true>(a, st);
        else nn_pick<__hip_bfloat16, false>(a, st);
    } else {
        if (veca && vecb) nn_pick<float, true>(a, st);
        else nn_pick<float, false>(a, st);
    }
    GRP_LAUNCH_CHECK();
    return GRP_OK;
}

// ------------------------------------------------------------------------------- TN
constexpr int TN_IDLE = 128;                  // a launch of fewer workgroups leaves half the chip idle
constexpr int TN_MAX_SPLITS = 256;
constexpr int64_t TN_STREAM_ROWS = (int64_t)1 << 23;
constexpr int N_CU = 256;                     // a product is cut into one full round of resident workgroups (768 slices at two per CU: 6-8 % slower)

struct TnPlan {
    int tiles_k, tiles_n, splits;
    int64_t chunk;
    int bk_tile, bn_tile;
};

static TnPlan tn_plan(int64_t M, int K, int N, int products = 1) {
    TnPlan p;
    p.bn_tile = N > 64 ? 128 : (N > 32 ? 64 : 32);
    p.bk_tile = (K <= 64 && p.bn_tile >= 64) ? 64 : 128;      // a short K fills a 64-row tile
    // 96 columns, or 96 rows, where fewer of the tiles' elements lie beyond the product then (1e5 rows, K = 75 / 256, us, tiles of 128 and 96 columns:
    // N = 72 47/39 and 64/55, 130 62/53 and 107/89, 280 84/70 and 231/201; 3e3 rows, K = 75: 14.2/12.6, 15.5/13.6, 18.0/15.2.
    // K = 72 / 280, N = 256: 63/54 and 231/199; 3e3 rows: 16.4/15.5, 22.8/21.2).
    if (N > 64 && p.bk_tile == 128) {
        const int64_t n128 = round_up(N, 128), n96 = round_up(N, 96), k128 = round_up(K, 128), k96 = round_up(K, 96);
        if (n96 * k128 < n128 * k128 && n96 * k128 <= n128 * k96) p.bn_tile = 96;
        else if (k96 < k128) p.bk_tile = 96;
    }
    p.tiles_k = (int)cdiv(K, p.bk_tile);
    p.tiles_n = (int)cdiv(N, p.bn_tile);
    // Products over very many rows are cut into up to eight times the slices: the chains of partial sums get that much shorter (at 256
    // slices of 1.7e7 rows an accumulator is rounded 2000 times), and the partial tiles cost nothing beside 10^7 rows (bf16 K = 64,
    // N = 128 over 1.7e7 rows 2.34 ms in one round of workgroups, 2.38 in four; K = 128, N = 16 1.95 and 1.94; at 3e5 rows four times the
    // slices cost 4 %).
    const bool stream = M >= TN_STREAM_ROWS;
    const int target = N_CU * tn_wgs(p.bk_tile * p.bn_tile / 4096);      // (tiles of 32 x 32 per wavefront)
    int64_t s = (stream ? 4 * target : target) / (p.tiles_k * p.tiles_n * products);
    // A lone workgroup spends over a microsecond on 32 rows: slices of 128, of fewer where that leaves most of the chip idle (with the
    // sum over the slices, us: K = N = 64 over 2500 rows 11.9 -> 9.7; K = N = 256 over 256 18.4 -> 11.9, 1024 19.1 -> 15.4, 2500 21.2 -> 19.2;
    // K = 128, N = 256 over 1024 18.4 -> 14.0).
    const int64_t tiles = (int64_t)p.tiles_k * p.tiles_n * products;
    const int rows_min = tiles * cdiv(M, 128) > TN_IDLE ? 128 : tiles * cdiv(M, 64) > TN_IDLE ? 64 : 32;
    if (s > cdiv(M, rows_min)) s = cdiv(M, rows_min);
    if (s > (stream ? 8 * TN_MAX_SPLITS : TN_MAX_SPLITS)) s = stream ? 8 * TN_MAX_SPLITS : TN_MAX_SPLITS;
    if (s < 1) s = 1;
    p.chunk = round_up(cdiv(M, s), BK);
    if (p.chunk < BK) p.chunk = BK;
    p.splits = (int)cdiv(M, p.chunk);
    if (p.splits < 1) p.splits = 1;
    return p;
}

// The most slices of any product of at most M rows.  The slices of a plan do not grow with its rows alone: rows_min doubles where they
// leave the chip less idle, and the rounding of a chunk drops slices (6000 rows at K = N = 128, two products: 94; 10 584 rows: 83).  A scratch
// array sized for an upper bound of the rows has to do for every launch below it.
static int64_t tn_most_splits(int64_t M, int K, int N, int products) {
    const TnPlan p = tn_plan(M, K, N, products);           // (tiles: the same for every M)
    const int64_t tiles = (int64_t)p.tiles_k * p.tiles_n * products;
    const bool stream = M >= TN_STREAM_ROWS;
    const int64_t target = N_CU * tn_wgs(p.bk_tile * p.bn_tile / 4096);
    int64_t s = cdiv(M, 128);
    for (int rows_min = 64; rows_min >= 32; rows_min /= 2)     // slices so short are made up to this many rows
        s = std::max(s, cdiv(std::min(M, 2 * rows_min * (TN_IDLE / tiles)), rows_min));
    s = std::min({s, (stream ? 4 * target : target) / tiles, (int64_t)(stream ? 8 : 1) * TN_MAX_SPLITS});
    return std::max<int64_t>(s, 1);
}

// (does not shrink as M grows)
size_t gemm_tn_workspace_bytes(int64_t M, int32_t K, int32_t N) {
    // room for one product, or for two from one launch: (2K + 1) rows of N, or (K + 1) rows of 2N
    size_t need = 0;
    for (int products = 1; products <= 2; ++products) {
        const int64_t splits = tn_most_splits(M, K, N, products);
        if (splits <= 1) continue;
        const size_t rows_n = products == 1 ? (size_t)(K + 1) * N : std::max((size_t)(2 * (size_t)K + 1) * N, (size_t)(K + 1) * 2 * N);
        need = std::max(need, (size_t)splits * rows_n * sizeof(float));
    }
    return need;
}

// Grid: x = NXCD * tiles * ceil(splits / NXCD).  Workgroup ids are mapped so that the output
// tiles of one slice of the node dimension run on the same L2 domain (they read the same rows).
// The matrix instruction wants eight consecutive k per lane, and k is the node dimension here: a staging thread loads
// four columns of eight consecutive rows, which in its registers are four runs of eight k values.  Column 4*g + q of a
// tile W columns wide is kept in tile row q*(W/4) + g, so that the lanes of a wavefront (consecutive g) write consecutive
// rows.  The first threads stage A, the next ones B (or the other way round).  LDS rows hold 32 k values (64 bytes, 4 places of 16); the eight k
// from 8*c of a row sit at place c ^ tn_turn(row).
// Whole 32-row steps load as they are; columns past K or N are read from clamped
// addresses and never masked, since they only reach output rows / columns that are not stored.
// GATHER: rows of A are taken through g.a_rows, or an operand is tightly packed.  cs_out (optional): the workgroups of the
// first row of output tiles also add up the columns of B they stream.

// Chosen so that neither side meets a bank conflict (counted: none): a 16-byte write serves eight consecutive lanes, here rows, per
// cycle over 32 banks, a 16-byte read sixteen lanes over 64 banks (lanes 0-3, 12-15, 20-27; 4-11, 16-19, 28-31; ...).
__device__ __forceinline__ int tn_turn(int row) {
    const int y = row >> 3;
    return ((row >> 1) ^ (2 * (y & 1)) ^ ((y ^ (y >> 1)) & 1)) & 3;
}

template <typename AT, bool VEC, bool GATHER, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void gemm_tn_kernel_body(unsigned gx, GemmTNArgs g, int tiles_k, int tiles_n, int dual, int splits, int64_t chunk,
                                                      float* __restrict__ out, float* __restrict__ out2, int64_t out_ld,
                                                      int64_t out_split_stride, float* __restrict__ cs_out,
                                                      int64_t cs_split_stride) {
    if (g.M_dev) {                                         // the launch was sized by an upper bound of M:
        g.M = *g.M_dev;                                    // the real rows are dealt evenly to its slices
        chunk = (g.M + splits - 1) / splits;
        chunk = (chunk + BK - 1) / BK * BK;
        if (chunk < BK) chunk = BK;
    }
    constexpr int BKA = WM * TM * 32, BN = WN * TN * 32;   // output tile: BKA (rows of C) x BN
    constexpr int PLANE_A = BKA * 64, PLANE_B = BN * 64;
    constexpr int QA = BKA / 4, QB = BN / 4;               // column groups of a tile
    constexpr int TA = QA * (BK / 8), TB = QB * (BK / 8);  // staging threads of each operand
    constexpr int A0 = TA % 64 == 0 ? 0 : TB, B0 = A0 ? 0 : TA;      // their first threads
    // (Written for either order, the narrowest bf16 tiles have 81 to 85 registers in their 40 bytes of scratch where 13 were: 3e5 rows, K = N = 64
    // 63.5 -> 50.8 us, K = 256, N = 32 83.2 -> 58.2, 3e3 rows 10.2 -> 9.9.)
    static_assert((A0 ? TB : TA) % 64 == 0 && TA + TB <= 256 && QA % 8 == 0 && QB % 8 == 0, "an operand is staged by whole wavefronts");
    __shared__ __attribute__((aligned(16))) unsigned char lds[3 * (PLANE_A + PLANE_B)];
    unsigned char* const As = lds;
    unsigned char* const Bs = lds + 3 * PLANE_A;

    // dual = 1: the second half of the tiles multiplies A2 instead of A; dual = 2: B2 instead of B
    const int tiles1 = tiles_k * tiles_n;
    const int tiles = tiles1 * (dual ? 2 : 1);
    const int hq = blockIdx.x / NXCD;
    const int tile_all = hq % tiles;
    const bool op2 = tile_all >= tiles1;
    const int tile = tile_all % tiles1;
    const int split = (hq / tiles) * NXCD + blockIdx.x % NXCD;
    if (split >= splits) return;
    const bool a2 = op2 && dual == 1, b2 = op2 && dual == 2;
    const bool a_one = sizeof(AT) == 2 && !a2;             // A is stored in bf16: one plane
    const int ka0 = (tile / tiles_n) * BKA;
    const int n0 = (tile % tiles_n) * BN;
    const int64_t m_begin = (int64_t)split * chunk;
    const int64_t m_end = m_begin + chunk < g.M ? m_begin + chunk : g.M;

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WN, wn = wave % WN;
    const bool is_a = tid >= A0 && tid < A0 + TA, is_b = tid >= B0 && tid < B0 + TB;
    const int q_n = is_a ? QA : QB;                        // the operand this thread stages:
    const int lt = tid - (is_a ? A0 : B0);
    const int grp = lt % q_n, mb = lt / q_n;               // four columns from 4 * grp, eight rows from 8 * mb
    const void* const op = is_a ? (a2 ? (const void*)g.A2 : g.A) : (const void*)(b2 ? g.B2 : g.B);
    const int64_t ld = is_a ? (a2 ? g.lda2 : g.lda) : (b2 ? g.ldb2 : g.ldb);
    const int width = is_a ? g.K : g.N;
    const int c_first = (is_a ? ka0 : n0) + 4 * grp;
    // the first column of an operand's last group: rows without room for all of it end it at their last element, and its
    // columns then repeat some of the group before
    const int last_a = (GATHER && g.a_tight && !a2) ? g.K - 4 : ((g.K + 3) & ~3) - 4;
    const int last_b = GATHER && g.b_tight ? g.N - 4 : ((g.N + 3) & ~3) - 4;
    const int col = imin(c_first, is_a ? last_a : last_b);
    const bool bf16 = is_a && a_one;
    const int32_t* const rows = (GATHER && is_a && !a2) ? g.a_rows : nullptr;
    const bool do_cs = cs_out != nullptr && ka0 == 0 && !op2;
    // What the matrix unit cuts off has always the same sign, which would add up over the tiles of a long reduction: every other tile is
    // multiplied as -A^T B and subtracted.
    uint32_t flip = 0;                                     // of the staged tile
    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    float csum[4] = {0.f, 0.f, 0.f, 0.f};
    uint4 raw[8];

    auto fetch = [&](int64_t mt) {
        if (!is_a && !is_b) return;
        const int64_t mr = mt + 8 * mb;
        if (VEC && !rows && mt + BK <= m_end) {
            if (sizeof(AT) == 2 && bf16) {
                const __hip_bfloat16* p = (const __hip_bfloat16*)op + mr * ld + col;
#pragma unroll
                for (int r = 0; r < 8; ++r) raw[r] = ldg_raw4<__hip_bfloat16, GATHER>(p + r * ld);
            } else {
                const float* p = (const float*)op + mr * ld + col;
#pragma unroll
                for (int r = 0; r < 8; ++r) raw[r] = ldg_raw4<float, GATHER>(p + r * ld);
            }
            return;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const bool ok = mr + r < m_end;
            const int64_t gm = lmin(mr + r, g.M - 1);
            const int64_t row = rows ? (int64_t)rows[gm] : gm;
            if constexpr (VEC) {
                if (sizeof(AT) == 2 && bf16) raw[r] = ldg_raw4<__hip_bfloat16, GATHER>((const __hip_bfloat16*)op + row * ld + col);
                else raw[r] = ldg_raw4<float, GATHER>((const float*)op + row * ld + col);
                if (!ok) raw[r] = make_uint4(0u, 0u, 0u, 0u);
            } else if (sizeof(AT) == 2 && bf16) {          // back to packed halves
                const uint4 f = ldg_safe4((const __hip_bfloat16*)op + row * ld, ok, c_first, width);
                raw[r] = make_uint4((f.x >> 16) | (f.y & 0xFFFF0000u), (f.z >> 16) | (f.w & 0xFFFF0000u), 0u, 0u);
            } else {
                raw[r] = ldg_safe4((const float*)op + row * ld, ok, c_first, width);
            }
        }
    };
    unsigned char* put[4];                                 // where the eight rows of column 4 * grp + q go: tile row q * q_n + grp
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = q * q_n + grp;
        put[q] = (is_a ? As : Bs) + 64 * row + 16 * (mb ^ tn_turn(row));
    }
    auto stage = [&]() {
        if (sizeof(AT) == 2 && bf16) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t sel = (q & 1) ? 0x07060302u : 0x05040100u;
                auto w = [&](int r) { return __builtin_amdgcn_perm(q < 2 ? raw[r + 1].x : raw[r + 1].y, q < 2 ? raw[r].x : raw[r].y, sel); };
                const uint32_t fl = flip | (flip >> 16);
                *reinterpret_cast<uint4*>(put[q]) = make_uint4(w(0) ^ fl, w(2) ^ fl, w(4) ^ fl, w(6) ^ fl);
            }
            return;
        }
        if (!is_a && !is_b) return;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint4 t = raw[r];
                v[r] = __uint_as_float(q == 0 ? t.x : q == 1 ? t.y : q == 2 ? t.z : t.w);
            }
            if (is_a) {
#pragma unroll
                for (int r = 0; r < 8; ++r) v[r] = __uint_as_float(__float_as_uint(v[r]) ^ flip);
                put_split8<PLANE_A>(put[q], v);
            } else {
                put_split8<PLANE_B>(put[q], v);
                if (do_cs) csum[q] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            }
        }
    };
    const int li = lane & 31, lk = lane >> 5;
    const unsigned char* const ap0 = As + 64 * (wm * TM * 32 + li);
    const unsigned char* const bp0 = Bs + 64 * (wn * TN * 32 + li);
    const int c0 = 16 * (lk ^ tn_turn(li));

    if (m_begin < m_end) {
        fetch(m_begin);
        stage();
        __syncthreads();
        for (int64_t mt = m_begin; mt < m_end; mt += BK) {
            const bool more = mt + BK < m_end;
            if (more) fetch(mt + BK);
            mma32<TM, TN, PLANE_A, PLANE_B, sizeof(AT) == 2>(ap0, bp0, c0, a_one, flip ? -1.f : 1.f, acc);
            __syncthreads();
            if (more) {
                flip ^= 0x80000000u;
                stage();
                __syncthreads();
            }
        }
    }

    // Partial tiles (out2 null): the second product's rows follow the first's K rows (dual = 1) or its
    // columns follow the first's N columns (dual = 2).  Direct output: out2 is the second matrix.
    float* o = (op2 && out2 ? out2 : out) + (int64_t)split * out_split_stride;
    if (op2 && !out2) o += a2 ? (int64_t)g.K * out_ld : (int64_t)g.N;
    // (an own copy of the thread's number: what is derived from it here need not be kept in registers during the loop above)
    int tid_e = tid;
    asm volatile("" : "+v"(tid_e));
    const int li_e = tid_e & 31, lk_e = (tid_e >> 5) & 1, wm_e = (tid_e >> 6) / WN, wn_e = (tid_e >> 6) % WN;
    auto col_of = [&](int j) {                        // the output column of this lane's accumulators [.][j] (g.N: none)
        const int row = wn_e * TN * 32 + 32 * j + li_e;
        const int c = n0 + 4 * (row % QB), cr = imin(c, last_b) + row / QB;
        return cr < g.N && (!GATHER || cr >= c) ? cr : g.N;      // (repeated: not stored)
    };
    auto row_of = [&](int i, int r) {                 // and the output row of accumulator [i][.][r] (g.K: none)
        const int row = wm_e * TM * 32 + 32 * i + 8 * (r / 4) + 4 * lk_e + (r % 4);
        const int kc = ka0 + 4 * (row % QA), ka = imin(kc, last_a) + row / QA;
        return ka < g.K && (!GATHER || ka >= kc) ? ka : g.K;
    };
    // Results that are not finite are added up again in plain fp32, as in gemm_nt_kernel.
    float odd[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) odd[r & 3] = fmaf(acc[i][j][r], 0.f, odd[r & 3]);
    if (!((odd[0] + odd[1]) + (odd[2] + odd[3]) == 0.f)) {
#pragma unroll 1
        for (int e = 0; e < TM * TN * 16; ++e) {
            auto each = [&](auto f) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[i][j][r] = f((i * TN + j) * 16 + r, acc[i][j][r]);
            };
            float v = 0.f;
            each([&](int at, float x) { v = at == e ? x : v; return x; });
            const int ka = row_of(e / (16 * TN), e % 16), c = col_of(e / 16 % TN);
            if (isfinite(v) || ka >= g.K || c >= g.N) continue;
            v = 0.f;
            for (int64_t m = m_begin; m < m_end && !isnan(v); ++m) {
                const float x = a2 ? g.A2[m * g.lda2 + ka] : to_f<AT>(((const AT*)g.A)[(g.a_rows ? (int64_t)g.a_rows[m] : m) * g.lda + ka]);
                v = fmaf(x, b2 ? g.B2[m * g.ldb2 + c] : g.B[m * g.ldb + c], v);
            }
            each([&](int at, float x) { return at == e ? v : x; });
        }
    }
    int cols[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) cols[j] = col_of(j);
    const bool pair = TN == 2 && BN == 128 && out_ld % 2 == 0 && ((uintptr_t)o % 8) == 0 && cols[TN - 1] < g.N &&
                      (!GATHER || (cols[0] < g.N && cols[0] % 2 == 0));      // neighbours
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ka = row_of(i, r);
            if (ka >= g.K) continue;
            float* orow = o + (int64_t)ka * out_ld;
            if constexpr (TN == 2) {
                if (pair) { *reinterpret_cast<float2*>(orow + cols[0]) = make_float2(acc[i][0][r], acc[i][1][r]); continue; }
            }
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (cols[j] < g.N) orow[cols[j]] = acc[i][j][r];
        }
    if (do_cs) {                                      // the main loop ended on a barrier: the tiles are free
        float* red = reinterpret_cast<float*>(lds);
        if (is_b) {
#pragma unroll
            for (int q = 0; q < 4; ++q) red[mb * BN + 4 * grp + q] = csum[q];
        }
        __syncthreads();
        if (tid < BN) {
            float t = 0.f;
#pragma unroll
            for (int u = 0; u < BK / 8; ++u) t += red[u * BN + tid];
            const int c = n0 + (tid & ~3), cr = imin(c, last_b) + (tid & 3);
            if (cr < g.N && cr >= c) cs_out[(int64_t)split * cs_split_stride + cr] = t;
        }
    }
}
template <typename AT, bool VEC, bool GATHER, int WM, int WN, int TM, int TN>
__global__ __launch_bounds__(256, tn_wgs(TM * TN)) void gemm_tn_kernel(GemmTNArgs g, int tiles_k, int tiles_n, int dual, int splits, int64_t chunk,
                                                      float* __restrict__ out, float* __restrict__ out2, int64_t out_ld,
                                                      int64_t out_split_stride, float* __restrict__ cs_out,
                                                      int64_t cs_split_stride) {
    gemm_tn_kernel_body<AT, VEC, GATHER, WM, WN, TM, TN>(gridDim.x, g, tiles_k, tiles_n, dual, splits, chunk, out, out2, out_ld, out_split_stride, cs_out, cs_split_stride);
}
template <typename AT, bool VEC, bool GATHER, int WM, int WN, int TM, int TN>
struct gemm_tn_kernel_op {
    static constexpr int THREADS = 256, WGS = tn_wgs(TM * TN);
    template <class... A> static __device__ __forceinline__ void run(unsigned gx, const A&... a) { gemm_tn_kernel_body<AT, VEC, GATHER, WM, WN, TM, TN>(gx, a...); }
};

__global__ __launch_bounds__(256) void tn_reduce_kernel(const float* __restrict__ part, int splits, int K, int N, int64_t part_stride,
                                                        float* __restrict__ C, int64_t ldc, float* __restrict__ colsum_out, int dual,
                                                        float* __restrict__ C2, int64_t total) {
    tn_reduce_block(blockIdx.x, part, splits, K, N, part_stride, C, ldc, colsum_out, dual, C2, total);
}
__global__ __launch_bounds__(256) void tn_reduce_vec_kernel(const float* __restrict__ part, int splits, int K, int N, int64_t part_stride,
                                                            float* __restrict__ C, int64_t ldc, float* __restrict__ colsum_out, int dual,
                                                            float* __restrict__ C2, int64_t total) {
    tn_reduce_vec_block(blockIdx.x, part, splits, K, N, part_stride, C, ldc, colsum_out, dual, C2, total);
}
__global__ __launch_bounds__(256) void tn_reduce_4way_kernel(const float* __restrict__ part, int splits, int K, int N, int64_t part_stride,
                                                             float* __restrict__ C, int64_t ldc, float* __restrict__ colsum_out, int dual,
                                                             float* __restrict__ C2, int64_t total) {
    tn_reduce_4way_block(blockIdx.x, part, splits, K, N, part_stride, C, ldc, colsum_out, dual, C2, total);
}

template <typename AT, bool VEC, bool GATHER>
static void tn_pick(const GemmTNArgs& a, const TnPlan& p, int dual, float* out, float* out2, int64_t out_ld, int64_t stride,
                    float* cs_out, hipStream_t st) {
    const unsigned blocks = (unsigned)(NXCD * p.tiles_k * p.tiles_n * (dual ? 2 : 1) * cdiv(p.splits, NXCD));
    dim3 grid(blocks);
#define GRP_TN_LAUNCH(WM_, WN_, TM_, TN_)                                                                              \
    do {                                                                                                               \
        if constexpr (VEC)                                                                                             \
            launch(gemm_tn_kernel<AT, VEC, GATHER, WM_, WN_, TM_, TN_>, gemm_tn_kernel_op<AT, VEC, GATHER, WM_, WN_, TM_, TN_>(), grid, st, a, \
                   p.tiles_k, p.tiles_n, dual, p.splits, p.chunk, out, out2, out_ld, stride, cs_out, stride);           \
        else                                                                                                           \
            launch_alone((gemm_tn_kernel<AT, VEC, GATHER, WM_, WN_, TM_, TN_>), grid, dim3(256), 0, st, a, p.tiles_k, \
                             p.tiles_n, dual, p.splits, p.chunk, out, out2, out_ld, stride, cs_out, stride);            \
    } while (0)
    if (p.bk_tile == 64 && p.bn_tile == 128) GRP_TN_LAUNCH(2, 2, 1, 2);
    else if (p.bk_tile == 64) GRP_TN_LAUNCH(2, 2, 1, 1);
    else if (p.bk_tile == 96) GRP_TN_LAUNCH(1, 4, 3, 1);
    else if (p.bn_tile == 128) GRP_TN_LAUNCH(2, 2, 2, 2);
    else if (p.bn_tile == 96) GRP_TN_LAUNCH(4, 1, 1, 3);
    else if (p.bn_tile == 64) GRP_TN_LAUNCH(4, 1, 1, 2);
    else GRP_TN_LAUNCH(4, 1, 1, 1);
#undef GRP_TN_LAUNCH
}

// One launch computes C = A^T B and, when a second operand is given, C2 = A2^T B (a.A2) or
// C2 = A^T B2 (a.B2); C2 has C's shape and leading dimension.  A2 is fp32 and never gathered.
grp_status launch_gemm_tn(const GemmTNArgs& a, hipStream_t st) {
    if (a.K <= 0 || a.N <= 0 || a.M < 0 || !a.C) return fail(GRP_EINVAL, "gemm_tn: bad arguments");
    if (a.M > 0 && (!a.A || !a.B)) return fail(GRP_EINVAL, "gemm_tn: null operand");
    if (a.A2 && a.B2) return fail(GRP_EINVAL, "gemm_tn: at most one second operand");
    const int dual = a.A2 ? 1 : (a.B2 ? 2 : 0);
    if (dual && !a.C2) return fail(GRP_EINVAL, "gemm_tn: second product without an output");
    const TnPlan p = tn_plan(a.M, a.K, a.N, dual ? 2 : 1);
    // partial tiles of one slice: the products' rows (dual = 1: 2K) by their columns (dual = 2: 2N), then
    // one more row for the column sums of B
    const int64_t krows = dual == 1 ? 2 * (int64_t)a.K : a.K;
    const int64_t width = dual == 2 ? 2 * (int64_t)a.N : a.N;
    const int64_t stride = p.splits > 1 ? (krows + 1) * width : 0;
    const size_t need = (size_t)p.splits * stride * sizeof(float);
    if (need > a.workspace_bytes || (need && !a.workspace))
        return fail(GRP_EWORKSPACE, "gemm_tn: workspace %zu < %zu bytes", a.workspace_bytes, need);
    const int elem = a.a_bf16 ? 2 : 4;
    // vector path: 16-byte friendly operands whose 32-row steps fit 32-bit element offsets
    const bool veca = a.M > 0 && a.lda % 4 == 0 && a.lda >= round_up(a.K, 4) && (uintptr_t)a.A % (4 * elem) == 0 && a.lda < (1 << 25);
    const bool vecb = a.M > 0 && a.ldb % 4 == 0 && a.ldb >= round_up(a.N, 4) && (uintptr_t)a.B % 16 == 0 && a.ldb < (1 << 25);
    const bool veca2 = !a.A2 || (a.lda2 % 4 == 0 && a.lda2 >= round_up(a.K, 4) && (uintptr_t)a.A2 % 16 == 0 && a.lda2 < (1 << 25));
    const bool vecb2 = !a.B2 || (a.ldb2 % 4 == 0 && a.ldb2 >= round_up(a.N, 4) && (uintptr_t)a.B2 % 16 == 0 && a.ldb2 < (1 << 25));
    float* out = p.splits > 1 ? (float*)a.workspace : a.C;
    float* out2 = p.splits > 1 ? nullptr : a.C2;
    const int64_t out_ld = p.splits > 1 ? width : a.ldc;
    float* cs_out = !a.colsum_out ? nullptr : (p.splits > 1 ? (float*)a.workspace + krows * width : a.colsum_out);
    {
        prof_detail("[M=%lld,K=%d,N=%d%s%s]", (long long)a.M, a.K, a.N, a.colsum_out ? ",colsum" : "",
                    dual == 1 ? ",A2" : (dual == 2 ? ",B2" : ""));
        const double prods = dual ? 2.0 : 1.0;
        ProfScope ps(a.a_bf16 ? "gemm_tn_bf16a" : "gemm_tn_f32", st, 2.0 * prods * a.M * a.K * a.N,
                     (double)a.M * a.K * (elem + (dual == 1 ? 4 : 0)) + 4.0 * a.M * a.N * (dual == 2 ? 2 : 1) + 4.0 * prods * a.K * a.N);
        // A2 and B2 come from the step's own arrays; A and B may have any pitch and alignment (see last_a, last_b)
        const bool vec = (veca || (a.K >= 4 && a.lda < (1 << 25))) && (vecb || (a.N >= 4 && a.ldb < (1 << 25) && !a.B2)) && veca2 && vecb2 && a.M > 0;
        GemmTNArgs t = a;
        t.a_tight = vec && !veca;
        t.b_tight = vec && !vecb;
        if (a.a_bf16) {
            if (vec && !a.a_rows && veca && vecb) tn_pick<__hip_bfloat16, true, false>(t, p, dual, out, out2, out_ld, stride, cs_out, st);
            else if (vec) tn_pick<__hip_bfloat16, true, true>(t, p, dual, out, out2, out_ld, stride, cs_out, st);
            else tn_pick<__hip_bfloat16, false, true>(t, p, dual, out, out2, out_ld, stride, cs_out, st);
        } else {
            if (vec && !a.a_rows && veca && vecb) tn_pick<float, true, false>(t, p, dual, out, out2, out_ld, stride, cs_out, st);
            else if (vec) tn_pick<float, true, true>(t, p, dual, out, out2, out_ld, stride, cs_out, st);
            else tn_pick<float, false, true>(t, p, dual, out, out2, out_ld, stride, cs_out, st);
        }
        GRP_LAUNCH_CHECK();
    }
    if (p.splits > 1) {
        const int64_t total = krows * width + (a.colsum_out ? a.N : 0);
        const SumKind kind = stride % 4 == 0 && total % 4 == 0 && (uintptr_t)a.workspace % 16 == 0 && p.splits >= 16 ? SUM_TN_VEC
                             : p.splits >= 16 ? SUM_TN_4WAY : SUM_TN;
        if (a.sums && a.ldc == a.N) {                      // left to the step's last launch
            a.sums->add(kind, a.workspace, p.splits, a.K, a.N, dual, a.C, a.C2, a.colsum_out, total);
            return GRP_OK;
        }
        ProfScope ps("gemm_tn_reduce", st, 0.0, 4.0 * total * (p.splits + 1.0));
        auto go = [&](auto kernel) {
            launch_alone(kernel, dim3((unsigned)cdiv(total, sum_block(kind))), dim3(256), 0, st, (const float*)a.workspace, p.splits, a.K, a.N, stride,
                         a.C, a.ldc, a.colsum_out, dual, a.C2, total);
        };
        if (kind == SUM_TN_VEC) go(tn_reduce_vec_kernel);
        else if (kind == SUM_TN_4WAY) go(tn_reduce_4way_kernel);
        else go(tn_reduce_kernel);
        GRP_LAUNCH_CHECK();
    }
    return GRP_OK;
}

}  // namespace grp

extern "C" grp_status grp_gemm_nn(int64_t M, int32_t N, int32_t K, const void* A, int64_t lda, int32_t a_dtype,
                                  const float* B, int64_t ldb, float* C, int64_t ldc, void* stream) {
    if (M < 0 || N <= 0 || K <= 0 || lda < K || ldb < N || ldc < N) return grp::fail(GRP_EINVAL, "grp_gemm_nn: bad shape");
    if (!B || (M > 0 && (!A || !C))) return grp::fail(GRP_EINVAL, "grp_gemm_nn: null argument");
    if (M == 0) return GRP_OK;                          // no rows: nothing to compute
    grp::GemmNNArgs a;
    a.M = M; a.N = N; a.K = K; a.A = A; a.lda = lda; a.a_bf16 = a_dtype == GRP_DTYPE_BF16;
    a.B = B; a.ldb = ldb; a.C = C; a.ldc = ldc;
    return grp::launch_gemm_nn(a, (hipStream_t)stream);
}

extern "C" grp_status grp_gemm_nt(int64_t M, int32_t N, int32_t K, const void* A, int64_t lda, int32_t a_dtype,
                                  const float* Bt, int64_t ldbt, float* C, int64_t ldc, void* stream) {
    if (!Bt || (M > 0 && (!A || !C))) return grp::fail(GRP_EINVAL, "grp_gemm_nt: null argument");
    if (M < 0 || N <= 0 || K <= 0 || lda < K || ldbt < K || ldc < N) return grp::fail(GRP_EINVAL, "grp_gemm_nt: bad shape");
    if (M == 0) return GRP_OK;                          // no rows: nothing to compute
    grp::GemmNNArgs a;
    a.M = M; a.N = N; a.K = K; a.A = A; a.lda = lda; a.a_bf16 = a_dtype == GRP_DTYPE_BF16;
    a.Bt = Bt; a.ldbt = ldbt; a.C = C; a.ldc = ldc;
    return grp::launch_gemm_nn(a, (hipStream_t)stream);
}

extern "C" size_t grp_gemm_tn_workspace_bytes(int64_t M, int32_t K, int32_t N) {
    if (M < 0 || K <= 0 || N <= 0) return 0;
    return grp::gemm_tn_workspace_bytes(M, K, N);
}

extern "C" grp_status grp_gemm_tn(int64_t M, int32_t K, int32_t N, const void* A, int64_t lda, int32_t a_dtype,
                                  const float* B, int64_t ldb, float* C, int64_t ldc, void* workspace,
                                  size_t workspace_bytes, void* stream) {
    if (!C || (M > 0 && (!A || !B))) return grp::fail(GRP_EINVAL, "grp_gemm_tn: null argument");
    if (M < 0 || N <= 0 || K <= 0 || lda < K || ldb < N || ldc < N) return grp::fail(GRP_EINVAL, "grp_gemm_tn: bad shape");
    grp::GemmTNArgs a;
    a.M = M; a.K = K; a.N = N; a.A = A; a.lda = lda; a.a_bf16 = a_dtype == GRP_DTYPE_BF16;
    a.B = B; a.ldb = ldb; a.C = C; a.ldc = ldc; a.workspace = workspace; a.workspace_bytes = workspace_bytes;
    return grp::launch_gemm_tn(a, (hipStream_t)stream);
}
