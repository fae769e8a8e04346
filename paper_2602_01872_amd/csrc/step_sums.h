// Sums over partial results, a workgroup at a time: of the transposed products' slices and of column sums.  The kernel of a lone
// product is built from them, and the launch that ends a step (step_sums_kernel), which does all that its products and column sums left.
#pragma once
#include "common.h"

namespace grp {

// Where element (row, col) of the reduced partials goes: rows [0, K) x cols [0, N) -> C; with two
// products the second one's rows [K, 2K) (dual = 1) or columns [N, 2N) (dual = 2) -> C2; the last row
// holds the column sums of B (its first N columns).
__device__ __forceinline__ void tn_store(int64_t e, float val, int K, int N, int dual, float* __restrict__ C,
                                         float* __restrict__ C2, int64_t ldc, float* __restrict__ colsum_out) {
    const int width = dual == 2 ? 2 * N : N;
    const int64_t row = e / width;
    const int col = (int)(e % width);
    const int krows = dual == 1 ? 2 * K : K;
    if (row >= krows) {
        if (colsum_out && col < N) colsum_out[col] = val;
    } else if (dual == 1 && row >= K) {
        C2[(row - K) * ldc + col] = val;
    } else if (dual == 2 && col >= N) {
        C2[row * ldc + (col - N)] = val;
    } else {
        C[row * ldc + col] = val;
    }
}

// C[e] = sum_p part[p][e], p ascending.  Four partial tiles are requested before the first is
// added (the adds stay in split order, so the result is the plain sequential sum).
__device__ __forceinline__ void tn_reduce_block(uint32_t block, const float* __restrict__ part, int splits, int K, int N,
                                                        int64_t part_stride, float* __restrict__ C, int64_t ldc,
                                                        float* __restrict__ colsum_out, int dual, float* __restrict__ C2,
                                                        int64_t total) {
    const int64_t e = (int64_t)block * 256 + threadIdx.x;
    if (e >= total) return;                           // total = (rows of products + the column-sum row) x width
    const float* p0 = part + e;
    float s = 0.f;
    int p = 0;
    for (; p + 4 <= splits; p += 4) {
        const float a = p0[(int64_t)p * part_stride], b = p0[(int64_t)(p + 1) * part_stride];
        const float c = p0[(int64_t)(p + 2) * part_stride], d = p0[(int64_t)(p + 3) * part_stride];
        s += a; s += b; s += c; s += d;
    }
    for (; p < splits; ++p) s += p0[(int64_t)p * part_stride];
    tn_store(e, s, K, N, dual, C, C2, ldc, colsum_out);
}

// The same sum for partials whose stride allows 16-byte loads: a workgroup owns 64 elements,
// 16 groups of threads each add a contiguous range of splits in ascending order, and the 16
// group sums are then added in ascending order: a fixed association, so still deterministic.
__device__ __forceinline__ void tn_reduce_vec_block(uint32_t block, const float* __restrict__ part, int splits, int K, int N,
                                                            int64_t part_stride, float* __restrict__ C, int64_t ldc,
                                                            float* __restrict__ colsum_out, int dual, float* __restrict__ C2,
                                                            int64_t total) {           // total: a multiple of 4
    __shared__ float4 red[16][16];
    const int c = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int64_t e = ((int64_t)block * 16 + c) * 4;
    const int per = (splits + 15) / 16;
    const int p_begin = grp * per, p_end = p_begin + per < splits ? p_begin + per : splits;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (e < total) {
        const float* p0 = part + e;
        int p = p_begin;
        for (; p + 4 <= p_end; p += 4) {
            const float4 a = *reinterpret_cast<const float4*>(p0 + (int64_t)p * part_stride);
            const float4 b = *reinterpret_cast<const float4*>(p0 + (int64_t)(p + 1) * part_stride);
            const float4 c4 = *reinterpret_cast<const float4*>(p0 + (int64_t)(p + 2) * part_stride);
            const float4 d = *reinterpret_cast<const float4*>(p0 + (int64_t)(p + 3) * part_stride);
            s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w;
            s.x += b.x; s.y += b.y; s.z += b.z; s.w += b.w;
            s.x += c4.x; s.y += c4.y; s.z += c4.z; s.w += c4.w;
            s.x += d.x; s.y += d.y; s.z += d.z; s.w += d.w;
        }
        for (; p < p_end; ++p) {
            const float4 a = *reinterpret_cast<const float4*>(p0 + (int64_t)p * part_stride);
            s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w;
        }
    }
    red[grp][c] = s;
    __syncthreads();
    if (grp == 0 && e < total) {
        float4 t = red[0][c];
        for (int u = 1; u < 16; ++u) { const float4 v = red[u][c]; t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w; }
        const float tv[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) tn_store(e + q, tv[q], K, N, dual, C, C2, ldc, colsum_out);
    }
}

// Scalar variant of the same scheme for strides that rule out 16-byte loads: a workgroup owns
// 64 elements, 4 groups of threads each add a contiguous quarter of the splits in ascending
// order, the 4 group sums are added in ascending order.
__device__ __forceinline__ void tn_reduce_4way_block(uint32_t block, const float* __restrict__ part, int splits, int K, int N,
                                                             int64_t part_stride, float* __restrict__ C, int64_t ldc,
                                                             float* __restrict__ colsum_out, int dual, float* __restrict__ C2,
                                                             int64_t total) {
    __shared__ float red[4][64];
    const int c = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int64_t e = (int64_t)block * 64 + c;
    const int per = (splits + 3) / 4;
    const int p_begin = grp * per, p_end = p_begin + per < splits ? p_begin + per : splits;
    float s = 0.f;
    if (e < total) {
        const float* p0 = part + e;
        int p = p_begin;
        for (; p + 4 <= p_end; p += 4) {
            const float a = p0[(int64_t)p * part_stride], b = p0[(int64_t)(p + 1) * part_stride];
            const float c2 = p0[(int64_t)(p + 2) * part_stride], d = p0[(int64_t)(p + 3) * part_stride];
            s += a; s += b; s += c2; s += d;
        }
        for (; p < p_end; ++p) s += p0[(int64_t)p * part_stride];
    }
    red[grp][c] = s;
    __syncthreads();
    if (grp == 0 && e < total) {
        const float t = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
        tn_store(e, t, K, N, dual, C, C2, ldc, colsum_out);
    }
}

// out[c] = sum_b part[b][c]: 8 columns per workgroup, 32 lanes per column take the blocks
// b = j, j + 32, ... and are added in lane order.
__device__ __forceinline__ void colsum_final_block(uint32_t block, const float* __restrict__ part, int64_t blocks, int N,
                                                           float* __restrict__ out) {
    __shared__ float red[32][8];
    const int cl = threadIdx.x & 7, j = threadIdx.x >> 3;
    const int c = block * 8 + cl;
    float s = 0.f;
    if (c < N) {
        int64_t b = j;
        for (; b + 7 * 32 < blocks; b += 8 * 32) {      // eight loads in flight, added in the same order (eight sums over 4096 blocks in the residual step: 59.46 -> 59.22 ms)
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = part[(b + 32 * q) * N + c];
#pragma unroll
            for (int q = 0; q < 8; ++q) s += v[q];
        }
        for (; b < blocks; b += 32) s += part[b * N + c];
    }
    red[j][cl] = s;
    __syncthreads();
    if (j == 0 && c < N) {
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < 32; ++q) t += red[q][cl];
        out[c] = t;
    }
}

}  // namespace grp
