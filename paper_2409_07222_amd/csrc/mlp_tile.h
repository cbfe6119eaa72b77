// Device pieces of the network kernels that keep a tile of rows in LDS through
// several layers (the forward pass, the training pass, the learned walk's step).
#pragma once
#include "labs_internal.h"

#include <type_traits>

namespace labsdev {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// GELU, tanh form (Hendrycks and Gimpel 2016), and its derivative.
__device__ __forceinline__ float gelu_f(float x) {
    const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
    return 0.5f * x * (1.0f + tanhf(u));
}
__device__ __forceinline__ float gelu_grad_f(float x) {
    const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
    const float t = tanhf(u);
    const float du = 0.7978845608028654f * (1.0f + 3.0f * 0.044715f * x * x);
    return 0.5f * (1.0f + t) + 0.5f * x * (1.0f - t * t) * du;
}

// The feature of lag 2m, bf16(c / len), len = L - 2m odd, |c| <= len < 1024, from the
// hardware reciprocal: a quotient other than 0 and +-1 (exact here too) is at least
// 1 / (512 len) of itself away from every midpoint of two bf16 values (nine bits), and
// the product errs by less than 2^-22.
__device__ __forceinline__ float corr_scale(int L, int m) { return __builtin_amdgcn_rcpf((float)(L - 2 * m)); }
__device__ __forceinline__ uint16_t corr_feature(int c, float scale) { return f2bf((float)c * scale); }

// Two bf16 values, round to nearest even, the first in the low half.
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

// bf16(gelu_f(x)) of four values.  x (1 - 1 / (1 + e^{2u})) from the hardware exponential
// and reciprocal lies within 1e-6 |x| of gelu_f's value (both are within 5e-7 |x| of the
// true one: tanhf and the sum 1 + tanh err by a few 2^-24, the exponential by
// 2^-23 + |2u| 2^-22 of its value, which the slope of 1 / (1 + e) makes at most 2^-23);
// where the two ends of that interval round to the same bf16, so does gelu_f's.  The few
// others (about one value in a thousand), infinities and NaN take gelu_f itself, which
// branches per value and leaves no two of them in flight.
__device__ __forceinline__ void gelu_bf16(const float (&x)[4], uint32_t (&h)[2]) {
    uint32_t far = 0;
    float lo[4], hi[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        // 2 u log2(e) = x (2.3022082 + 0.10294324 x^2)
        const float w = x[j] * fmaf(0.10294324f, x[j] * x[j], 2.3022082f);
        const float q = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(w));
        const float r = fmaf(-x[j], q, x[j]);
        lo[j] = fmaf(fabsf(x[j]), -1e-6f, r);
        hi[j] = fmaf(fabsf(x[j]), 1e-6f, r);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        h[j] = f2bf2(lo[2 * j], lo[2 * j + 1]);
        far |= h[j] ^ f2bf2(hi[2 * j], hi[2 * j + 1]);
    }
    if (far || !(fabsf(x[0] + x[1] + x[2] + x[3]) < 1e30f)) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            h[j] = f2bf(gelu_f(x[2 * j])) | ((uint32_t)f2bf(gelu_f(x[2 * j + 1])) << 16);
    }
}

// Adam (Kingma and Ba 2015) of parameter i, FP32 masters; every operation rounded
// separately (contraction into FMAs is switched off) so that a float32 host computation
// in the same order matches bit for bit.
__device__ __forceinline__ void adam_update(int64_t i, float g, float* __restrict__ P, uint16_t* __restrict__ Pb,
                                            float* __restrict__ M, float* __restrict__ V, float b1, float omb1,
                                            float b2, float omb2, float bc1, float bc2, float lr, float eps) {
#pragma clang fp contract(off)
    const float m = b1 * M[i] + omb1 * g;
    const float v = b2 * V[i] + (omb2 * g) * g;
    M[i] = m;
    V[i] = v;
    const float mh = m / bc1, vh = v / bc2;
    const float p = P[i] - (lr * mh) / (sqrtf(vh) + eps);   // sqrtf and '/' are correctly rounded
    P[i] = p;
    Pb[i] = f2bf(p);
}

// LDS of a workgroup.  The kernels that take more than the default limit have it raised to
// this, less their static part, and not to what a call needs: the limit is the process's,
// so another thread's smaller network would lower it before this one's launch.
constexpr int kLdsBytes = 160 * 1024;

// Chunks of rows of a bias gradient's sum.
constexpr int kColChunks = 64;

// Splits of a weight gradient's sum over K rows when its output has `tiles` 64 x 64 tiles,
// and the rows of each: enough for two workgroups a CU, at least 256 rows.
constexpr int kMaxSplits = 16;
inline int product_splits(long long tiles, int K, int* chunk) {
    int splits = 1;
    *chunk = (K + 31) / 32 * 32;
    if (tiles < 512 && K >= 2 * 256) {
        splits = (int)((512 + tiles - 1) / tiles);
        if (splits > kMaxSplits) splits = kMaxSplits;
        if (splits > K / 256) splits = K / 256;
        *chunk = ((K + splits - 1) / splits + 31) / 32 * 32;
        splits = (K + *chunk - 1) / *chunk;
    }
    return splits;
}

// Zeroes the elements of an 8-element bf16 chunk that start at index k and reach K.
__device__ __forceinline__ uint4 mask_tail(uint4 v, int k, int K) {
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (k + 2 * j >= K) w[j] = 0;
        else if (k + 2 * j + 1 >= K) w[j] &= 0xFFFFu;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// Weights in fragment order: of column tile t (16 rows of W) and step kc (32 columns),
// lane l's 16 bytes are W[16 t + l % 16][32 kc + 8 (l / 16) .. + 7], so a wave's operand is
// one contiguous kilobyte (rows of W themselves would touch 64 cache lines).  The tiles of
// a step follow one another, as the waves of a workgroup read them.
__host__ __device__ inline int64_t packed_elems(int ncols, int K) {
    return (int64_t)((ncols + 15) / 16) * ((K + 31) / 32) * 512;
}

// Chunk i (8 elements) of a matrix in fragment order: element (row, k) at W[row * ld + k],
// or with TR at W[k * ld + row].
template <bool TR>
__device__ __forceinline__ void pack_chunk(uint16_t* __restrict__ out, const uint16_t* __restrict__ W, int rows, int K,
                                           int ld, int64_t i) {
    const int tiles = (rows + 15) / 16;
    const int lane = (int)(i & 63), t = (int)((i >> 6) % tiles), kc = (int)((i >> 6) / tiles);
    const int row = 16 * t + (lane & 15), k = 32 * kc + 8 * (lane >> 4);
    uint4 v = make_uint4(0, 0, 0, 0);
    if (row < rows && k < K) {
        if constexpr (TR) {
            uint32_t w[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t a = k + 2 * q < K ? W[(int64_t)(k + 2 * q) * ld + row] : 0u;
                const uint32_t b = k + 2 * q + 1 < K ? W[(int64_t)(k + 2 * q + 1) * ld + row] : 0u;
                w[q] = a | (b << 16);
            }
            v = make_uint4(w[0], w[1], w[2], w[3]);
        } else {
            v = *(const uint4*)(W + (int64_t)row * ld + k);
            if (k + 8 > K) v = mask_tail(v, k, K);
        }
    }
    ((uint4*)out)[i] = v;
}

// A workgroup is 8 waves over 16 MR rows; a wave takes every row and two column tiles at
// a time, so each weight is read once a workgroup and each fragment of the rows feeds
// two products.
constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kTilePF = 4;

// acc[c][r] = (16 columns of tile t[c]) (tile rows 16 r .. + 15)^T over the steps of K, in
// order: the layer's columns are the matrix product's rows, so a lane ends with four
// consecutive columns 4 (lane / 16) .. + 3 of row lane % 16.  A: the rows in LDS, stride
// sa bytes.  WP: packed weights, nch steps of `tiles` tiles, read kTilePF steps ahead (at
// the end the last step again); the rows are read one step ahead, at the end past them.
template <int MR, int CT>
__device__ __forceinline__ void tile_product(f32x4 (&acc)[CT][MR], const char* A, int sa, const uint16_t* __restrict__ WP,
                                             const int (&t)[CT], int tiles, int nch) {
    constexpr int PF = kTilePF;
    const int lane = threadIdx.x & 63;
    const uint4* wp[CT];     // wave-uniform; the lane joins at the load
#pragma unroll
    for (int c = 0; c < CT; ++c) wp[c] = (const uint4*)(WP) + t[c] * 64;
    const char* ap = A + (lane & 15) * sa + 16 * (lane >> 4);
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < MR; ++r) acc[c][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto rows = [&](int kc, bf16x8 (&a)[MR]) {
#pragma unroll
        for (int r = 0; r < MR; ++r) a[r] = *(const bf16x8*)(ap + 16 * r * sa + 64 * kc);
    };
    auto multiply = [&](const uint4 (&w)[CT], const bf16x8 (&a)[MR]) {
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int r = 0; r < MR; ++r)
                acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[c]), a[r], acc[c][r], 0,
                                                                   0, 0);
    };
    uint4 q[PF][CT];
    bf16x8 a[2][MR];
    auto fetch = [&](int kc, uint4 (&d)[CT]) {
#pragma unroll
        for (int c = 0; c < CT; ++c) d[c] = wp[c][64 * tiles * min(kc, nch - 1) + lane];
    };
    // The scheduling barriers keep the loads where they are written: left alone, the
    // compiler moves them next to their uses and every step waits for the L2.
#pragma unroll
    for (int d = 0; d < PF; ++d) fetch(d, q[d]);
    rows(0, a[0]);
    int kc = 0;
    for (; kc + PF <= nch; kc += PF) {
#pragma unroll
        for (int d = 0; d < PF; ++d) {
            rows(kc + d + 1, a[(d + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            multiply(q[d], a[d & 1]);
            __builtin_amdgcn_sched_barrier(0);
            fetch(kc + d + PF, q[d]);
        }
    }
#pragma unroll
    for (int d = 0; d < PF - 1; ++d)
        if (kc + d < nch) {
            rows(kc + d + 1, a[(d + 1) & 1]);
            multiply(q[d], a[d & 1]);
        }
}

// Every column of a layer for the workgroup's rows: store(col, row, bias, v) takes four
// consecutive columns of one row and their biases.
template <int MR, int NW = kTileWaves, class Store>
__device__ __forceinline__ void tile_layer(const char* A, int sa, const uint16_t* __restrict__ WP,
                                           const float* __restrict__ bias, int ncols, int K, Store store) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles = (ncols + 15) >> 4, nch = (K + 31) >> 5;
    auto run = [&](auto ctc, const int t0) {
        constexpr int CT = decltype(ctc)::value;
        f32x4 acc[CT][MR];
        int t[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) t[c] = t0 + NW * c;
        float bv[CT][4];
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) bv[c][j] = bias[min(16 * t[c] + 4 * (lane >> 4) + j, ncols - 1)];
        tile_product<MR, CT>(acc, A, sa, WP, t, tiles, nch);
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int r = 0; r < MR; ++r) store(16 * t[c] + 4 * (lane >> 4), 16 * r + (lane & 15), bv[c], acc[c][r]);
    };
    for (int t0 = wave; t0 < tiles; t0 += 2 * NW) {
        if (t0 + NW < tiles) run(std::integral_constant<int, 2>(), t0);
        else run(std::integral_constant<int, 1>(), t0);
    }
}

// bf16(gelu(v + bias)) of four columns into the next layer's LDS rows (the columns of a
// hidden layer are a multiple of 16).
__device__ __forceinline__ void store_hidden(char* H, int sh, const float (&bias)[4], int col, int row, f32x4 v) {
    float x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = v[j] + bias[j];
    uint32_t h[2];
    gelu_bf16(x, h);
    *(uint2*)(H + row * sh + 2 * col) = make_uint2(h[0], h[1]);
}

// Row strides in bytes of an LDS tile of `ld` bf16 columns: 16 bytes more than the row,
// so the 16 rows of a fragment start in distinct banks.
__host__ __device__ inline int tile_stride(int ld) { return 2 * ld + 16; }

}  // namespace labsdev
