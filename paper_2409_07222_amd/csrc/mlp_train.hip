// Gradients and training step of the learned proposal for hidden layers of up to 256
// units, in four launches:
//   k_pack_train   the weights, and the two transposes the backward pass needs, in
//                  fragment order;
//   k_train_rows   16 rows through forward, cross-entropy and backward in one workgroup;
//                  its operands of the weight gradients leave in the fragment order of
//                  products over the batch;
//   k_weight_grads the three batch products, split over the batch, the columns' sums over
//                  64 chunks of rows, and the loss;
//   k_grads_final  the sums over the splits and chunks, and Adam.
// Every sum has the order of the separate products' path (mlp.hip), so gradients do not
// depend on which of the two computes them.
// As some twenty launches of products, column sums, split sums and elementwise passes the
// step took 189 us at L = 501, hidden 256, n = 4,096; now 56 (packing 5, rows 29, batch
// products 16, sums and Adam 9).
#include "labs_internal.h"

#include <cmath>

#include "mlp_tile.h"

namespace labsdev {

namespace {

constexpr int kRows = 16;                     // rows of a workgroup of k_train_rows
constexpr int kRowWaves = 16, kRowThreads = 64 * kRowWaves;   // a wave a row, a column tile
constexpr int kSeqWords = 36;                 // packed words of a row with zeros behind
constexpr int kGradTile = 64;                 // tile edge of a weight gradient product

struct TrainArgs {
    labs_mlp_layout y;
    int n, ksteps;                            // rows; batch steps of 32 rows
    int splits[3], per[3];                    // of each weight gradient: splits, steps a split
    const float* P;
    const uint16_t* Pb;
    const uint32_t* seqs;                     // features' source, or X
    const uint16_t* X;
    const uint32_t* mask;
    const int32_t* labels;
    uint16_t *W1, *W2, *W3, *W2T, *W3T;       // packed
    uint16_t *FX, *F1, *F2, *FZ, *FD2, *FD1;  // columns of X, h1, h2, dz, da2, da1 over the batch
    float* D;                                 // [n][bias_ld]: da1, da2, dz in FP32
    float* bias_part;                         // [kColChunks][bias_ld]: their column sums
    float* rowloss;
    float* part;                              // [most splits][n_params]
    float* loss;
};

__host__ __device__ inline int bias_ld(const labs_mlp_layout& y) { return (2 * y.hidden + y.d_out + 3) & ~3; }

// ------------------------------------------------------------------ packing
__global__ __launch_bounds__(256) void k_pack_train(TrainArgs T) {
    const labs_mlp_layout& y = T.y;
    const int H = y.hidden;
    const int64_t n1 = packed_elems(H, y.d_in) / 8, n2 = packed_elems(H, H) / 8, n3 = packed_elems(y.d_out, H) / 8,
                  n4 = packed_elems(H, y.d_out) / 8;
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n1) return pack_chunk<false>(T.W1, T.Pb + y.off_W1, H, y.d_in, y.ld_in, i);
    if ((i -= n1) < n2) return pack_chunk<false>(T.W2, T.Pb + y.off_W2, H, H, H, i);
    if ((i -= n2) < n3) return pack_chunk<false>(T.W3, T.Pb + y.off_W3, y.d_out, H, H, i);
    if ((i -= n3) < n2) return pack_chunk<true>(T.W2T, T.Pb + y.off_W2, H, H, H, i);
    if ((i -= n2) < n4) pack_chunk<true>(T.W3T, T.Pb + y.off_W3, H, y.d_out, H, i);
}

// ------------------------------------------------------------------ rows
// Byte offsets of the LDS areas of a workgroup: rows of X, h1 (later da1), h2 (later da2),
// the logits, dz in bf16; one step of reads past the end.
struct RowsLds {
    int x, h1, h2, z, dz, bytes, sx, sh, sz, sd;
};
__host__ __device__ inline RowsLds rows_lds(const labs_mlp_layout& y) {
    RowsLds o;
    o.sx = tile_stride(y.ld_in);
    o.sh = tile_stride(y.hidden);
    o.sz = 4 * y.ld_out + 16;
    o.sd = tile_stride(y.ld_out);
    o.x = 0;
    o.h1 = o.x + kRows * o.sx;
    o.h2 = o.h1 + kRows * o.sh;
    o.z = o.h2 + kRows * o.sh;
    o.dz = o.z + kRows * o.sz;
    o.bytes = o.dz + kRows * o.sd + 64;
    return o;
}

// The columns of 16 LDS rows into the fragment order of a product over the batch: 8 rows
// of one column are 16 bytes, workgroups of even and odd index fill the two halves of a
// step's fragments.
__device__ __forceinline__ void write_columns(uint16_t* __restrict__ F, const char* A, int sa, int ncols) {
    const int tiles = (ncols + 15) >> 4, kc = blockIdx.x >> 1;
    for (int it = threadIdx.x; it < 32 * tiles; it += kRowThreads) {
        const int t = it >> 5, l = it & 31;
        const char* a = A + 8 * (l >> 4) * sa + 2 * (16 * t + (l & 15));
        uint32_t w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            w[q] = *(const uint16_t*)(a + 2 * q * sa) | ((uint32_t)*(const uint16_t*)(a + (2 * q + 1) * sa) << 16);
        *(uint4*)(F + (((int64_t)kc * tiles + t) * 64 + 32 * (blockIdx.x & 1) + l) * 8) =
            make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// A wave's column tile of a product with up to 256 columns.
__device__ __forceinline__ void tile_one(f32x4& acc, const char* A, int sa, const uint16_t* WP, int ncols, int K) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles = ncols >> 4, nch = (K + 31) >> 5;
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
    if (wave < tiles) {
        f32x4 v[1][1];
        const int t[1] = {wave};
        tile_product<1, 1>(v, A, sa, WP, t, tiles, nch);
        acc = v[0][0];
    }
}

// Hidden layer: h = gelu(v + b) as bf16 into LDS, gelu'(v + b) kept in FP32 registers
// (the backward product of the layer ends in the same lanes).
__device__ __forceinline__ void hidden_forward(f32x4& grad, const f32x4& acc, const float* bias, char* H,
                                               int sh, int ncols) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = 16 * wave + 4 * (lane >> 4);
    if (col >= ncols) return;
    uint32_t h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float x = acc[j] + bias[col + j];
        h[j] = f2bf(gelu_f(x));
        grad[j] = gelu_grad_f(x);
    }
    *(uint2*)(H + (lane & 15) * sh + 2 * col) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
}

// d = dh gelu': FP32 rows to memory, bf16 rows into LDS.
__device__ __forceinline__ void hidden_backward(const f32x4& dh, const f32x4& grad, float* D, int ldd, int rows,
                                                char* H, int sh, int ncols) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane & 15;
    const int col = 16 * wave + 4 * (lane >> 4);
    if (col >= ncols) return;
    float d[4];
    uint32_t h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        d[j] = dh[j] * grad[j];
        h[j] = f2bf(d[j]);
    }
    *(uint2*)(H + row * sh + 2 * col) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    if (row < rows) *(float4*)(D + (int64_t)row * ldd + col) = make_float4(d[0], d[1], d[2], d[3]);
}

__device__ __forceinline__ float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// 16 rows, so the training batch (4,096) is one workgroup a CU; bound by the latency of its
// chain of five products with a barrier each, so every wave takes one column tile (29 us;
// eight waves with two tiles 36, and of those the lags' popcounts, GELU and the columns'
// writes 1 to 3 each; weights read 8 or 12 steps ahead no less).
template <bool SEQ>
__global__ __launch_bounds__(kRowThreads) void k_train_rows(TrainArgs T) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ uint32_t sw[kRows][kSeqWords];
    const labs_mlp_layout& y = T.y;
    const RowsLds o = rows_lds(y);
    char *const X = lds + o.x, *const H1 = lds + o.h1, *const H2 = lds + o.h2, *const Z = lds + o.z,
         *const DZ = lds + o.dz;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m0 = kRows * blockIdx.x;
    const int ldd = bias_ld(y), rows = T.n - m0;
    float* const D = T.D + (int64_t)m0 * ldd;

    // ---- features; rows past n repeat the last one, and have a zero dz
#pragma unroll
    for (int i = 0; i < kRows / kRowWaves; ++i) {
        const int row = wave + kRowWaves * i;
        const int64_t r = min(m0 + row, T.n - 1);
        char* const x = X + row * o.sx;
        if constexpr (SEQ) {
            const int L = y.L, k = y.k, W = (L + 31) >> 5;
            if (lane < kSeqWords) sw[row][lane] = lane < W ? T.seqs[r * W + lane] : 0u;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const uint32_t* u = sw[row];
            for (int e = lane; e < k; e += 64) {
                const uint32_t b = ~u[e >> 4] << (2 * (e & 15));
                ((uint32_t*)x)[e] = 0x3F803F80u | ((b >> 16) & 0x8000u) | ((b & 0x40000000u) << 1);
            }
            if (lane == 0) ((uint16_t*)x)[L - 1] = packed_bit(u, L) ? 0x3F80 : 0xBF80;
            for (int e = lane; e < y.ld_in - L; e += 64)
                ((uint16_t*)x)[L + e] =
                    e < k ? corr_feature(packed_corr(u, L, 2 * e + 2), corr_scale(L, e + 1)) : (uint16_t)0;
        } else {
            for (int c = lane; c < y.ld_in / 8; c += 64) {
                uint4 v = *(const uint4*)(T.X + r * y.ld_in + 8 * c);
                if (8 * c + 8 > y.d_in) v = mask_tail(v, 8 * c, y.d_in);
                *(uint4*)(x + 16 * c) = v;
            }
        }
    }
    __syncthreads();

    // ---- forward
    f32x4 acc, g1, g2;
    tile_one(acc, X, o.sx, T.W1, y.hidden, y.d_in);
    hidden_forward(g1, acc, T.P + y.off_b1, H1, o.sh, y.hidden);
    write_columns(T.FX, X, o.sx, y.d_in);
    __syncthreads();
    tile_one(acc, H1, o.sh, T.W2, y.hidden, y.hidden);
    hidden_forward(g2, acc, T.P + y.off_b2, H2, o.sh, y.hidden);
    write_columns(T.F1, H1, o.sh, y.hidden);
    __syncthreads();
    tile_layer<1, kRowWaves>(H2, o.sh, T.W3, T.P + y.off_b3, y.d_out, y.hidden,
                  [&](int col, int row, const float (&b)[4], f32x4 v) {
                      *(float4*)(Z + row * o.sz + 4 * col) =
                          make_float4(v[0] + b[0], v[1] + b[1], v[2] + b[2], v[3] + b[3]);
                  });
    write_columns(T.F2, H2, o.sh, y.hidden);
    __syncthreads();

    // ---- cross-entropy over the admissible logits (mask bit set, or the label):
    // loss = logsumexp - z_label, dz = (softmax - onehot) / n there, 0 elsewhere
    const float inv_n = 1.0f / (float)T.n;
#pragma unroll
    for (int i = 0; i < kRows / kRowWaves; ++i) {
        const int row = wave + kRowWaves * i, r = m0 + row;
        const bool in = r < T.n;
        const float* const z = (const float*)(Z + row * o.sz);
        uint16_t* const dz = (uint16_t*)(DZ + row * o.sd);
        const int lab = in ? T.labels[r] : 0;
        const uint32_t* const mr = T.mask + (int64_t)(in ? r : 0) * y.mask_words;
        constexpr int PER = 8;                // d_out <= 512
        float zv[PER];
        bool ok[PER];
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            const int j = lane + 64 * c;
            ok[c] = j < y.d_out && (j == lab || ((mr[j >> 5] >> (j & 31)) & 1));
            zv[c] = ok[c] ? z[j] : -INFINITY;
            mx = fmaxf(mx, zv[c]);
        }
        const float zl = lab >= 0 && lab < y.d_out ? z[lab] : 0.f;
        mx = wave_max(mx);
        float se = 0.f;
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            zv[c] = ok[c] ? expf(zv[c] - mx) : 0.f;
            se += zv[c];
        }
        se = wave_sum(se);
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            const int j = lane + 64 * c;
            if (j >= y.ld_out) break;
            const float d = in && ok[c] ? (zv[c] / se - (j == lab ? 1.f : 0.f)) * inv_n : 0.f;
            dz[j] = f2bf(d);
            if (in && j < y.d_out) D[(int64_t)row * ldd + 2 * y.hidden + j] = d;
        }
        if (in && lane == 0) T.rowloss[r] = logf(se) + mx - zl;
    }
    __syncthreads();

    // ---- backward
    tile_one(acc, DZ, o.sd, T.W3T, y.hidden, y.d_out);
    hidden_backward(acc, g2, D + y.hidden, ldd, rows, H2, o.sh, y.hidden);
    write_columns(T.FZ, DZ, o.sd, y.d_out);
    __syncthreads();
    tile_one(acc, H2, o.sh, T.W2T, y.hidden, y.hidden);
    hidden_backward(acc, g1, D, ldd, rows, H1, o.sh, y.hidden);
    write_columns(T.FD2, H2, o.sh, y.hidden);
    __syncthreads();
    write_columns(T.FD1, H1, o.sh, y.hidden);
}

// ------------------------------------------------------------------ batch products
// A wave takes a 64 x 64 tile of one weight gradient over one split of the batch; a
// workgroup four splits of a tile.  Operands come from memory in fragment order without
// LDS, 16 products a step for 8 KB, kGradPF steps ahead: a wave a SIMD, bound by those
// loads' latency.  Behind the tiles, blocks of 64 columns and one chunk of rows for the
// bias gradients, and one for the loss.
constexpr int kGradPF = 3;

struct GradTile {
    const uint16_t *A, *B;      // columns of the layer's input, of its d
    int M, N, m0, n0, ld, which, split0;
    int64_t off;
};

__host__ __device__ inline int grad_blocks(const labs_mlp_layout& y, const int (&splits)[3]) {
    const int th = (y.hidden + 63) / 64, t1 = (y.d_in + 63) / 64, t3 = (y.d_out + 63) / 64;
    return t1 * th * ((splits[0] + 3) / 4) + th * th * ((splits[1] + 3) / 4) + th * t3 * ((splits[2] + 3) / 4);
}

__device__ __forceinline__ GradTile grad_tile(const TrainArgs& T, int b) {
    const labs_mlp_layout& y = T.y;
    const int th = (y.hidden + 63) / 64, t1 = (y.d_in + 63) / 64, t3 = (y.d_out + 63) / 64;
    const int q0 = (T.splits[0] + 3) / 4, q1 = (T.splits[1] + 3) / 4, q2 = (T.splits[2] + 3) / 4;
    GradTile g;
    int t, tn, q;
    if (b < t1 * th * q0) {
        g = GradTile{T.FX, T.FD1, y.d_in, y.hidden, 0, 0, y.ld_in, 0, 0, y.off_W1};
        t = b / q0, tn = th, q = b % q0;
    } else if ((b -= t1 * th * q0) < th * th * q1) {
        g = GradTile{T.F1, T.FD2, y.hidden, y.hidden, 0, 0, y.hidden, 1, 0, y.off_W2};
        t = b / q1, tn = th, q = b % q1;
    } else {
        b -= th * th * q1;
        g = GradTile{T.F2, T.FZ, y.hidden, y.d_out, 0, 0, y.hidden, 2, 0, y.off_W3};
        t = b / q2, tn = t3, q = b % q2;
    }
    g.m0 = kGradTile * (t / tn);
    g.n0 = kGradTile * (t % tn);
    g.split0 = 4 * q;
    return g;
}

__global__ __launch_bounds__(256, 1) void k_weight_grads(TrainArgs T, int blocks) {
    __shared__ float red[4][64];
    const labs_mlp_layout& y = T.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int b = (int)blockIdx.x - blocks;
    if (b >= 0) {
        const int cols = 2 * y.hidden + y.d_out, ld = bias_ld(y), cb = (cols + 63) / 64;
        float s = 0.f;
        if (b < cb * kColChunks) {
            const int c = 64 * (b % cb) + lane, chunk = b / cb;
            const int per = (T.n + kColChunks - 1) / kColChunks, r0 = chunk * per, r1 = min(r0 + per, T.n);
            if (c < cols) {
#pragma unroll 4
                for (int r = r0 + wave; r < r1; r += 4) s += T.D[(int64_t)r * ld + c];
            }
            red[wave][lane] = s;
            __syncthreads();
            if (wave == 0 && c < cols)
                T.bias_part[(int64_t)chunk * ld + c] = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
        } else {
            float* const part = &red[0][0];
            const int per = (T.n + 255) / 256, r0 = threadIdx.x * per, r1 = min(r0 + per, T.n);
            for (int r = r0; r < r1; ++r) s += T.rowloss[r];
            part[threadIdx.x] = s;
            __syncthreads();
            for (int w = 128; w > 0; w >>= 1) {
                if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
                __syncthreads();
            }
            if (threadIdx.x == 0) *T.loss = part[0] / (float)T.n;
        }
        return;
    }
    const GradTile g = grad_tile(T, blockIdx.x);
    const int split = g.split0 + wave;
    if (split >= T.splits[g.which]) return;
    const int ta = (g.M + 15) / 16, tb = (g.N + 15) / 16;
    const int k0 = split * T.per[g.which], k1 = min(k0 + T.per[g.which], T.ksteps);
    const uint4 *pa[4], *pb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // tiles past the matrix repeat its last one and are not stored
        pa[i] = (const uint4*)g.A + (int64_t)min(g.m0 / 16 + i, ta - 1) * 64 + lane;
        pb[i] = (const uint4*)g.B + (int64_t)min(g.n0 / 16 + i, tb - 1) * 64 + lane;
    }
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 fa[kGradPF][4], fb[kGradPF][4];
    auto fetch = [&](int k, int d) {
        const int64_t kk = min(k, k1 - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            fa[d][i] = pa[i][kk * ta * 64];
            fb[d][i] = pb[i][kk * tb * 64];
        }
    };
    auto multiply = [&](int d) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[d][i]),
                                                                   __builtin_bit_cast(bf16x8, fb[d][j]), acc[i][j], 0, 0,
                                                                   0);
    };
#pragma unroll
    for (int d = 0; d < kGradPF; ++d) fetch(k0 + d, d);
    for (int k = k0; k < k1; k += kGradPF) {
#pragma unroll
        for (int d = 0; d < kGradPF; ++d) {
            __builtin_amdgcn_sched_barrier(0);
            if (k + d < k1) multiply(d);
            __builtin_amdgcn_sched_barrier(0);
            fetch(k + d + kGradPF, d);
        }
    }
    // element (m, n): m = 16 i + 4 (lane / 16) + r, n = 16 j + lane % 16
    float* const out = T.part + (int64_t)split * y.n_params + g.off;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = g.n0 + 16 * j + (lane & 15);
        if (n >= g.N) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = g.m0 + 16 * i + 4 * (lane >> 4);
            // a row's end is padded to 64 columns, so whole fours are written
            if (m < g.M) *(f32x4*)(out + (int64_t)n * g.ld + m) = acc[i][j];
        }
    }
}

// ------------------------------------------------------------------ sum of the splits, Adam
struct AdamArgs {
    float *P, *M, *V;
    uint16_t* Pb;
    float b1, omb1, b2, omb2, bc1, bc2, lr, eps;
};

// The caller's gradients need only be aligned for their elements.
struct __attribute__((packed, aligned(4))) FourGrads {
    float v[4];
};

// Gradient of four consecutive parameters (a region's start and row lengths are multiples
// of 64), zero in the pads; with ADAM also the update.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_grads_final(TrainArgs T, float* __restrict__ G, AdamArgs A) {
    const labs_mlp_layout& y = T.y;
    const int64_t i0 = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
    if (i0 >= y.n_params) return;
    const float* part = T.part + i0;           // parts to add, a stride apart
    int live = 4, parts;                       // parameters of the four
    int64_t stride = y.n_params;
    auto within = [&](int64_t v, int64_t end) { return (int)(v >= end ? 0 : end - v < 4 ? end - v : 4); };
    auto bias = [&](int64_t c) {
        part = T.bias_part + c;
        stride = bias_ld(y);
        parts = kColChunks;
    };
    if (i0 < y.off_b1) {
        live = within((int)i0 % y.ld_in, y.d_in);
        parts = T.splits[0];
    } else if (i0 < y.off_W2) {
        bias(i0 - y.off_b1);
    } else if (i0 < y.off_b2) {
        parts = T.splits[1];
    } else if (i0 < y.off_W3) {
        bias(i0 - y.off_b2 + y.hidden);
    } else if (i0 < y.off_b3) {
        live = within(i0 - y.off_W3, (int64_t)y.d_out * y.hidden);
        parts = T.splits[2];
    } else {
        live = within(i0 - y.off_b3, y.d_out);
        bias(i0 - y.off_b3 + 2 * y.hidden);
    }
    float g[4] = {0.f, 0.f, 0.f, 0.f};
    if (live > 0) {
#pragma unroll 8
        for (int s = 0; s < parts; ++s) {
            const float4 v = *(const float4*)(part + s * stride);
            g[0] += v.x;
            g[1] += v.y;
            g[2] += v.z;
            g[3] += v.w;
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (r >= live) g[r] = 0.f;
    *(FourGrads*)(G + i0) = FourGrads{{g[0], g[1], g[2], g[3]}};
    if constexpr (ADAM) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            adam_update(i0 + r, g[r], A.P, A.Pb, A.M, A.V, A.b1, A.omb1, A.b2, A.omb2, A.bc1, A.bc2, A.lr, A.eps);
    }
}

// The splits of the batch products, as the separate products choose them.
void split_batch(TrainArgs& T) {
    const int th = (T.y.hidden + 63) / 64, t1 = (T.y.d_in + 63) / 64, t3 = (T.y.d_out + 63) / 64;
    const int tiles[3] = {t1 * th, th * th, t3 * th};
    for (int q = 0; q < 3; ++q) {
        int chunk = 0;
        T.splits[q] = product_splits(tiles[q], T.n, &chunk);
        T.per[q] = chunk / 32;
    }
}

size_t carve_train(const labs_mlp_layout& y, int64_t n, void* ws, size_t wsb, TrainArgs* out) {
    Carve cv(ws, wsb);
    TrainArgs T{};
    T.y = y;
    T.n = (int)n;
    T.ksteps = (int)((n + 31) / 32);
    split_batch(T);
    const int H = y.hidden;
    T.W1 = cv.take<uint16_t>((size_t)packed_elems(H, y.d_in));
    T.W2 = cv.take<uint16_t>((size_t)packed_elems(H, H));
    T.W3 = cv.take<uint16_t>((size_t)packed_elems(y.d_out, H));
    T.W2T = cv.take<uint16_t>((size_t)packed_elems(H, H));
    T.W3T = cv.take<uint16_t>((size_t)packed_elems(H, y.d_out));
    const int64_t rows = 32 * (int64_t)T.ksteps;
    T.FX = cv.take<uint16_t>((size_t)packed_elems(y.d_in, 1) / 32 * rows);
    T.F1 = cv.take<uint16_t>((size_t)H * rows);
    T.F2 = cv.take<uint16_t>((size_t)H * rows);
    T.FZ = cv.take<uint16_t>((size_t)packed_elems(y.d_out, 1) / 32 * rows);
    T.FD2 = cv.take<uint16_t>((size_t)H * rows);
    T.FD1 = cv.take<uint16_t>((size_t)H * rows);
    T.D = cv.take<float>((size_t)n * bias_ld(y));
    T.bias_part = cv.take<float>((size_t)kColChunks * bias_ld(y));
    T.rowloss = cv.take<float>((size_t)n);
    // no more splits than this, which does not fall as n grows (the splits may)
    const int64_t most = n / 256 < 1 ? 1 : n / 256 < kMaxSplits ? n / 256 : kMaxSplits;
    T.part = cv.take<float>((size_t)most * y.n_params);
    if (out) {
        *out = T;
        if (!cv.ok() || !T.part) return 0;
    }
    return cv.used;
}

}  // namespace

size_t mlp_train_ws(const labs_mlp_layout& y, int64_t n) {
    return carve_train(y, n, nullptr, 0, nullptr) + 256;
}

labs_status mlp_train(const labs_mlp_layout& y, float* P, uint16_t* Pb, int64_t n, const uint32_t* seqs,
                      const uint16_t* X, const uint32_t* mask, const int32_t* labels, float* G, float* loss,
                      const MlpAdam* adam, void* ws, size_t wsb, hipStream_t st) {
    TrainArgs T;
    if (!carve_train(y, n, ws, wsb, &T)) return LABS_E_NOMEM;
    T.P = P;
    T.Pb = Pb;
    T.seqs = seqs;
    T.X = X;
    T.mask = mask;
    T.labels = labels;
    T.loss = loss;
    const int H = y.hidden;
    const int64_t chunks = (packed_elems(H, y.d_in) + 2 * packed_elems(H, H) + packed_elems(y.d_out, H) +
                            packed_elems(H, y.d_out)) / 8;
    hipLaunchKernelGGL(k_pack_train, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st, T);
    LABS_LAUNCHED("k_pack_train");
    const dim3 rows((unsigned)(2 * T.ksteps));
    const int lds = rows_lds(y).bytes;
    constexpr int kLimit = kLdsBytes - kRows * kSeqWords * (int)sizeof(uint32_t);
    if (seqs) {
        LABS_HIP(hipFuncSetAttribute((const void*)k_train_rows<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kLimit));
        hipLaunchKernelGGL(k_train_rows<true>, rows, dim3(kRowThreads), lds, st, T);
    } else {
        LABS_HIP(hipFuncSetAttribute((const void*)k_train_rows<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     kLimit));
        hipLaunchKernelGGL(k_train_rows<false>, rows, dim3(kRowThreads), lds, st, T);
    }
    LABS_LAUNCHED("k_train_rows");
    const int blocks = grad_blocks(y, T.splits);
    hipLaunchKernelGGL(k_weight_grads, dim3((unsigned)(blocks + (2 * H + y.d_out + 63) / 64 * kColChunks + 1)), dim3(256),
                       0, st, T, blocks);
    LABS_LAUNCHED("k_weight_grads");
    const dim3 grid((unsigned)((y.n_params / 4 + 255) / 256));
    if (adam) {
        const AdamArgs A{P, adam->M, adam->V, Pb, (float)adam->b1, (float)(1.0 - adam->b1), (float)adam->b2,
                         (float)(1.0 - adam->b2), (float)(1.0 - std::pow(adam->b1, (double)adam->t)),
                         (float)(1.0 - std::pow(adam->b2, (double)adam->t)), (float)adam->lr, (float)adam->eps};
        hipLaunchKernelGGL(k_grads_final<true>, grid, dim3(256), 0, st, T, G, A);
    } else {
        hipLaunchKernelGGL(k_grads_final<false>, grid, dim3(256), 0, st, T, G, AdamArgs{});
    }
    LABS_LAUNCHED("k_grads_final");
    return LABS_OK;
}

}  // namespace labsdev
