// Energies and exact neighbour energy changes (Sec. 1 definitions; the
// neighbourhoods of Algorithm 1 and Algorithm 2).
//
// One wavefront per sequence.  C_d is a popcount over the packed bits.  A flip of
// position a changes C_d by -2 s_a (s_{a+d} + s_{a-d}), so
//   dE(a) = -4 s_a H_a + 4 (L - 1) + 8 P_a,   H_a = sum_{i != a} s_i C_{|i-a|},
//   P_a = sum_{d >= 1} s_{a+d} s_{a-d}
// with elements outside the sequence zero.  H is a Toeplitz product on the matrix cores,
// P another popcount (the sequence against its reverse).  For a pair {a, b = L + 1 - a}
// with gap g = b - a, s = s_a s_b and V = sum_i s_i s_{L+1-i}, expanding the square gives
//   dE = dE(a) + dE(b) + 16 s C_g + 8 s V - 32 - 16 (s_b s_{a-g} + s_a s_{b+g}).
#include "labs_internal.h"

namespace labsdev {

namespace {

constexpr int kWaves = 4;    // sequences a workgroup
constexpr int kMaxW = 32;

// Popcounts of the lags are the bound.  4,096 sequences at L = 501 with C: byte loops over
// LDS 222 us, now 9.6.
__global__ __launch_bounds__(64 * kWaves) void k_energy(int L, int64_t n, const uint32_t* __restrict__ seqs,
                                                        int32_t* __restrict__ E, int32_t* __restrict__ C) {
    __shared__ uint32_t sw[kWaves][kMaxW + 2];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t j = (int64_t)blockIdx.x * kWaves + wv;
    const int W = (L + 31) >> 5;
    if (lane < kMaxW + 2) sw[wv][lane] = j < n && lane < W ? seqs[j * W + lane] : 0u;
    __syncthreads();
    if (j >= n) return;
    int e = 0;
    for (int d = 1 + lane; d <= L - 1; d += 64) {
        const int c = packed_corr(sw[wv], L, d);
        if (C) C[j * (L - 1) + (d - 1)] = c;
        e += c * c;
    }
    e = __ockl_wfred_add_i32(e);
    if (lane == 0) E[j] = e;
}

// sum_{i < len} u_i v_{i + d}, len = L - d, of packed +-1 strings (zero words behind).
__device__ __forceinline__ int packed_cross(const uint32_t* u, const uint32_t* v, int L, int d) {
    const int len = L - d, q = (d + 31) >> 5, sh = (32 - d) & 31;
    const int full = len >> 5;
    uint32_t pc = 0, hi = v[q - 1];
    for (int w = 0; w < full; ++w) {
        const uint32_t lo = v[w + q];
        pc = bcnt_add(u[w] ^ __builtin_amdgcn_alignbit(hi, lo, sh), pc);
        hi = lo;
    }
    const int rem = len & 31;
    if (rem) pc = bcnt_add((u[full] ^ __builtin_amdgcn_alignbit(hi, v[full + q], sh)) & ~(0xFFFFFFFFu >> rem), pc);
    return len - 2 * (int)pc;
}

// s of 1-based position x, 0 outside 1..L.
__device__ __forceinline__ int element(const uint32_t* pk, int L, int x) {
    return x < 1 || x > L ? 0 : packed_bit(pk, x) ? 1 : -1;
}

// LDS of one sequence of up to 256 NT elements: the packed string and its reverse (a zero
// word ahead, zero words behind), C_{|t|} at DB + t as low bytes and the bytes above them,
// (C + 128) >> 8, and a word a position.
template <int NT>
struct FlipLds {
    static constexpr int DB = 256 * NT, DN = DB + 256 * NT + 128;
    uint32_t fwd[kMaxW + 4], rev[kMaxW + 4];
    int8_t lo[DN] __attribute__((aligned(16)));
    int8_t hi[DN] __attribute__((aligned(16)));
    int32_t v[256 * NT] __attribute__((aligned(16)));
};

// The bytes of four elements from their bits (LSB first, 1 where the element is -1).
__device__ __forceinline__ uint32_t signs4(uint32_t nibble) {
    const uint32_t z = (nibble * 0x204081u) & 0x01010101u;
    return 0x01010101u + (z << 8) - (z << 1);
}
__device__ __forceinline__ uint32_t mask4(uint32_t nibble) {
    const uint32_t z = (nibble * 0x204081u) & 0x01010101u;
    return (z << 8) - z;
}

// H_a for a = 256 u + 16 col + row (from 0): row i of A holds s from element i - 16 on
// (expanded from the bits in registers), column j of tile u of B holds C_{|t|} from
// t = -16 - 256 u - 16 j on, so every load of B is 16 aligned bytes; low and high bytes
// of C are two products.  The popcounts of C and P bound it.  Byte loops over LDS, O(L)
// a neighbour, took 572 us for 4,096 sequences at L = 501; this takes 22, and
// the same for pairs.
template <int NT>
__global__ __launch_bounds__(64 * kWaves) void k_flip_deltas(int L, int p, int skew, int64_t n,
                                                             const uint32_t* __restrict__ seqs,
                                                             int32_t* __restrict__ dE) {
    typedef FlipLds<NT> T;
    __shared__ T SS[kWaves];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t j = (int64_t)blockIdx.x * kWaves + wv;
    if (j >= n) return;                           // waves do not meet again
    T& S = SS[wv];
    const int W = (L + 31) >> 5, pad = 32 * W - L;
    const uint32_t word = lane >= 1 && lane <= W ? seqs[j * W + lane - 1] : 0u;
    if (lane < kMaxW + 4) S.fwd[lane] = word;
    lds_order();
    if (lane < kMaxW + 4) {
        // word w of the reverse: the padded string reversed, less its `pad` leading bits
        const int w = lane - 1;
        const uint32_t a = w >= 0 && w < W ? __brev(S.fwd[W - w]) : 0u;
        const uint32_t b = w >= 0 && w + 1 < W ? __brev(S.fwd[W - w - 1]) : 0u;
        S.rev[lane] = pad ? (a << pad) | (b >> (32 - pad)) : a;
    }
    lds_order();
    const uint32_t* const fw = S.fwd + 1;
    const uint32_t* const rv = S.rev + 1;

    if (lane == 0) S.lo[T::DB] = S.hi[T::DB] = 0;
    for (int d = 1 + lane; d <= L - 1; d += 64) {
        const int c = packed_corr(fw, L, d);
        const int8_t lo = (int8_t)c, hi = (int8_t)((c + 128) >> 8);
        S.lo[T::DB + d] = S.lo[T::DB - d] = lo;
        S.hi[T::DB + d] = S.hi[T::DB - d] = hi;
    }
    for (int a = lane; a < L; a += 64) {
        const bool left = 2 * a <= L - 1;
        const int len = 2 * (left ? a : L - 1 - a) + 1;
        S.v[a] = (packed_cross(left ? fw : rv, left ? rv : fw, L, L - len) - 1) >> 1;
    }
    lds_order();

    const int lj = lane & 15, lg = lane >> 4;
    v4i lo[NT], hi[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) lo[u] = hi[u] = v4i{0, 0, 0, 0};
    for (int m = 0; 64 * m < L + 16; ++m) {
        const int i0 = lj + 64 * m + 16 * lg - 16;            // this lane's 16 elements
        const int q = (i0 + 31) >> 5;
        // past the string's last zero word every element is outside
        const uint32_t b = q <= W ? __builtin_amdgcn_alignbit(fw[q - 1], fw[q], (32 - i0) & 31) : 0u;
        const uint32_t z = ~__brev(b);
        uint32_t a[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = signs4((z >> (4 * r)) & 15u);
        if (m == 0 || 64 * m + 63 >= L) {
            const int first = i0 < 0 ? -i0 : 0, last = min(max(L - i0, 0), 16);
            const uint32_t in = ((1u << last) - 1u) & ~((1u << first) - 1u);
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] &= mask4((in >> (4 * r)) & 15u);
        }
        const v4i av = {(int)a[0], (int)a[1], (int)a[2], (int)a[3]};
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int off = T::DB + 64 * m + 16 * lg - 16 - 256 * u - 16 * lj;
            lo[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, *(const v4i*)(S.lo + off), lo[u], 0, 0, 0);
            hi[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, *(const v4i*)(S.hi + off), hi[u], 0, 0, 0);
        }
    }
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int a0 = 256 * u + 16 * lj + 4 * lg;
        const v4i P = *(const v4i*)(S.v + a0);
        const uint32_t bits = fw[a0 >> 5] << (a0 & 31);
        v4i d;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int h = lo[u][r] + 256 * hi[u][r];
            d[r] = ((bits >> (31 - r)) & 1u ? -4 * h : 4 * h) + 4 * (L - 1) + 8 * P[r];
        }
        if (skew) {
            *(v4i*)(S.v + a0) = d;
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (a0 + r < L) dE[j * L + a0 + r] = d[r];
        }
    }
    if (!skew) return;
    lds_order();
    const int k = (L - 1) / 2, nf = k + 1 - p;
    const int V = packed_cross(fw, rv, L, 0);
    for (int a = p + 1 + lane; a <= k + 1; a += 64) {
        const int b = L + 1 - a, g = b - a;
        int d = S.v[a - 1];
        if (g > 0) {
            const int sa = element(fw, L, a), sb = element(fw, L, b);
            const int c = S.lo[T::DB + g] + 256 * S.hi[T::DB + g];
            d += S.v[b - 1] + sa * sb * (16 * c + 8 * V) - 32 -
                 16 * (sb * element(fw, L, a - g) + sa * element(fw, L, b + g));
        }
        dE[j * nf + (a - p - 1)] = d;
    }
}

}  // namespace

labs_status launch_energy(int32_t L, int64_t n, const uint32_t* seqs, int32_t* E, int32_t* C,
                          hipStream_t st) {
    if (n == 0) return LABS_OK;
    hipLaunchKernelGGL(k_energy, dim3((unsigned)((n + kWaves - 1) / kWaves)), dim3(64 * kWaves), 0, st, L, n, seqs, E,
                       C);
    LABS_LAUNCHED("k_energy");
    return LABS_OK;
}

labs_status launch_flip_deltas(int32_t L, int32_t p, int32_t skew, int64_t n,
                               const uint32_t* seqs, int32_t* dE, hipStream_t st) {
    if (n == 0) return LABS_OK;
    const dim3 grid((unsigned)((n + kWaves - 1) / kWaves)), block(64 * kWaves);
    switch ((L + 255) / 256) {
        case 1: hipLaunchKernelGGL(k_flip_deltas<1>, grid, block, 0, st, L, p, skew, n, seqs, dE); break;
        case 2: hipLaunchKernelGGL(k_flip_deltas<2>, grid, block, 0, st, L, p, skew, n, seqs, dE); break;
        case 3: hipLaunchKernelGGL(k_flip_deltas<3>, grid, block, 0, st, L, p, skew, n, seqs, dE); break;
        default: hipLaunchKernelGGL(k_flip_deltas<4>, grid, block, 0, st, L, p, skew, n, seqs, dE); break;
    }
    LABS_LAUNCHED("k_flip_deltas");
    return LABS_OK;
}

}  // namespace labsdev
