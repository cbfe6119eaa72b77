// First step (Algorithm 1, with a tabu tenure or with its Bloom filter): walker
// init and the walk.
//
// One wavefront runs one walker.  Notation: L = 2k+1, even lags d = 2m,
// m = 1..K with K = k (odd-lag C vanish for skew sequences, Sec. 1).  Free
// positions a = p+1..k+1 (Eq. (3)); a lane owns four consecutive ones of one class (below)
// in each tile of 256.
//
// Energy change of the skew flip of a (partner b = L+1-a, partner lag
// mp = (b-a)/2 = k+1-a).  Flipping a and b changes C_{2m} by -4 s_a u_m with
//   u_m = s_{a+2m}[a+2m <= L, a+2m != b] + s_{a-2m}[a-2m >= 1]
// (for even lags the partner's contribution equals a's by Eq. (2), and the
// s_a s_b product inside C_{b-a} is unchanged), so
//   dE_a = sum_m (2 C dC + dC^2) = -8 s_a G_a + 16 Q_a,
//   G_a  = sum_m C_{2m} u_m,   Q_a = sum_m u_m^2.
// The centre a = k+1 flips alone: dC_{2m} = -4 s_a s_{a-2m}.
//
// The class of a position is its parity: cl = 0 holds the odd x, cl = 1 the even x, and
// index n = (x - 1) >> 1 counts them, so the lag 2m is a step of m indices inside a
// class.  With x_cl[n] the class (0 outside the sequence), the sum over all lags is
//   H_a = sum_{n' != n} x_cl[n'] C_{2|n' - n|} = G_a + C_{2mp} s_b,
// a product of the class with a symmetric Toeplitz matrix of the C table.  It runs on
// the matrix cores (v_mfma_i32_16x16x64_i8): rows are (class, n mod 8), columns n div 8,
//   A[(cl, i)][kap] = x_cl[i + kap - kz],   B[kap][j] = C_{2|kap - kz - n0 - 8 j|},
// so 256 positions take one 16x16 tile and ceil((k+12)/64) products a step, whose
// operands are aligned LDS reads: eight shifted copies of each class, and one table of
// the C.  A step changes two elements of the copies and rewrites the table.  C fits a
// signed byte in all but the first steps of a walk; while some |C| may pass 127 within
// four steps the bytes above are kept in a second table and multiplied too, so the
// scan is exact for every state.  By Eq. (2) s_a s_b is constant, and
//   Q_a = Mf + Mb - 1 + 2 Y_a - 2 s_b s_{a-2mp},   Y_a = sum_m s_{a+2m} s_{a-2m},
// Mf = (L-a)/2, Mb = (a-1)/2.  Y_a changes with a flip of index f by the one product
// of f and 2 n_a - f, so it is kept per slot (v_dot4 on the bytes around the flip).
// At the centre the two halves of H are equal: dE = -4 s_a H + 16 Mb.
//
// What bounds it: instruction issue and the LDS together.  At L = 501 a walker-step takes
// 103 vector and 96 scalar instructions on its SIMD and 117 LDS cycles on its CU, most of
// them the operands: 0.68 of the VALU and 0.72 of the LDS peak.  The popcount form this
// replaces needed 915 vector instructions: 16,384 walkers at L = 501, p = 16, 26.7 -> 4.1 us
// a step (1.44 -> 9.5e11 flip-evaluations/s); L = 301: 14.6 -> 3.56, L = 639: 42.5 -> 8.0 us.
#include "walk_impl.h"

#include <climits>

namespace labsdev {

using namespace walkimpl;

namespace {

struct InitLds {
    int8_t sv[640];                             // sv[x - 1] = s_x
    uint32_t pk[24];
};

// One wavefront a walker.  The even-lag C come from popcounts of the packed bits (16
// words a lag at L = 501): 16,384 walkers 437 -> 24 us; the byte products before read
// the LDS twice a term.
__device__ void walker_init_body(const WalkArgs& A, int64_t j, InitLds& S) {
    const int lane = threadIdx.x;
    const int64_t w = A.walker_begin + j;
    const int L = A.L, k = A.k, p = A.p;
    const uint64_t key = walker_key(A.seed, L, w);
    if (A.start_ticks && lane == 0) atomicMin(A.start_ticks, __builtin_amdgcn_s_memrealtime());
    // s_i for i = 1..k+1 from stream outputs i-1; s_1 = +1 when p >= 1; Eq. (2) for the rest
    for (int i = 1 + lane; i <= k + 1; i += 64) {
        uint64_t d = sm64_at(key, (uint64_t)(i - 1));
        int s = (d >> 63) ? 1 : -1;
        if (i == 1 && p >= 1) s = 1;
        S.sv[i - 1] = (int8_t)s;
        if (i <= k) {
            int ii = k + 1 - i;               // s_{k+1+ii} = (-1)^ii s_{k+1-ii}
            S.sv[k + ii] = (int8_t)((ii & 1) ? -s : s);
        }
    }
    if (lane < 24) S.pk[lane] = 0;
    __syncthreads();
    // pack
    const int W = A.W;
    for (int base = 0; base < 32 * W; base += 64) {
        int x = base + lane + 1;
        bool bit = x <= L && S.sv[x - 1] > 0;
        uint64_t m = __ballot(bit);
        // lane 0..31 bits map to MSB-first positions: bit (31 - (x-1)%32)
        if (lane == 0) {
            uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
            S.pk[base >> 5] = __builtin_bitreverse32(lo);
            if ((base >> 5) + 1 < W) S.pk[(base >> 5) + 1] = __builtin_bitreverse32(hi);
        }
    }
    __syncthreads();
    // energy from even lags (odd lags vanish under Eq. (2))
    int e = 0;
    for (int m = 1 + lane; m <= k; m += 64) {
        const int c = packed_corr(S.pk, L, 2 * m);
        e += c * c;
    }
    e = __ockl_wfred_add_i32(e);
    const uint64_t span = (uint64_t)(A.tenure_hi - A.tenure_lo + 1);
    const int ten = A.tenure_lo + (int)(sm64_at(key, (uint64_t)(k + 1)) % span);
    if (lane < W) {
        A.seq[j * W + lane] = S.pk[lane];
        A.bestSeq[j * W + lane] = S.pk[lane];
    }
    if (A.tabu)   // null for Bloom-filter walks
        for (int i = lane; i < A.nf; i += 64) A.tabu[j * A.nf + i] = 0;
    if (lane == 0) {
        A.E[j] = e;
        A.tenure[j] = ten;
        A.halted[j] = 0;
        A.bestE[j] = e;
        A.bestT[j] = 0;
    }
    if (A.n_levels > 0 && e <= pending_level(A)) stamp_levels(A, e, lane);
}

__global__ __launch_bounds__(64) void k_walker_init(WalkArgs A) {
    __shared__ InitLds S;
    walker_init_body(A, blockIdx.x, S);
}

// Init for a batch of (configuration, walker) items.
__global__ __launch_bounds__(64) void k_walker_init_items(const WalkArgs* args, const int2* items) {
    __shared__ InitLds S;
    const int2 it = items[blockIdx.x];
    const WalkArgs A = args[it.x];
    walker_init_body(A, (int64_t)it.y, S);
}

// Bloom-filter walks: the key of each walker's initial sequence (Zobrist XOR over
// the +1 elements among s_1..s_{k+1}), and its filter holding only that key.
__global__ __launch_bounds__(64) void k_bloom_init(WalkArgs A) {
    const int lane = threadIdx.x;
    const int64_t j = blockIdx.x;
    const uint32_t* s = A.seq + j * A.W;
    uint64_t h = 0;
    for (int i = 1 + lane; i <= A.k + 1; i += 64)
        if (packed_bit(s, i)) h ^= zobrist_at(i - 1);
    uint32_t lo = (uint32_t)h, hi = (uint32_t)(h >> 32);
    for (int o = 32; o > 0; o >>= 1) {
        lo ^= (uint32_t)__shfl_xor((int)lo, o, 64);
        hi ^= (uint32_t)__shfl_xor((int)hi, o, 64);
    }
    h = ((uint64_t)hi << 32) | lo;
    const int nbw = 1 << (A.bloom_log2 - 5);
    const uint32_t mask = (1u << A.bloom_log2) - 1u;
    const uint32_t g2 = hi | 1u;
    uint32_t* f = A.bloom + j * (int64_t)nbw;
    for (int w = lane; w < nbw; w += 64) {
        uint32_t v = 0, x = lo;
        for (int q = 0; q < A.bloom_hashes; ++q) {
            const uint32_t b = x & mask;
            if ((int)(b >> 5) == w) v |= 1u << (b & 31);
            x += g2;
        }
        f[w] = v;
    }
    if (lane == 0) A.zh[j] = h;
}

// Offer every walker's best sequence to the staging buffer: a workgroup takes the places of
// its kOffer walkers at once (an atomic a walker on the one counter took 190 us for 16,384
// walkers, now 13), a wave writes one record after the other.
constexpr int kOffer = 64;
__global__ __launch_bounds__(256) void k_offer_best(WalkArgs A) {
    __shared__ uint32_t base;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t j0 = (int64_t)blockIdx.x * kOffer;
    const int m = (int)(A.n - j0 < kOffer ? A.n - j0 : kOffer);
    if (threadIdx.x == 0) base = atomicAdd(A.st_count, (uint32_t)m);
    __syncthreads();
    const int W = A.W;
    for (int i = wv; i < m; i += 4) {
        const int64_t j = j0 + i;
        const uint32_t slot = base + (uint32_t)i;
        if (slot >= A.st_cap || lane >= W + 3) continue;
        uint32_t v;
        if (lane == 0) v = (uint32_t)A.bestE[j];
        else if (lane <= W) v = A.bestSeq[j * W + lane - 1];
        else if (lane == W + 1) v = (uint32_t)(A.walker_begin + j);
        else v = (uint32_t)A.bestT[j];
        A.rec[(int64_t)lane * A.rec_stride + slot] = v;
    }
}

__global__ void k_walk_outputs(WalkArgs A, uint32_t* final_seqs, int32_t* final_E,
                               uint32_t* best_seqs, int32_t* best_E, int32_t* best_step,
                               int64_t* flip_evals) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int W = A.W;
    if (i < A.n * W) {
        if (final_seqs) final_seqs[i] = A.seq[i];
        if (best_seqs) best_seqs[i] = A.bestSeq[i];
    }
    if (i < A.n) {
        if (final_E) final_E[i] = A.E[i];
        if (best_E) best_E[i] = A.bestE[i];
        if (best_step) best_step[i] = A.bestT[i];
    }
    if (flip_evals) {
        int64_t v = 0;
        if (i < A.n) {
            const int h = A.halted[i];
            const int taken = h ? h - 1 : A.t1;
            v = (int64_t)taken * A.nf;
        }
        // wave sum then one atomic per wave
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0 && v) atomicAdd((unsigned long long*)flip_evals, (unsigned long long)v);
    }
}

}  // namespace

bool walk_kernels(const WalkShape& s, WalkKernels* out) {
    if (s.KH <= 8) return s.NT == 1 && s.NQ == 1 && (walk_kernels_a(s.KH, out) || walk_kernels_b(s.KH, out));
    return walk_kernels_c(s.KH, s.NT, s.NQ, out);
}

bool walk_shape_supported(int L, int p) {
    WalkKernels wk;
    return walk_kernels(walk_shape(L, p), &wk);
}

labs_status launch_walker_init_items(const WalkArgs* args, const int2* items, int n_items, hipStream_t st) {
    if (n_items <= 0) return LABS_OK;
    hipLaunchKernelGGL(k_walker_init_items, dim3((unsigned)n_items), dim3(64), 0, st, args, items);
    LABS_LAUNCHED("k_walker_init_items");
    return LABS_OK;
}

labs_status launch_walker_init(const WalkArgs& A, hipStream_t st) {
    hipLaunchKernelGGL(k_walker_init, dim3((unsigned)A.n), dim3(64), 0, st, A);
    LABS_LAUNCHED("k_walker_init");
    return LABS_OK;
}

labs_status launch_bloom_init(const WalkArgs& A, hipStream_t st) {
    hipLaunchKernelGGL(k_bloom_init, dim3((unsigned)A.n), dim3(64), 0, st, A);
    LABS_LAUNCHED("k_bloom_init");
    return LABS_OK;
}

labs_status launch_walk(const WalkArgs& A, hipStream_t st) {
    WalkKernels wk;
    if (!walk_kernels(walk_shape(A.L, A.p), &wk)) return invalid("no walker kernel for L=%d p=%d", A.L, A.p);
    if (A.bloom) {
        const size_t lds = sizeof(uint32_t) << (A.bloom_log2 - 5);
        hipLaunchKernelGGL(wk.bloom, dim3((unsigned)A.n), dim3(64), lds, st, A);
        LABS_LAUNCHED("k_walk_bloom");
        return LABS_OK;
    }
    const int group = walk_group(A.L, A.p, A.n);
    if (group > 1) return launch_walk_group(A, group, st);
    hipLaunchKernelGGL(wk.plain, dim3((unsigned)A.n), dim3(64), 0, st, A);
    LABS_LAUNCHED("k_walk");
    return LABS_OK;
}

labs_status launch_walk_log(const WalkArgs& A, hipStream_t st) {
    WalkKernels wk;
    if (!walk_kernels(walk_shape(A.L, A.p), &wk)) return invalid("no walker kernel for L=%d p=%d", A.L, A.p);
    hipLaunchKernelGGL(wk.log, dim3((unsigned)A.n), dim3(64), 0, st, A);
    LABS_LAUNCHED("k_walk_log");
    return LABS_OK;
}

labs_status launch_offer_best(const WalkArgs& A, hipStream_t st) {
    hipLaunchKernelGGL(k_offer_best, dim3((unsigned)((A.n + kOffer - 1) / kOffer)), dim3(256), 0, st, A);
    LABS_LAUNCHED("k_offer_best");
    return LABS_OK;
}

labs_status launch_walk_outputs(const WalkArgs& A, const labs_step1_out& o, hipStream_t st) {
    const int64_t total = A.n * A.W > A.n ? A.n * A.W : A.n;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(k_walk_outputs, dim3(blocks), dim3(256), 0, st, A, o.final_seqs, o.final_E,
                       o.best_seqs, o.best_E, o.best_step, o.flip_evals);
    LABS_LAUNCHED("k_walk_outputs");
    return LABS_OK;
}

}  // namespace labsdev
