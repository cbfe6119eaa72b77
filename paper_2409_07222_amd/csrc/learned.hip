// First-step walk with a proposer narrowing the candidate flips (the learned
// form): every candidate is rescored with its exact integer energy change, and
// every fallback_every-th step is the plain walker's full scan.
//
// A full scan is a launch of the plain walker's logging kernel over one step (over
// thousands of steps when every step is one).  The steps between are two launches each, the
// network's pass over all walkers and k_lw_step; the walker state lives in HBM between
// them: packed sequence, C_{2m} as 16-bit integers, energy, tabu deadlines, tenure, best.
#include "labs_internal.h"

#include <climits>

namespace labsdev {

namespace {

constexpr int kLwLmax = 639;
constexpr int kLogSegment = 4096;   // steps a launch of the logging walk
constexpr int kTabuPad = 320;       // readable integers around the tabu deadlines

struct LwArgs {
    int32_t L, p, k, nf, W, MW, ld_out, ldc;
    int32_t top_m, mode, log_every, steps, t;
    int64_t n, walker_begin;
    uint64_t prop_seed;
    int32_t e_max;
    uint32_t* seq;
    int16_t* C;            // [n * ldc], C_{2m} at m - 1, zeros behind k
    int32_t* E;
    const int32_t* tenure;
    int32_t* halted;
    int32_t* tabu;
    int32_t* bestE;
    int32_t* bestT;
    uint32_t* bestSeq;
    int64_t* evals;
    int32_t* hit;
    // first-hit stamps (n_levels = 0: off); hitmask [n] holds each walker's stamped levels
    int32_t n_levels;
    int32_t level_E[16];
    unsigned long long* hit_ticks;
    uint32_t* hitmask;
    const float* logits;
    int32_t* traj;
    int32_t* moves;
    int16_t* cands;
    uint32_t* log_seqs;
    uint32_t* log_mask;
    int32_t* log_label;
};

// Order-preserving map of an FP32 score to uint32 (-0 counts as +0).
__device__ __forceinline__ uint32_t score_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if (u == 0x80000000u) u = 0;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// A walker is a row of 16 lanes; lane patterns that exchange its halves, quarters, pairs.
constexpr int kSwap1 = 0xB1, kSwap2 = 0x4E, kSwap4 = 0x141, kSwap8 = 0x140;
template <int CTRL>
__device__ __forceinline__ int swapped(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double swapped(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)swapped<CTRL>((int)(uint32_t)u), hi = (uint32_t)swapped<CTRL>((int)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int row_min(int v) {
    v = min(v, swapped<kSwap1>(v));
    v = min(v, swapped<kSwap2>(v));
    v = min(v, swapped<kSwap4>(v));
    return min(v, swapped<kSwap8>(v));
}

// A candidate's key: a double of exponent 0 whose mantissa is the 32-bit score and, below
// it, 2^20 - 1 - position, so one FP64 minimum or maximum orders (score, lower position
// first) exactly; 0 where there is none.
__device__ __forceinline__ double make_key(uint32_t score, int pos) {
    return __builtin_bit_cast(double, (uint64_t)(0x3FF00000u | (score >> 12)) << 32 |
                                          ((score << 20) | (uint32_t)(0xFFFFF - pos)));
}
__device__ __forceinline__ int key_pos(double key) {
    return 0xFFFFF - (int)((uint32_t)__builtin_bit_cast(uint64_t, key) & 0xFFFFF);
}
__device__ __forceinline__ double kmax(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ void order2(double& a, double& b) {   // a >= b
    const double hi = __builtin_fmax(a, b), lo = __builtin_fmin(a, b);
    a = hi;
    b = lo;
}
// Sorts a bitonic list, largest first.
template <int M>
__device__ __forceinline__ void bitonic(double (&v)[M]) {
#pragma unroll
    for (int d = M / 2; d > 0; d /= 2)
#pragma unroll
        for (int i = 0; i < M; ++i)
            if (!(i & d)) order2(v[i], v[i + d]);
}
// The M largest of this lane's list and its partner's, sorted, in both lanes.
template <int CTRL, int M>
__device__ __forceinline__ void merge_lanes(double (&v)[M]) {
    double o[M];
#pragma unroll
    for (int i = 0; i < M; ++i) o[i] = swapped<CTRL>(v[M - 1 - i]);
#pragma unroll
    for (int i = 0; i < M; ++i) v[i] = kmax(v[i], o[i]);
    bitonic(v);
}

// LDS of one walker: class rows (class 0: odd positions, 1: even; index n = (x - 1) >> 1)
// as bytes +-1, zeros around them, and the bytes of C of four lags a group, {low, the
// bytes above: (C + 128) >> 8}.
template <int NQ>
struct LwLds {
    static constexpr int PAD = 24, ST = 64 * NQ + 2 * PAD;
    int8_t x[2][ST] __attribute__((aligned(16)));
    uint2 ct[16 * NQ] __attribute__((aligned(16)));
    int32_t cand[64] __attribute__((aligned(16)));
};

// Four bits 6, 4, 2, 0 to the lowest bits of four bytes.
__device__ __forceinline__ uint32_t spread4(uint32_t t) {
    return ((t | (t << 10) | (t << 20) | (t << 30)) >> 6) & 0x01010101u;
}

// One narrow step: the top_m admissible positions by score, their exact dE, the move.
// NQ: groups of 64 lags or positions, M: length of the candidate list a lane keeps (64:
// the candidates are taken one at a time).  Bound by issue, so a walker is 16 lanes and
// every part is spread over them without idle ones: keys (four positions a lane and
// group), a merge of sorted lists instead of top_m reductions, and dE of a candidate by
// 16/M lanes, four lags a dot product:
//   dC_{2m} = -4 s_a (x[n+m] + x[n-m]) for a flipped pair (x[n+m] = s_b left out; at the
//   centre -2 s_a), by the symmetry of the pair, so
//   dE = 16 (k - 1 - cl) + 32 (sum_m x[n+m] x[n-m]) - 8 s_a sum_m C_{2m} (x[n+m] + x[n-m])
//   with the partner's terms taken out, and at the centre 16 n - 4 s_a sum_m (same).
// A wave a walker that rebuilt C, read the network's features' sources element by element
// and wrote the features took 82 us a step of 16,384 walkers at L = 501, top 8; this takes
// 17.6.
template <int NQ, int M>
__global__ __launch_bounds__(256) void k_lw_step(LwArgs A) {
    typedef LwLds<NQ> T;
    typedef short v2s __attribute__((ext_vector_type(2)));
    struct __attribute__((packed, aligned(4))) int4u { int v[4]; };
    constexpr int PER = M == 8 ? 8 : 16, NH = 16 / PER;
    __shared__ T SS[16];
    T& S = SS[threadIdx.x >> 4];
    const int l = threadIdx.x & 15;
    const int64_t j = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const int L = A.L, k = A.k, p = A.p, W = A.W, t = A.t;
    if (j >= A.n) return;                        // whole rows leave; rows do not meet again
    const int64_t ti = j * A.steps + (t - 1);
    const int64_t tb = j * A.nf - p;

    if (A.halted[j]) {
        if (l == 0) {
            if (A.traj) A.traj[ti] = -1;
            if (A.moves) A.moves[ti] = -1;
        }
        if (A.cands)
            for (int i = l; i < A.top_m; i += 16) A.cands[ti * A.top_m + i] = -1;
        return;
    }

    const int E0 = A.E[j], bE0 = A.bestE[j], tenure = A.tenure[j];
    uint32_t word[2];
    word[0] = l < W ? A.seq[j * W + l] : 0;
    word[1] = NQ > 4 && l + 16 < W ? A.seq[j * W + l + 16] : 0;
    v2s c01[NQ], c23[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const uint2 v = *(const uint2*)(A.C + j * A.ldc + 4 * (l + 16 * q));
        c01[q] = __builtin_bit_cast(v2s, v.x);
        c23[q] = __builtin_bit_cast(v2s, v.y);
    }

    // ---- keys of the admissible positions (position a - 1 = 4 (l + 16 q) + r)
    double key[4 * NQ];
    uint32_t adm = 0;                             // bit 4 q + r
    const uint64_t rkey = A.mode == LABS_PROPOSE_RANDOM ? walker_key(A.prop_seed, L, A.walker_begin + j) : 0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int pos0 = 4 * (l + 16 * q);
        const int4u until = *(const int4u*)(A.tabu + tb + pos0);
        uint32_t sc[4] = {0, 0, 0, 0};
        if (A.mode == LABS_PROPOSE_MLP) {
            if (64 * q < A.ld_out) {
                const float4 z = *(const float4*)(A.logits + j * A.ld_out + pos0);
                sc[0] = score_bits(z.x);
                sc[1] = score_bits(z.y);
                sc[2] = score_bits(z.z);
                sc[3] = score_bits(z.w);
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                sc[r] = (uint32_t)(sm64_at(rkey, (uint64_t)(t - 1) * (uint64_t)(k + 1) + (uint64_t)(pos0 + r)) >> 32);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool ok = pos0 + r >= p && pos0 + r <= k && until.v[r] < t;
            adm |= (ok ? 1u : 0u) << (4 * q + r);
            key[4 * q + r] = ok ? make_key(sc[r], pos0 + r) : 0.0;
        }
    }

    // ---- class rows and the bytes of C
#pragma unroll
    for (int h = 0; h < (NQ > 4 ? 2 : 1); ++h) {
        const int w = l + 16 * h;
        if (w < W) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                uint32_t d[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t z = spread4((~word[h] >> (24 - 8 * q + 1 - c)) & 0x55u);   // 1 where x = -1
                    d[q] = 0x01010101u + (z << 8) - (z << 1);
                }
                *(uint2*)(S.x[c] + T::PAD + 16 * w) = make_uint2(d[0], d[1]);
                *(uint2*)(S.x[c] + T::PAD + 16 * w + 8) = make_uint2(d[2], d[3]);
            }
        }
    }
    lds_order();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        // zeros ahead, behind the last element (k + 1 of class 0, k of class 1), behind the words
        const int size = k + 1 - c;
        if (size + l < 16 * W) S.x[c][T::PAD + size + l] = 0;
        if (l < 6) *(uint32_t*)(S.x[c] + 4 * l) = 0;
        if (l < 6) *(uint32_t*)(S.x[c] + T::PAD + 16 * W + 4 * l) = 0;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const v2s bias = {128, 128};
        uint2 v;
        v.x = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, c23[q]), __builtin_bit_cast(uint32_t, c01[q]),
                                    0x06040200u);
        v.y = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, (v2s)(c23[q] + bias)),
                                    __builtin_bit_cast(uint32_t, (v2s)(c01[q] + bias)), 0x07050301u);
        S.ct[l + 16 * q] = v;
    }

    // ---- the candidates
    int ncand = 0;
    if constexpr (M <= 16) {
        double v[M];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            double* s = key + 4 * q;
            order2(s[0], s[1]);
            order2(s[2], s[3]);
            order2(s[0], s[2]);
            order2(s[1], s[3]);
            order2(s[1], s[2]);
            if (q == 0) {
#pragma unroll
                for (int i = 0; i < M; ++i) v[i] = i < 4 ? s[i] : 0.0;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[M - 4 + i] = kmax(v[M - 4 + i], s[3 - i]);
                bitonic(v);
            }
        }
        merge_lanes<kSwap1>(v);
        merge_lanes<kSwap2>(v);
        merge_lanes<kSwap4>(v);
        merge_lanes<kSwap8>(v);
#pragma unroll
        for (int i = 0; i < M; ++i) {
            ncand += v[i] != 0.0 && i < A.top_m ? 1 : 0;
            if (l == 0) S.cand[i] = key_pos(v[i]) + 1;
        }
    } else {
        for (; ncand < A.top_m; ++ncand) {
            double best = key[0];
#pragma unroll
            for (int i = 1; i < 4 * NQ; ++i) best = kmax(best, key[i]);
            best = kmax(best, swapped<kSwap1>(best));
            best = kmax(best, swapped<kSwap2>(best));
            best = kmax(best, swapped<kSwap4>(best));
            best = kmax(best, swapped<kSwap8>(best));
            if (best == 0.0) break;
#pragma unroll
            for (int i = 0; i < 4 * NQ; ++i)
                if (key[i] == best) key[i] = 0.0;
            if (l == 0) S.cand[ncand] = key_pos(best) + 1;
        }
    }
    lds_order();

    if (ncand == 0) {   // no admissible move: the walk halts here
        if (l == 0) {
            A.halted[j] = t;
            if (A.traj) A.traj[ti] = -1;
            if (A.moves) A.moves[ti] = -1;
        }
        if (A.cands)
            for (int i = l; i < A.top_m; i += 16) A.cands[ti * A.top_m + i] = -1;
        return;
    }

    // ---- exact dE of every candidate, blocks of 16 lags
    int dE = INT_MAX, a = INT_MAX;
    for (int c0 = 0; c0 < ncand; c0 += PER) {
        const int c = c0 + (l % PER);
        const int ca = S.cand[c < ncand ? c : 0], x1 = ca - 1, cl = x1 & 1, n = x1 >> 1;
        const int8_t* const x = S.x[cl] + T::PAD;
        const int size = k + 1 - cl;
        const int8_t* const pf = x + ((n + 1) & ~3);
        const int8_t* const pb = x + ((n - 4) & ~3);
        const uint32_t sf = 0x03020100u + 0x01010101u * (uint32_t)((n + 1) & 3);
        const uint32_t sb = 0x00010203u + 0x01010101u * (uint32_t)(n & 3);
        int lo = 0, hi = 0, y = 0;
        for (int b0 = 16 * (l / PER); b0 < k; b0 += 16 * NH) {
            if (n + 1 + b0 >= size) break;        // both ends of every pair are outside
            const uint4 g0 = *(const uint4*)&S.ct[b0 / 4], g1 = *(const uint4*)&S.ct[b0 / 4 + 2];
            const uint32_t cl4[4] = {g0.x, g0.z, g1.x, g1.z}, ch4[4] = {g0.y, g0.w, g1.y, g1.w};
            uint32_t f[4], w[5];
#pragma unroll
            for (int i = 0; i < 5; ++i) w[i] = *(const uint32_t*)(pf + b0 + 4 * i);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f[i] = __builtin_amdgcn_perm(w[i + 1], w[i], sf);
                lo = __builtin_amdgcn_sdot4((int)f[i], (int)cl4[i], lo, false);
                hi = __builtin_amdgcn_sdot4((int)f[i], (int)ch4[i], hi, false);
            }
            if (b0 < n) {
#pragma unroll
                for (int i = 0; i < 5; ++i) w[i] = *(const uint32_t*)(pb - b0 + 4 - 4 * i);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t g = __builtin_amdgcn_perm(w[i], w[i + 1], sb);
                    lo = __builtin_amdgcn_sdot4((int)g, (int)cl4[i], lo, false);
                    hi = __builtin_amdgcn_sdot4((int)g, (int)ch4[i], hi, false);
                    y = __builtin_amdgcn_sdot4((int)g, (int)f[i], y, false);
                }
            }
        }
        int s = lo + 256 * hi;
        if constexpr (NH > 1) {
            s += swapped<0x128>(s);               // row_ror:8
            y += swapped<0x128>(y);
        }
        const int sa = x[n], nb = k - n - cl, mp = nb - n;
        int d;
        if (mp == 0) {
            d = 16 * n - 4 * sa * s;
        } else {
            const int xb = x[nb], xm = x[n - mp > -1 ? n - mp : -1];
            const uint2 g = S.ct[(mp - 1) >> 2];
            const int sh = 8 * ((mp - 1) & 3);
            const int cm = (int8_t)(g.x >> sh) + 256 * (int8_t)(g.y >> sh);
            d = 16 * (k - 1 - cl) + 32 * (y - xb * xm) - 8 * sa * (s - cm * xb);
        }
        if (c < ncand && (d < dE || (d == dE && ca < a))) {
            dE = d;
            a = ca;
        }
    }
    const int dmin = row_min(dE);
    a = row_min(dE == dmin ? a : INT_MAX);
    const int newE = E0 + dmin;
    const int x1 = a - 1, cl = x1 & 1, n = x1 >> 1, nb = k - n - cl;
    const bool cen = n == nb;

    // ---- training log: the state before the move
    if (A.log_every > 0 && t % A.log_every == 0) {
        const int64_t r = (int64_t)(t / A.log_every - 1) * A.n + j;   // step-major records
        if (l < W) A.log_seqs[r * W + l] = word[0];
        if (NQ > 4 && l + 16 < W) A.log_seqs[r * W + l + 16] = word[1];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            int bits = (int)(((adm >> (4 * q)) & 15u) << (4 * (l & 7)));   // 8 lanes a word
            bits |= swapped<kSwap1>(bits);
            bits |= swapped<kSwap2>(bits);
            bits |= swapped<kSwap4>(bits);
            const int w = 2 * q + (l >> 3);
            if ((l & 7) == 0 && w < A.MW) A.log_mask[r * A.MW + w] = (uint32_t)bits;
        }
        if (l == 0) A.log_label[r] = a - 1;
    }
    if (A.cands)
        for (int i = l; i < A.top_m; i += 16)
            A.cands[ti * A.top_m + i] = i < ncand ? (int16_t)S.cand[i] : (int16_t)-1;

    // ---- apply: C with the partner's byte out of its row
    int8_t* const x = S.x[cl] + T::PAD;
    const int sa = x[n];
    lds_order();
    if (l == 0 && !cen) x[nb] = 0;
    lds_order();
    {
        const uint32_t sf = 0x03020100u + 0x01010101u * (uint32_t)((n + 1) & 3);
        const uint32_t sb = 0x00010203u + 0x01010101u * (uint32_t)(n & 3);
        const short mul = (short)(cen ? -2 * sa : -4 * sa);
        const v2s mul2 = {mul, mul};
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int m0 = 4 * (l + 16 * q);
            const int of = min(((n + 1) & ~3) + m0, 16 * W + 16), ob = max(((n - 4) & ~3) - m0, -8);
            const uint32_t f = __builtin_amdgcn_perm(*(const uint32_t*)(x + of + 4), *(const uint32_t*)(x + of), sf);
            const uint32_t b = __builtin_amdgcn_perm(*(const uint32_t*)(x + ob + 4), *(const uint32_t*)(x + ob), sb);
            const v2s u01 = __builtin_bit_cast(v2s, __builtin_amdgcn_perm(f, f, 0x010C000Cu)) +
                            __builtin_bit_cast(v2s, __builtin_amdgcn_perm(b, b, 0x010C000Cu));
            const v2s u23 = __builtin_bit_cast(v2s, __builtin_amdgcn_perm(f, f, 0x030C020Cu)) +
                            __builtin_bit_cast(v2s, __builtin_amdgcn_perm(b, b, 0x030C020Cu));
            c01[q] += (u01 >> 8) * mul2;
            c23[q] += (u23 >> 8) * mul2;
            *(uint2*)(A.C + j * A.ldc + m0) =
                make_uint2(__builtin_bit_cast(uint32_t, c01[q]), __builtin_bit_cast(uint32_t, c23[q]));
        }
    }
    const int x2 = L - a;                         // the partner's place in the string
#pragma unroll
    for (int h = 0; h < (NQ > 4 ? 2 : 1); ++h) {
        const int w = l + 16 * h;
        uint32_t v = word[h];
        if (w == x1 >> 5) v ^= 1u << (31 - (x1 & 31));
        if (w == x2 >> 5 && !cen) v ^= 1u << (31 - (x2 & 31));
        if (w < W) {
            if (v != word[h]) A.seq[j * W + w] = v;
            if (newE < bE0) A.bestSeq[j * W + w] = v;
        }
    }
    if (l == 0) {
        A.E[j] = newE;
        A.tabu[tb + x1] = t + tenure;
        if (A.traj) A.traj[ti] = newE;
        if (A.moves) A.moves[ti] = a;
        A.evals[j] += ncand;
        if (A.e_max >= 0 && newE <= A.e_max && A.hit[j] < 0) A.hit[j] = t;
        if (A.n_levels > 0) {
            const unsigned long long now = __builtin_amdgcn_s_memrealtime();
            uint32_t hm = A.hitmask[j];
            const uint32_t hm0 = hm;
            for (int q = 0; q < A.n_levels; ++q)
                if (!((hm >> q) & 1u) && newE <= A.level_E[q]) {
                    atomicMin(&A.hit_ticks[q], now);
                    hm |= 1u << q;
                }
            if (hm != hm0) A.hitmask[j] = hm;
        }
        if (newE < bE0) {
            A.bestE[j] = newE;
            A.bestT[j] = t;
        }
    }
}

// After a full scan: C of the walker's sequence, and no candidates logged for the step.
__global__ __launch_bounds__(256) void k_lw_corr(LwArgs A) {
    __shared__ uint32_t sw[4][24];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t j = (int64_t)blockIdx.x * 4 + wv;
    if (lane < 24) sw[wv][lane] = j < A.n && lane < A.W ? A.seq[j * A.W + lane] : 0u;
    __syncthreads();
    if (j >= A.n) return;
    for (int i = lane; i < A.ldc; i += 64)
        A.C[j * A.ldc + i] = i < A.k ? (int16_t)packed_corr(sw[wv], A.L, 2 * i + 2) : (int16_t)0;
    if (A.cands)
        for (int i = lane; i < A.top_m; i += 64) A.cands[(j * A.steps + A.t - 1) * A.top_m + i] = -1;
}

// 64-lag groups of the step's kernel: 2, 4 or 5.
int lw_groups(int k) { return k < 128 ? 2 : k < 256 ? 4 : 5; }

template <int NQ>
void launch_lw_step_nq(const LwArgs& A, hipStream_t st) {
    const dim3 grid((unsigned)((A.n + 15) / 16)), block(256);
    if (A.top_m <= 8) hipLaunchKernelGGL((k_lw_step<NQ, 8>), grid, block, 0, st, A);
    else if (A.top_m <= 16) hipLaunchKernelGGL((k_lw_step<NQ, 16>), grid, block, 0, st, A);
    else hipLaunchKernelGGL((k_lw_step<NQ, 64>), grid, block, 0, st, A);
}

labs_status launch_lw_step(const LwArgs& A, hipStream_t st) {
    switch (A.ldc) {
        case 128: launch_lw_step_nq<2>(A, st); break;
        case 256: launch_lw_step_nq<4>(A, st); break;
        default: launch_lw_step_nq<5>(A, st); break;
    }
    LABS_LAUNCHED("k_lw_step");
    return LABS_OK;
}

__global__ void k_lw_init(int64_t n, int64_t* evals, int32_t* hit, uint32_t* hitmask) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        evals[i] = 0;
        hit[i] = -1;
        hitmask[i] = 0;
    }
}

__global__ void k_lw_outputs(LwArgs A, uint32_t* final_seqs, int32_t* final_E, uint32_t* best_seqs,
                             int32_t* best_E, int32_t* best_step, int32_t* hit_step) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < A.n * A.W) {
        if (final_seqs) final_seqs[i] = A.seq[i];
        if (best_seqs) best_seqs[i] = A.bestSeq[i];
    }
    if (i < A.n) {
        if (final_E) final_E[i] = A.E[i];
        if (best_E) best_E[i] = A.bestE[i];
        if (best_step) best_step[i] = A.bestT[i];
        if (hit_step) hit_step[i] = A.hit[i];
    }
}

__global__ __launch_bounds__(256) void k_fill_i16(int64_t n, int16_t* p, int16_t v) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = v;
}

// One workgroup, eight values a thread in flight (16,384 walkers: 17 -> 4.6 us).
__global__ __launch_bounds__(1024) void k_sum_i64(int64_t n, const int64_t* v, int64_t* out) {
    __shared__ int64_t part[16];
    int64_t s = 0;
    for (int64_t i = threadIdx.x; i < n; i += 8 * 1024) {
        int64_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = i + 1024 * u < n ? v[i + 1024 * u] : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += x[u];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        s = 0;
        for (int w = 0; w < 16; ++w) s += part[w];
        *out = s;
    }
}

struct LwBuffers {
    WalkArgs wa;
    LwArgs la;
    void* fwd_ws;
    size_t fwd_bytes;
    uint16_t* X;    // features, for a network that does not pack
    size_t bytes;   // workspace used
    bool ok;
};

LwBuffers carve_lw(const labs_step1_cfg& c, const labs_proposer& pr, const labs_mlp_layout* lay, void* ws,
                   size_t wsb) {
    LwBuffers B{};
    Carve cv(ws, wsb);
    const int L = c.L, k = (L - 1) / 2, nf = k + 1 - c.p, W = words_of(L);
    const int64_t n = c.n_walkers;
    WalkArgs& w = B.wa;
    w.L = L; w.p = c.p; w.k = k; w.nf = nf; w.W = W;
    w.t0 = 0; w.t1 = 0; w.steps_total = c.steps;
    w.n = n; w.walker_begin = c.walker_begin; w.seed = c.seed;
    w.tenure_lo = c.tenure_lo; w.tenure_hi = c.tenure_hi;
    w.seq = cv.take<uint32_t>((size_t)n * W);
    w.E = cv.take<int32_t>(n);
    w.tenure = cv.take<int32_t>(n);
    w.halted = cv.take<int32_t>(n);
    w.tabu = cv.take<int32_t>((size_t)n * nf + 2 * kTabuPad);
    if (w.tabu) w.tabu += kTabuPad;
    w.bestE = cv.take<int32_t>(n);
    w.bestT = cv.take<int32_t>(n);
    w.bestSeq = cv.take<uint32_t>((size_t)n * W);
    w.traj = nullptr;
    w.e_max = c.e_max;
    LwArgs& a = B.la;
    a.L = L; a.p = c.p; a.k = k; a.nf = nf; a.W = W; a.MW = (k + 1 + 31) / 32;
    a.ldc = 64 * lw_groups(k);
    a.ld_out = lay ? lay->ld_out : 0;
    a.top_m = pr.top_m; a.mode = pr.mode;
    a.log_every = pr.log_every; a.steps = c.steps;
    a.n = n; a.walker_begin = c.walker_begin; a.prop_seed = pr.seed; a.e_max = c.e_max;
    a.seq = w.seq; a.E = w.E; a.tenure = w.tenure; a.halted = w.halted; a.tabu = w.tabu;
    a.bestE = w.bestE; a.bestT = w.bestT; a.bestSeq = w.bestSeq;
    a.C = cv.take<int16_t>((size_t)n * a.ldc);
    a.evals = cv.take<int64_t>(n);
    a.hit = cv.take<int32_t>(n);
    a.hitmask = cv.take<uint32_t>(n);
    if (lay) {
        B.X = mlp_packs(*lay) ? nullptr : cv.take<uint16_t>((size_t)n * lay->ld_in);
        a.logits = cv.take<float>((size_t)n * lay->ld_out);
        B.fwd_bytes = mlp_forward_ws(*lay, n);
        B.fwd_ws = cv.take<char>(B.fwd_bytes);
    }
    B.bytes = cv.used;
    B.ok = cv.ok() && ws != nullptr;
    return B;
}

}  // namespace

size_t learned_walk_ws(const labs_step1_cfg& c, const labs_proposer& pr) {
    labs_mlp_layout lay;
    const bool mlp = pr.mode == LABS_PROPOSE_MLP && mlp_layout(c.L, pr.hidden, &lay);
    return carve_lw(c, pr, mlp ? &lay : nullptr, nullptr, 0).bytes + 256;
}

bool learned_walk_supported(int L) { return L <= kLwLmax; }

labs_status learned_walk(const labs_step1_cfg& c, const labs_proposer& pr, const labs_learned_out& o, void* ws,
                         size_t wsb, hipStream_t st) {
    labs_mlp_layout lay;
    const bool mlp = pr.mode == LABS_PROPOSE_MLP;
    if (mlp && !mlp_layout(c.L, pr.hidden, &lay)) return invalid("unsupported network width %d", pr.hidden);
    LwBuffers B = carve_lw(c, pr, mlp ? &lay : nullptr, ws, wsb);
    if (!B.ok) return invalid("workspace too small");
    LwArgs& A = B.la;
    A.traj = o.traj_E;
    A.moves = o.moves;
    A.cands = o.cands;
    A.log_seqs = o.log_seqs;
    A.log_mask = o.log_mask;
    A.log_label = o.log_label;
    {
        labs_status ss = set_stamps(B.wa, o);
        if (ss != LABS_OK) return ss;
        A.n_levels = B.wa.n_levels;
        for (int l = 0; l < LABS_MAX_LEVELS; ++l) A.level_E[l] = B.wa.level_E[l];
        A.hit_ticks = B.wa.hit_ticks;
    }
    const int64_t n = A.n;
    labs_status s = launch_walker_init(B.wa, st);
    if (s) return s;
    hipLaunchKernelGGL(k_lw_init, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, A.evals, A.hit, A.hitmask);
    LABS_LAUNCHED("k_lw_init");

    const int64_t tot = n * A.W > n ? n * A.W : n;
    const int F = pr.fallback_every;
    // Full scans by the plain walker's kernel, whose matrix-core scan costs a hundredth of
    // one by candidates (16,384 walkers at L = 501, a record every 7 steps: 705 -> 5.6 us a
    // step, 92 with its setup in a launch of its own).
    WalkArgs& w = B.wa;
    w.traj = o.traj_E;
    w.moves = o.moves;
    w.hit = A.hit;
    w.evals = A.evals;
    w.log_every = A.log_every;
    w.MW = A.MW;
    w.log_seqs = A.log_seqs;
    w.log_mask = A.log_mask;
    w.log_label = A.log_label;
    const bool packed = mlp && mlp_packs(lay);
    if (F > 1 && c.steps > 1 && packed && (s = mlp_pack(lay, pr.params_bf16, B.fwd_ws, B.fwd_bytes, st))) return s;
    for (int t = 1; t <= c.steps;) {
        if ((t - 1) % F == 0) {
            w.t0 = t - 1;
            w.t1 = F > 1 ? t : (t - 1 + kLogSegment < c.steps ? t - 1 + kLogSegment : c.steps);
            if ((s = launch_walk_log(w, st))) return s;
            t = w.t1 + 1;
            if (F > 1) {
                A.t = w.t1;
                hipLaunchKernelGGL(k_lw_corr, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, A);
                LABS_LAUNCHED("k_lw_corr");
            }
            continue;
        }
        if (packed) {
            s = mlp_forward_state(lay, pr.params, B.fwd_ws, n, A.seq, A.C, A.ldc, const_cast<float*>(A.logits), st);
        } else if (mlp) {
            s = launch_features(c.L, n, A.seq, B.X, lay.ld_in, st);
            if (!s) s = mlp_forward(lay, pr.params, pr.params_bf16, n, B.X, const_cast<float*>(A.logits), B.fwd_ws,
                                    B.fwd_bytes, st);
        }
        if (s) return s;
        A.t = t++;
        if ((s = launch_lw_step(A, st))) return s;
    }
    if (F == 1 && o.cands) {
        const int64_t cn = n * c.steps * A.top_m;
        hipLaunchKernelGGL(k_fill_i16, dim3((unsigned)(cn / 256 + 1 < 65536 ? cn / 256 + 1 : 65536)), dim3(256), 0, st,
                           cn, o.cands, (int16_t)-1);
        LABS_LAUNCHED("k_fill_i16");
    }

    hipLaunchKernelGGL(k_lw_outputs, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, A, o.final_seqs,
                       o.final_E, o.best_seqs, o.best_E, o.best_step, o.hit_step);
    LABS_LAUNCHED("k_lw_outputs");
    hipLaunchKernelGGL(k_sum_i64, dim3(1), dim3(1024), 0, st, n, A.evals, o.flip_evals);
    LABS_LAUNCHED("k_sum_i64");
    return LABS_OK;
}

}  // namespace labsdev
