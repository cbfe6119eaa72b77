// Templates of the first-step walker (shared by the instantiation units).
// See walk.hip for the method and the notation.
#pragma once
#include "labs_internal.h"

#include <climits>

namespace labsdev {
namespace walkimpl {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef short v2s __attribute__((ext_vector_type(2)));

// a * b, |a|, |b| < 2^23, one instruction with a sum behind it (the intrinsic, not inline
// assembly: the compiler has to see the hazards behind dot and matrix products).
extern "C" __device__ int labs_mul_i24(int a, int b) __asm("llvm.amdgcn.mul.i24.i32");
extern "C" __device__ int labs_mul_u24(int a, int b) __asm("llvm.amdgcn.mul.u24.i32");

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// X holds, for class cl and shift i = 0..7, row cl*8 + i: byte kap is x_cl[i + kap - kz]
// (0 outside the sequence), so any dword or 8-byte run of a class is one aligned
// read of the row with the matching shift; each row ends in 16 zero bytes or more.  A row
// length of 2 mod 4 units of 16 bytes keeps the 16-byte operand reads free of bank
// conflicts (the 16 lanes served together are eight rows at one step and eight at the next;
// at odd lengths they take twice the cycles), so rows are 32 bytes longer at even KH:
// 16,384 walkers at L = 301 3.61 -> 3.56 us a step, L = 451 4.16 -> 4.07.  At odd KH that
// takes 64 bytes, and the LDS costs a wave (L = 501 4.30 -> 4.59); so it does beside a
// Bloom filter.
// D holds -C_{2|t|} at db + t (0 at t = 0), low bytes; DH the bytes above them.
// T holds the tabu deadlines of the slots, four of a lane in one 16-byte read (with a
// Bloom filter there are none).
template <int KH, int NT, int NQ, bool BL = false>
struct Lds {
    static constexpr int ROW = 32 * KH;
    static constexpr int ST = ROW + (BL || (KH & 1) ? 16 : 32);
    static constexpr int DNEG = NQ == 1 ? 336 : 520;
    static constexpr int DPOS = (ROW > 256 * NQ ? ROW : 256 * NQ) + 32;
    int8_t D[DNEG + DPOS] __attribute__((aligned(16)));   // first: short offsets of paired reads
    int8_t DH[DNEG + DPOS] __attribute__((aligned(16)));
    int8_t guard[16] __attribute__((aligned(16)));        // zeros before the first row
    int8_t X[16 * ST];
    int32_t T[BL ? 4 : 256 * NT] __attribute__((aligned(16)));
    uint32_t pk[24];
};

// Zobrist words of the free positions (zobrist_at), a table in constant memory.
struct ZobristTable {
    uint64_t z[320];
};
constexpr uint64_t zobrist_const(uint64_t i) {
    uint64_t x = kZobristState + (i + 1ull) * 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
constexpr ZobristTable zobrist_table() {
    ZobristTable t{};
    for (int i = 0; i < 320; ++i) t.z[i] = zobrist_const((uint64_t)i);
    return t;
}
static __device__ const ZobristTable g_zobrist = zobrist_table();

// Minimum over the wavefront (all lanes active), wave-uniform.
__device__ __forceinline__ int wave_min(int v) {
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// Index of the first slot: the first free position's, or one before it.
__host__ __device__ inline int first_index(int k, int p) {
    const int nmin = p >> 1;
    const int want = ((k & 1) ? (k - 3) >> 1 : k >> 1) & 1;
    return (nmin & 1) == want ? nmin : nmin - 1;
}

// One walker (walker index j of configuration A) for steps t0+1..t1.
// BL: self-avoidance by the walker's Bloom filter (copied into `bl` in LDS for the
// segment) instead of the tabu tenure.  LG: the training log's outputs.
template <int KH, int NT, int NQ, bool BL, bool LG>
__device__ __forceinline__ void walk_body(const WalkArgs& A, int64_t j, Lds<KH, NT, NQ, BL>& S, uint32_t* bl) {
    typedef Lds<KH, NT, NQ, BL> T;
    constexpr int ST = T::ST, ROW = T::ROW;
    const int lane = threadIdx.x & 63;
    const int L = A.L, k = A.k, p = A.p, W = A.W, nf = A.nf;
    const int t0 = A.t0, t1 = A.t1;

    int halted = A.halted[j];
    if (halted) {
        for (int t = t0 + 1 + lane; t <= t1; t += 64) {
            if (A.traj) A.traj[j * A.steps_total + (t - 1)] = -1;
            if constexpr (LG)
                if (A.moves) A.moves[j * A.steps_total + (t - 1)] = -1;
        }
        return;
    }
    int vpk = lane < W ? (int)A.seq[j * W + lane] : 0;
    int vbest = lane < W ? (int)A.bestSeq[j * W + lane] : 0;
    lds_order();
    if (lane < 24) S.pk[lane] = (uint32_t)vpk;
    if (lane < 4) ((int*)S.guard)[lane] = 0;
    for (int i = lane; i < (T::DNEG + T::DPOS) / 4; i += 64) {
        ((int*)S.D)[i] = 0;
        ((int*)S.DH)[i] = 0;
    }
    lds_order();

    // ---- geometry (wave-uniform).  Slot positions: class cl (0: odd x, 1: even x),
    // index n = (x - 1) >> 1 = n0 + 128 tau + 8 j + i; the parity of n0 lets a lane read
    // the C_{2mp} of its four slots from two aligned dwords (see coff below).
    const int nc = k >> 1, cc = k & 1;
    const int n0 = first_index(k, p);
    const int kz = 8 + ((3 - n0) & 3);
    const int db = T::DNEG + ((n0 + kz) & 7);
    int kz1 = kz + 1, kzm = kz - 4;
    asm("" : "+s"(kz1), "+s"(kzm));
    const int lj = lane & 15, lg = lane >> 4;
    const int cl = lg >> 1;
    const int nb = n0 + 8 * lj + 4 * (lg & 1);

    // ---- the class rows
    for (int i = lane; i < 16 * ST / 4; i += 64) {
        const int row = i / (ST / 4), kap = 4 * (i - row * (ST / 4));
        const int rc = row >> 3, n = (row & 7) + kap - kz;
        uint32_t v = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int x = 2 * (n + b) + 1 + rc;
            if (n + b >= 0 && x <= L && kap < ROW) v |= (packed_bit(S.pk, x) ? 0x01u : 0xFFu) << (8 * b);
        }
        ((uint32_t*)S.X)[i] = v;
    }
    // ---- -C_{2m} of this lane's m = 4 lane + 1 .. + 4 (group q: + 256), packed 16-bit
    v2s c01[NQ], c23[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        int c[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int m = 256 * q + 4 * lane + 1 + b;
            c[b] = m <= k ? -packed_corr(S.pk, L, 2 * m) : 0;
        }
        c01[q] = v2s{(short)c[0], (short)c[1]};
        c23[q] = v2s{(short)c[2], (short)c[3]};
    }
    lds_order();

    // Stores the C tables: low bytes, and the bytes above them while `wide`.
    auto store_c = [&](bool wide) {
        int last = 0;                             // the dword before lane 0's
        auto shifted = [&](uint32_t f, int q) -> uint32_t {     // wave_shr:1
            return q == 0 ? (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, 0x138, 0xf, 0xf, true)
                          : (uint32_t)__builtin_amdgcn_update_dpp(last, (int)f, 0x138, 0xf, 0xf, false);
        };
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t u01 = __builtin_bit_cast(uint32_t, c01[q]), u23 = __builtin_bit_cast(uint32_t, c23[q]);
            const uint32_t f = __builtin_amdgcn_perm(u23, u01, 0x06040200u);
            *(uint32_t*)(S.D + db + 256 * q + 4 * lane + 1) = f;
            const uint32_t prev = shifted(f, q);
            *(uint32_t*)(S.D + db - 256 * q - 4 * lane - 3) = __builtin_amdgcn_perm(prev, f, 0x07000102u);
            if (q + 1 < NQ) last = __builtin_amdgcn_readlane((int)f, 63);
        }
        if (wide) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                // the low byte is signed, so the high part is (C + 128) >> 8
                const v2s bias = {128, 128};
                const uint32_t f = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, (v2s)(c23[q] + bias)),
                                                         __builtin_bit_cast(uint32_t, (v2s)(c01[q] + bias)), 0x07050301u);
                *(uint32_t*)(S.DH + db + 256 * q + 4 * lane + 1) = f;
                const uint32_t prev = shifted(f, q);
                *(uint32_t*)(S.DH + db - 256 * q - 4 * lane - 3) = __builtin_amdgcn_perm(prev, f, 0x07000102u);
                if (q + 1 < NQ) last = __builtin_amdgcn_readlane((int)f, 63);
            }
        }
    };
    // Whether some C may leave [-128, 127] within the next four steps (a step moves
    // a C by at most 8).
    auto need_wide = [&]() -> bool {
        uint32_t any = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const v2s bias = {96, 96};            // -96 <= C <= 95  <=>  0 <= C + 96 < 192
            const uint32_t t01 = __builtin_bit_cast(uint32_t, (v2s)(c01[q] + bias));
            const uint32_t t23 = __builtin_bit_cast(uint32_t, (v2s)(c23[q] + bias));
            any |= (t01 | t23) & 0xFF00FF00u;
            any |= ((t01 & (t01 << 1)) | (t23 & (t23 << 1))) & 0x00800080u;   // 192..255
        }
        return __ballot(any != 0) != 0;
    };
    bool wide = need_wide();
    store_c(wide);

    // ---- slots
    const int sig = ((k - cl) & 1) ? -1 : 1;      // s_a s_b of a free pair (Eq. (2))
    // weights of a byte of a dword (kept in registers, not shifted each step)
    int w40 = (-4 * sig) & 0xFF, w41 = w40 << 8, w42 = w40 << 16, w43 = w40 << 24;
    asm("" : "+v"(w40), "+v"(w41), "+v"(w42), "+v"(w43));
    int az[NT][4];                                // a - 1 of the lane's slots
    int Y[NT][4];                                 // dE/4 without the terms in H and C
    int sgs[NT][4];                               // 1, the centre 0
    int least[NT][4];                             // Bloom: INT_MIN, where no slot is INT_MAX
    int xso[NT], xeo[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int n1 = nb + 128 * u;
        // the slots' own elements (four consecutive indices), and x_cl[3n - k + cl],
        // the backward element at the partner's lag (bytes 0, 3, 6, 9 of 12)
        const int is = (n0 + kz) & 3, ks = n1 + kz - is;
        xso[u] = ks < ROW ? (cl * 8 + is) * ST + ks : ROW;
        const int e = 3 * n1 - k + cl + kz, ie = e & 3;
        xeo[u] = (e - ie >= -16 && e - ie <= ROW + 4) ? (cl * 8 + ie) * ST + e - ie : ROW;
        v4i tb;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = n1 + r, x = 2 * n + 1 + cl;
            const bool valid = n >= 0 && x > p && x <= k + 1;
            const int i = x - p - 1;
            tb[r] = !valid ? INT_MAX : BL ? 0 : A.tabu[j * nf + i];
            least[u][r] = valid ? INT_MIN : INT_MAX;
            // sum_m x[n + m] x[n - m]
            int y = 0;
            if (valid) {
                const int uf = n + 1 + kz, rf = cl * 8 + (uf & 3);
                const int ub = n - 4 + kz, rb = cl * 8 + (ub & 3);
                int of = rf * ST + uf - (uf & 3), ob = rb * ST + ub - (ub & 3);
                for (int m = 0; m < n; m += 4) {
                    const uint32_t f = *(const uint32_t*)(S.X + of);
                    const uint32_t b = *(const uint32_t*)(S.X + (ob < rb * ST ? rb * ST : ob));
                    y = __builtin_amdgcn_sdot4((int)f, (int)__builtin_amdgcn_perm(b, b, 0x00010203u), y, false);
                    of += 4;
                    ob -= 4;
                }
            }
            const bool centre = x == k + 1;
            Y[u][r] = centre ? 4 * nc + 4 : 4 * (k - cl - 1) + 8 * y;
            sgs[u][r] = centre ? 0 : 1;
            asm("" : "+v"(sgs[u][r]));
            az[u][r] = 2 * n + cl;
            asm("" : "+v"(az[u][r]));             // kept, not recomputed each step
        }
        if constexpr (!BL) *(v4i*)(S.T + cl * 128 * NT + 128 * u + 8 * lj + 4 * (lg & 1)) = tb;
    }
    const int aoff = (lane & 15) * ST + 16 * lg;
    const int boff = db + 16 * lg - kz - n0 - 8 * lj;
    // C_{2mp}, mp = k - cl - 2n, of slots 0 and 1 (2 and 3): every other byte of two
    // aligned dwords, for even k at +mp (falling with n), for odd k at -mp (rising)
    const bool rise = k & 1;
    const int cw0 = db + (rise ? 2 * nb + cl - k : k - cl - 2 * nb - 6);   // first byte, 0 or 1 mod 4
    const int co01 = (cw0 & ~3) + (rise ? 0 : 4), co23 = (cw0 & ~3) + (rise ? 4 : 0);
    const int cstep = rise ? 256 : -256;
    const int cwA = ((-2 * sig) & 0xFF) << (8 * ((cw0 & 1) + (rise ? 0 : 2)));
    const int cwB = ((-2 * sig) & 0xFF) << (8 * ((cw0 & 1) + (rise ? 2 : 0)));
    const int toff = cl * 128 * NT + 8 * lj + 4 * (lg & 1);

    // byte of the row (shift lane & 7) that holds index n of class 0, less n
    const int xwl = (lane & 7) * ST + kz - (lane & 7);
    const int second = (lane >> 3) & 1;           // lanes 8..15 write the partner
    // Word `lane` of the packed sequence, from the class rows (16 indices of each
    // class a word; the bits of +1 bytes, lowest index first)
    auto packed_words = [&]() -> int {
        uint32_t bits[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint32_t v = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i0 = kz & 3;
                const int kap = 16 * (lane < W ? lane : 0) + 4 * q + kz - i0;
                const uint32_t d = *(const uint32_t*)(S.X + (c * 8 + i0) * ST + (kap < ROW ? kap : ROW));
                // +1 is 0x01, -1 is 0xFF, outside 0: bit 0 of the byte and not bit 7
                const uint32_t one = d & ~(d >> 7) & 0x01010101u;
                v |= ((one * 0x08040201u) >> 24) << (4 * (3 - q));   // bit 3 - b: byte b
            }
            bits[c] = v;                          // bit 15 - (n mod 16)
        }
        uint32_t w = 0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint32_t v = bits[c];
            v = (v | (v << 8)) & 0x00FF00FFu;
            v = (v | (v << 4)) & 0x0F0F0F0Fu;
            v = (v | (v << 2)) & 0x33333333u;
            v = (v | (v << 1)) & 0x55555555u;
            w |= v << (1 - c);
        }
        return (int)w;
    };

    uint32_t* gbl = nullptr;
    const int nbw = BL ? 1 << (A.bloom_log2 - 5) : 0;
    const uint32_t bmask = BL ? (1u << A.bloom_log2) - 1u : 0u;
    const int nh = BL ? A.bloom_hashes : 0;
    const int probe = lane < nh ? lane : nh - 1;   // every lane tests a bit, some the same
    uint64_t hk = 0;
    if constexpr (BL) {
        gbl = A.bloom + j * (int64_t)nbw;
        for (int i = lane; i < nbw; i += 64) bl[i] = gbl[i];
        hk = A.zh[j];
        lds_order();
    }
    int E = uni(A.E[j]);
    int bestE = uni(A.bestE[j]);
    int bestT = uni(A.bestT[j]);
    // Bloom: undoing the last move returns to a sequence the filter holds (no false
    // negatives), so the last slot is out for one step without a probe
    int last = -1;
    const int tenure = BL ? 0 : uni(A.tenure[j]);
    const int thr = !LG && A.e_max >= 0 ? A.e_max : INT_MIN;   // sieve threshold
    const int64_t wid = A.walker_begin + j;
    int pend = pending_level(A);          // first-hit stamps: largest level energy above E
    int rare = uni(max(max(pend, thr), bestE - 1));   // energies above need no bookkeeping
    int hit = 0, logr = 0, lognext = 0;
    int64_t evals = 0;
    if constexpr (LG) {
        hit = uni(A.hit[j]);
        evals = A.evals[j];
        if (A.log_every > 0) {
            logr = t0 / A.log_every;
            lognext = (logr + 1) * A.log_every;
        }
    }

    // One 16x16 tile: rows (class, n mod 8) of X against columns (n div 8) of a table of
    // D; 64 indices a product, the last 32 alone when KH is odd.
    v4i at = {0, 0, 0, 0}, bt = {0, 0, 0, 0};
    asm("" : "+v"(at), "+v"(bt));
    auto product = [&](const int8_t* pb) -> v4i {
        v4i h = {0, 0, 0, 0};
#pragma unroll
        for (int m = 0; m < KH / 2; ++m) {
            const v4i a = *(const v4i*)(S.X + aoff + 64 * m);
            const v2i b0 = *(const v2i*)(pb + 64 * m), b1 = *(const v2i*)(pb + 64 * m + 8);
            const v4i b = {b0.x, b0.y, b1.x, b1.y};
            h = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, h, 0, 0, 0);
        }
        if constexpr (KH & 1) {
            // the same product (another shape must not follow it on one accumulator)
            // with zeros in the upper half of each lane's bytes
            const v2i a = *(const v2i*)(S.X + aoff + 32 * (KH - 1) - 8 * lg);
            const v2i b = *(const v2i*)(pb + 32 * (KH - 1) - 8 * lg);
            at.x = a.x;
            at.y = a.y;
            bt.x = b.x;
            bt.y = b.y;
            h = __builtin_amdgcn_mfma_i32_16x16x64_i8(at, bt, h, 0, 0, 0);
        }
        return h;
    };
    int32_t* const traj = A.traj ? A.traj + j * A.steps_total : nullptr;
    for (int t = t0 + 1; t <= t1; ++t) {
        // ---- H[n] = minus the sum over the class of x[n'] C_{2|n' - n|}
        v4i H[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) H[u] = product(S.D + boff - 128 * u);
        int key[NT][4], xs[NT];
        int kmin = INT_MAX;
        int ncand = 0;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            xs[u] = *(const int*)(S.X + xso[u]);
            const int* pe = (const int*)(S.X + xeo[u]);
            const int e0 = pe[0], e1 = pe[1], e2 = pe[2];
            const int cd0 = *(const int*)(S.D + co01 + cstep * u), cd1 = *(const int*)(S.D + co23 + cstep * u);
            v4i tb = {0, 0, 0, 0};
            if constexpr (!BL) tb = *(const v4i*)(S.T + toff + 128 * u);
            if (wide) {
                const v4i Hh = product(S.DH + boff - 128 * u);
                const int ch0 = *(const int*)(S.DH + co01 + cstep * u), ch1 = *(const int*)(S.DH + co23 + cstep * u);
                int gw[4];
                gw[0] = __builtin_amdgcn_sdot4(ch0, cwA, 0, false);
                gw[1] = __builtin_amdgcn_sdot4(ch0, cwB, 0, false);
                gw[2] = __builtin_amdgcn_sdot4(ch1, cwA, 0, false);
                gw[3] = __builtin_amdgcn_sdot4(ch1, cwB, 0, false);
                // the partner's term joins H here: s (128 s gw) 2 = 256 gw (0 at the centre)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int s = (int)((uint32_t)xs[u] << (24 - 8 * r)) >> 24;
                    H[u][r] += 256 * Hh[r] + s * 128 * gw[r];
                }
            }
            int v[4];
            v[0] = __builtin_amdgcn_sdot4(e0, w40, H[u][0], false);
            v[1] = __builtin_amdgcn_sdot4(e0, w43, H[u][1], false);
            v[2] = __builtin_amdgcn_sdot4(e1, w42, H[u][2], false);
            v[3] = __builtin_amdgcn_sdot4(e2, w41, H[u][3], false);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // dE/4 = Y - 2 s_a s_b C_{2mp} + 2 s v (the centre: Y + s v), and the order
                // key 512 dE/8 + (a - 1)
                const int s = (int)((uint32_t)xs[u] << (24 - 8 * r)) >> 24;
                int d = (labs_mul_i24(s, v[r]) << sgs[u][r]) + Y[u][r];
                d = __builtin_amdgcn_sdot4(r < 2 ? cd0 : cd1, r & 1 ? cwB : cwA, d, false);
                const int kk = (d << 8) + az[u][r];
                if constexpr (BL) {
                    key[u][r] = az[u][r] == last ? INT_MAX : max(kk, least[u][r]);
                } else {
                    const bool adm = tb[r] < t;
                    if constexpr (LG) ncand += __popcll(__ballot(adm));
                    key[u][r] = adm ? kk : INT_MAX;
                }
                if constexpr (!BL) kmin = min(kmin, key[u][r]);
            }
        }
        uint64_t hnext = 0;
        uint32_t bsel = 0;        // Bloom: this lane's bit of the chosen key
        if constexpr (!BL) {
            kmin = wave_min(kmin);
        } else {
            // the lowest (dE, a) not in the filter: the best candidate is tested (probe q
            // on lane q), a member is excluded and the next best taken, so each pass
            // removes one slot and the loop ends
            for (;;) {
                kmin = INT_MAX;
#pragma unroll
                for (int u = 0; u < NT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) kmin = min(kmin, key[u][r]);
                kmin = wave_min(kmin);
                if (kmin == INT_MAX) break;
                const uint64_t hkey = hk ^ g_zobrist.z[kmin & 511];
                // at most 2^18 bits, so the low 24 bits of the product are enough
                bsel = ((uint32_t)hkey + (uint32_t)labs_mul_u24(probe, (int)((uint32_t)(hkey >> 32) | 1u))) & bmask;
                if (__ballot(!((bl[bsel >> 5] >> (bsel & 31)) & 1u))) {
                    hnext = hkey;
                    break;
                }
#pragma unroll
                for (int u = 0; u < NT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (key[u][r] == kmin) key[u][r] = INT_MAX;
            }
        }
        if (kmin == INT_MAX) {
            halted = t;
            break;
        }
        E += 8 * (kmin >> 9);
        // ---- the flipped pair: class cs, indices n and nbs
        const int z = kmin & 511, n = z >> 1, cs = z & 1;
        last = z;
        const int q = n - n0;
        const int nbs = k - n - cs;
        const bool cen = n == nbs;
        const int ow = ((cs * 2 + ((q >> 2) & 1)) << 4) | ((q >> 3) & 15);
        int sd = __builtin_amdgcn_readlane(xs[0], ow);
        if (NT > 1 && q >= 128) sd = __builtin_amdgcn_readlane(xs[NT - 1], ow);
        const int sa = (sd << (24 - 8 * (q & 3))) >> 24;
        const int sb = ((k - cs) & 1) ? -sa : sa;

        if constexpr (LG) {
            evals += ncand;
            if (t == lognext) {
                const int64_t rec = (int64_t)logr * A.n + j;
                ++logr;
                lognext += A.log_every;
                const int word = packed_words();
                if (lane < W) A.log_seqs[rec * W + lane] = (uint32_t)word;
                if (lane < 24) S.pk[lane] = 0;
                lds_order();
#pragma unroll
                for (int u = 0; u < NT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (key[u][r] != INT_MAX) {
                            const int pos = 2 * (nb + 128 * u + r) + cl;
                            atomicOr(&S.pk[pos >> 5], 1u << (pos & 31));
                        }
                lds_order();
                if (lane < A.MW) A.log_mask[rec * A.MW + lane] = S.pk[lane];
                if (lane == 0) A.log_label[rec] = z;
            }
            if (A.moves && lane == 0) A.moves[j * A.steps_total + (t - 1)] = z + 1;
        }

        // ---- the pair's bytes are zero while the other elements are read: u_m is
        // without the partner, and a slot's own product does not enter Y
        int8_t* const xw = S.X + (xwl + labs_mul_i24(second, nbs - n) + (cs * 8 * ST + n));
        lds_order();
        if (lane < 16) {
            *xw = 0;
            if constexpr (!BL) S.T[cs * 128 * NT + q] = t + tenure;
        }
        lds_order();
        // ---- Y: the pairs (n_f, 2 na - n_f) of each flipped index n_f change sign
        v2i yd[NT][2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int nfl = e ? nbs : n;
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                const int s0 = 2 * (n0 + 128 * u) - nfl + kz;
                const int row = cs * 8 + (s0 & 7);
                const int off = 16 * lj + 8 * (lg & 1) + (s0 - (s0 & 7));
                const bool in = (unsigned)off < (unsigned)ROW && cl == cs;
                yd[u][e] = *(const v2i*)(S.X + (in ? row * ST + off : ROW));
            }
        }
        // ---- C_{2m} -= 4 s u_m (the centre alone: the backward element only, and there
        // forward and backward are equal)
        {
            const int uf = n + kz1, rf = cs * 8 + (uf & 3);
            const int ub = n + kzm, rb = cs * 8 + (ub & 3);
            const short mul = (short)(cen ? 2 * sa : 4 * sa);
            const v2s mul2 = {mul, mul};
#pragma unroll
            for (int g = 0; g < NQ; ++g) {
                const uint32_t f = *(const uint32_t*)(S.X + rf * ST + min((uf & ~3) + 4 * lane + 256 * g, ROW));
                v2s u01 = __builtin_bit_cast(v2s, __builtin_amdgcn_perm(f, f, 0x010C000Cu));
                v2s u23 = __builtin_bit_cast(v2s, __builtin_amdgcn_perm(f, f, 0x030C020Cu));
                if (g == 0) {                     // backward lags end at n < 256
                    const uint32_t b = *(const uint32_t*)(S.X + rb * ST + max((ub & ~3) - 4 * lane, 0));
                    u01 += __builtin_bit_cast(v2s, __builtin_amdgcn_perm(b, b, 0x020C030Cu));
                    u23 += __builtin_bit_cast(v2s, __builtin_amdgcn_perm(b, b, 0x000C010Cu));
                }
                c01[g] += (u01 >> 8) * mul2;
                c23[g] += (u23 >> 8) * mul2;
            }
        }
        lds_order();
        if (lane < 16) *xw = (int8_t)(second * (sa - sb) - sa);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int wgt = (e ? (cen ? 0 : -16 * sb) : -16 * sa) & 0xFF;
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                Y[u][0] = __builtin_amdgcn_sdot4(yd[u][e].x, wgt, Y[u][0], false);
                Y[u][1] = __builtin_amdgcn_sdot4(yd[u][e].x, wgt << 16, Y[u][1], false);
                Y[u][2] = __builtin_amdgcn_sdot4(yd[u][e].y, wgt, Y[u][2], false);
                Y[u][3] = __builtin_amdgcn_sdot4(yd[u][e].y, wgt << 16, Y[u][3], false);
            }
        }
        if ((t & 3) == 0) wide = need_wide();
        store_c(wide);
        if constexpr (BL) {
            // insert the new sequence's key
            hk = hnext;
            if (lane < nh) atomicOr(&bl[bsel >> 5], 1u << (bsel & 31));
        }
        lds_order();
        if (traj) {
            if (lane == 0) traj[t - 1] = E;
        }
        if constexpr (LG) {
            if (hit < 0 && A.e_max >= 0 && E <= A.e_max) hit = t;
        }
        if (E > rare) continue;
        if (E < bestE) {
            bestE = E;
            bestT = t;
            vbest = packed_words();
        }
        if (E <= pend) pend = stamp_levels(A, E, lane);
        if (E <= thr) {
            uint32_t slot = 0;
            if (lane == 0) slot = atomicAdd(A.st_count, 1u);
            slot = (uint32_t)uni((int)slot);
            const int word = __shfl(packed_words(), lane - 1, 64);
            if (slot < A.st_cap && lane < W + 3) {
                uint32_t v;
                if (lane == 0) v = (uint32_t)E;
                else if (lane <= W) v = (uint32_t)word;
                else if (lane == W + 1) v = (uint32_t)wid;
                else v = (uint32_t)t;
                A.rec[(int64_t)lane * A.rec_stride + slot] = v;
            }
        }
        rare = uni(max(max(pend, thr), bestE - 1));
    }
    if (halted)
        for (int t = halted + lane; t <= t1; t += 64) {
            if (A.traj) A.traj[j * A.steps_total + (t - 1)] = -1;
            if constexpr (LG)
                if (A.moves) A.moves[j * A.steps_total + (t - 1)] = -1;
        }
    vpk = packed_words();
    if (lane < W) {
        A.seq[j * W + lane] = (uint32_t)vpk;
        A.bestSeq[j * W + lane] = (uint32_t)vbest;
    }
    if constexpr (BL) {
        for (int i = lane; i < nbw; i += 64) gbl[i] = bl[i];
        if (lane == 0) A.zh[j] = hk;
    } else {
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int x = 2 * (nb + 128 * u + r) + 1 + cl;
                if (x > p && x <= k + 1) A.tabu[j * nf + x - p - 1] = S.T[toff + 128 * u + r];
            }
    }
    if (lane == 0) {
        A.E[j] = E;
        A.bestE[j] = bestE;
        A.bestT[j] = bestT;
        A.halted[j] = halted;
        if constexpr (LG) {
            A.hit[j] = hit;
            A.evals[j] = evals;
        }
    }
}

// Waves per SIMD the registers are held to: what the LDS (7.3 KB a walker at KH = 9,
// 160 KB a CU) lets reside.  Fewer registers for one wave more spill and gain nothing,
// since issue is the bound (16,384 walkers, us a step: seven waves in place of six at
// L = 301 3.7 -> 4.0, eight at L = 201 3.48 -> 3.55).
template <int KH, int NT>
struct WavesPerSimd {
    static constexpr int value = NT == 2 ? 3 : KH >= 11 ? 4 : KH >= 9 ? 5 : 6;
};

template <int KH, int NT, int NQ>
__global__ __launch_bounds__(64, (WavesPerSimd<KH, NT>::value)) void k_walk(WalkArgs A) {
    __shared__ Lds<KH, NT, NQ> S;
    walk_body<KH, NT, NQ, false, false>(A, blockIdx.x, S, nullptr);
}

// Bloom-filter form: the walker's filter (2^bloom_log2 bits) in dynamic LDS, which decides
// how many walkers reside; without the tabu deadlines a walker takes 1 KB less.  Registers
// for five waves where the plain walk has six: 16,384 walkers at L = 451, us a step at 2^12,
// 2^13, 2^15, 2^16 bits: 5.28, 5.13, 5.93, 7.35 (six 4.99, 5.28, 6.08, 7.47; with the
// deadlines in LDS 5.44, 5.72, 6.53, 7.95).  At 2^15 bits a walker-step takes 123 vector and
// 126 scalar instructions and 112 LDS cycles, 0.55 of the VALU's and 0.50 of the LDS's time:
// neither is full, the probes' chain and too few waves to cover it are the bound.
template <int KH, int NT, int NQ>
__global__ __launch_bounds__(64, (WavesPerSimd<KH, NT>::value > 5 ? 5 : WavesPerSimd<KH, NT>::value)) void k_walk_bloom(WalkArgs A) {
    __shared__ Lds<KH, NT, NQ, true> S;
    extern __shared__ uint32_t bloom_words[];
    walk_body<KH, NT, NQ, true, false>(A, blockIdx.x, S, bloom_words);
}

// The plain walk with the learned walk's outputs: moves, first hit, evaluations (the
// admissible positions of every step) and the training log.
template <int KH, int NT, int NQ>
__global__ __launch_bounds__(64, (WavesPerSimd<KH, NT>::value)) void k_walk_log(WalkArgs A) {
    __shared__ Lds<KH, NT, NQ> S;
    walk_body<KH, NT, NQ, false, true>(A, blockIdx.x, S, nullptr);
}

// Persistent form: each wavefront takes (configuration, walker) items from a
// queue until it is empty, so every wavefront exits.
template <int KH, int NT, int NQ>
__global__ __launch_bounds__(64, (WavesPerSimd<KH, NT>::value)) void k_walk_persistent(const WalkArgs* __restrict__ args, const int2* items,
                                                        int n_items, unsigned* head) {
    __shared__ Lds<KH, NT, NQ> S;
    for (;;) {
        unsigned it = 0;
        if (threadIdx.x == 0) it = atomicAdd(head, 1u);
        // a wave-uniform item (readfirstlane, not a shuffle), so the item and its
        // configuration's arguments load into scalar registers as a plain launch's do
        it = __builtin_amdgcn_readfirstlane(it);
        if (it >= (unsigned)n_items) break;
        const int2 w = items[it];
        // by reference: the fields load on demand, as from a plain launch's arguments
        const WalkArgs& A = args[__builtin_amdgcn_readfirstlane(w.x)];
        walk_body<KH, NT, NQ, false, false>(A, (int64_t)w.y, S, nullptr);
    }
}

typedef void (*walk_kernel_t)(WalkArgs);
typedef void (*walk_persistent_t)(const WalkArgs*, const int2*, int, unsigned*);

}  // namespace walkimpl

// Kernels of the shape class of (L, p).  KH: the class rows in units of 32 indices,
// NT: 128-index tiles of slots a class, NQ: groups of 256 lags.
struct WalkKernels {
    walkimpl::walk_kernel_t plain, bloom, log;
    walkimpl::walk_persistent_t persistent;
};
struct WalkShape {
    int KH, NT, NQ;
};
// A row has to hold the k + 1 indices of a class, its shift (up to 7) and the zeros
// before the first element (up to 11, see kz).
inline WalkShape walk_shape(int L, int p) {
    const int k = (L - 1) / 2;
    WalkShape s;
    s.KH = k + 12 <= 64 ? 2 : (k + 12 + 31) / 32;
    s.NT = (k >> 1) - walkimpl::first_index(k, p) + 1 > 128 ? 2 : 1;
    s.NQ = k > 256 ? 2 : 1;
    return s;
}
bool walk_kernels(const WalkShape& s, WalkKernels* out);
bool walk_kernels_a(int KH, WalkKernels* out);                    // KH 2..5
bool walk_kernels_b(int KH, WalkKernels* out);                    // KH 6..8
bool walk_kernels_c(int KH, int NT, int NQ, WalkKernels* out);    // KH 9..11

}  // namespace labsdev
