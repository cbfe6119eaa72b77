// The first-step walk for short sequences: G walkers a wavefront (see walk.hip for the
// method and the notation; tabu tenure, no log).
//
// A walk at L = 101 has 43 slots and 50 lags, so one walker a wave leaves most lanes of
// every vector instruction idle, and the issue of those instructions is what bounds a
// walk.  Here a walker takes 64 / G lanes: its four consecutive slots a lane are G times
// fewer columns, its lags four a lane as before.  One 16x16 tile holds G walkers by rows,
// R = 16 / G shifted copies of a class each:
//   A_w[(w', i)][kap] = x_cl[i + kap - kz] of walker w for w' = w, else 0,
//   B_w[kap][j] = C_{2|kap - kz - n0 - R (j & 7)|} of walker w,
// and the sum of the G products is H of every walker: rows 4 lg .. + 3 of columns 0..7 for
// class 0, the same with the copies of class 1 in columns 8..15.  So a lane's walker is its
// row of 16 lanes (G = 4) or half of the wave (G = 2), and what a wave decides for one
// walker with scalars a group decides in its lanes.
// Bound by issue and the LDS together: a wave and step take 169 vector and 51 scalar
// instructions and 146 LDS cycles with four walkers (0.77 of the VALU's time, 0.67 of the
// LDS's), 155 LDS cycles with two (0.78, 0.72); reading each copy once and masking it instead
// changes nothing.  65,536 walkers at L = 101: 12.6 us a step with a wave a walker, 5.4 here.
#include "walk_impl.h"

namespace labsdev {
namespace walkimpl {

// LDS of one walker of a group (KB: 64-byte blocks of a class row).
template <int KB, int G>
struct GroupLds {
    static constexpr int R = 16 / G;
    static constexpr int ROW = 64 * KB, ST = ROW + 16;
    static constexpr int DNEG = 16 * R + 32, DPOS = (ROW > 16 * R ? ROW : 16 * R) + 48;
    int8_t D[DNEG + DPOS] __attribute__((aligned(16)));
    int8_t DH[DNEG + DPOS] __attribute__((aligned(16)));
    int8_t guard[16] __attribute__((aligned(16)));
    int8_t X[2 * R * ST];
    int32_t T[16 * R] __attribute__((aligned(16)));
    uint32_t pk[12];
};

template <int KB, int G>
struct GroupWave {
    typedef GroupLds<KB, G> W;
    W w[G];
    // what the rows of other walkers read: zeros for both classes' copies
    int8_t zero[W::R * W::ST + W::ROW] __attribute__((aligned(16)));
};

// Minimum over the lanes of a walker, in all of them.
template <int G>
__device__ __forceinline__ int group_min(int v) {
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true));    // pairs
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true));    // quads
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true));   // halves of 8
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true));   // rows of 16
    if constexpr (G == 2) {
        const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
        v = min((int)r[0], (int)r[1]);
    }
    return v;
}

template <int KB, int G>
__global__ __launch_bounds__(64, 4) void k_walk_group(WalkArgs A) {
    typedef GroupLds<KB, G> T;
    constexpr int R = T::R, ST = T::ST, ROW = T::ROW, LW = 64 / G;   // lanes a walker
    __shared__ GroupWave<KB, G> SW;
    const int lane = threadIdx.x & 63, wl = lane & (LW - 1), wk = lane / LW;
    const int64_t jw = (int64_t)blockIdx.x * G + wk;
    const bool exists = jw < A.n;
    const int64_t j = exists ? jw : A.n - 1;
    T& S = SW.w[wk];
    const int L = A.L, k = A.k, p = A.p, W = A.W, nf = A.nf;
    const int t0 = A.t0, t1 = A.t1;

    for (int i = lane; i < (int)sizeof(SW) / 4; i += 64) ((int*)&SW)[i] = 0;
    int halted = A.halted[j];
    bool live = exists && !halted;
    if (!__ballot(live)) {                        // nothing but the trajectory's -1
        if (exists && A.traj)
            for (int t = t0 + 1 + wl; t <= t1; t += LW) A.traj[j * A.steps_total + (t - 1)] = -1;
        return;
    }
    int vbest = wl < W ? (int)A.bestSeq[j * W + wl] : 0;
    lds_order();
    if (wl < W) S.pk[wl] = A.seq[j * W + wl];
    lds_order();

    // ---- geometry
    const int nc = k >> 1;
    const int n0 = first_index(k, p);
    const int kz = 8 + ((3 - n0) & 3);
    const int db = T::DNEG + ((n0 + kz) & 7);
    const int lj = lane & 15, lg = lane >> 4;
    const int cl = lj >> 3;                       // class of the lane's slots
    const int isub = 4 * (lg & (R / 4 - 1));
    const int n1 = n0 + R * (lj & 7) + isub;      // the first of its four

    // ---- the class rows
    for (int i = wl; i < 2 * R * ST / 4; i += LW) {
        const int row = i / (ST / 4), kap = 4 * (i - row * (ST / 4));
        const int rc = row / R, n = (row & (R - 1)) + kap - kz;
        uint32_t v = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int x = 2 * (n + b) + 1 + rc;
            if (n + b >= 0 && x <= L && kap < ROW) v |= (packed_bit(S.pk, x) ? 0x01u : 0xFFu) << (8 * b);
        }
        ((uint32_t*)S.X)[i] = v;
    }
    // ---- -C_{2m} of this lane's m = 4 wl + 1 .. + 4
    v2s c01, c23;
    {
        int c[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int m = 4 * wl + 1 + b;
            c[b] = m <= k ? -packed_corr(S.pk, L, 2 * m) : 0;
        }
        c01 = v2s{(short)c[0], (short)c[1]};
        c23 = v2s{(short)c[2], (short)c[3]};
    }
    lds_order();
    auto shifted = [&](uint32_t f) -> uint32_t {  // the walker's lane before, 0 at its first
        if constexpr (G == 4) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, 0x111, 0xf, 0xf, true);
        const uint32_t v = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, 0x138, 0xf, 0xf, true);
        return wl == 0 ? 0u : v;
    };
    auto store_c = [&](bool wide) {
        const uint32_t u01 = __builtin_bit_cast(uint32_t, c01), u23 = __builtin_bit_cast(uint32_t, c23);
        const uint32_t f = __builtin_amdgcn_perm(u23, u01, 0x06040200u);
        *(uint32_t*)(S.D + db + 4 * wl + 1) = f;
        *(uint32_t*)(S.D + db - 4 * wl - 3) = __builtin_amdgcn_perm(shifted(f), f, 0x07000102u);
        if (wide) {
            const v2s bias = {128, 128};
            const uint32_t h = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, (v2s)(c23 + bias)),
                                                     __builtin_bit_cast(uint32_t, (v2s)(c01 + bias)), 0x07050301u);
            *(uint32_t*)(S.DH + db + 4 * wl + 1) = h;
            *(uint32_t*)(S.DH + db - 4 * wl - 3) = __builtin_amdgcn_perm(shifted(h), h, 0x07000102u);
        }
    };
    auto need_wide = [&]() -> bool {
        const v2s bias = {96, 96};                // -96 <= C <= 95  <=>  0 <= C + 96 < 192
        const uint32_t t01 = __builtin_bit_cast(uint32_t, (v2s)(c01 + bias));
        const uint32_t t23 = __builtin_bit_cast(uint32_t, (v2s)(c23 + bias));
        uint32_t any = (t01 | t23) & 0xFF00FF00u;
        any |= ((t01 & (t01 << 1)) | (t23 & (t23 << 1))) & 0x00800080u;
        return __ballot(any != 0) != 0;
    };
    bool wide = need_wide();
    store_c(wide);

    // ---- slots
    const int sig = ((k - cl) & 1) ? -1 : 1;
    const int w40 = (-4 * sig) & 0xFF, w41 = w40 << 8, w42 = w40 << 16, w43 = w40 << 24;
    int az[4], Y[4], sgs[4], xso, xeo;
    {
        const int is = (n0 + kz) & 3, ks = n1 + kz - is;
        xso = ks < ROW ? (cl * R + is) * ST + ks : ROW;
        const int e = 3 * n1 - k + cl + kz, ie = e & 3;
        xeo = (e - ie >= -16 && e - ie <= ROW + 4) ? (cl * R + ie) * ST + e - ie : ROW;
        v4i tb;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = n1 + r, x = 2 * n + 1 + cl;
            const bool valid = n >= 0 && x > p && x <= k + 1;
            tb[r] = valid ? A.tabu[j * nf + x - p - 1] : INT_MAX;
            int y = 0;                            // sum_m x[n + m] x[n - m]
            if (valid) {
                const int uf = n + 1 + kz, rf = cl * R + (uf & 3);
                const int ub = n - 4 + kz, rb = cl * R + (ub & 3);
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
            Y[r] = centre ? 4 * nc + 4 : 4 * (k - cl - 1) + 8 * y;
            sgs[r] = centre ? 0 : 1;
            az[r] = 2 * n + cl;
        }
        *(v4i*)(S.T + 8 * R * cl + R * (lj & 7) + isub) = tb;
    }
    const int toff = 8 * R * cl + R * (lj & 7) + isub;
    const bool rise = k & 1;
    const int cw0 = db + (rise ? 2 * n1 + cl - k : k - cl - 2 * n1 - 6);
    const int co01 = (cw0 & ~3) + (rise ? 0 : 4), co23 = (cw0 & ~3) + (rise ? 4 : 0);
    const int cwA = ((-2 * sig) & 0xFF) << (8 * ((cw0 & 1) + (rise ? 0 : 2)));
    const int cwB = ((-2 * sig) & 0xFF) << (8 * ((cw0 & 1) + (rise ? 2 : 0)));
    // operands: a lane's row of A is copy lj % R of walker lj / R; its column of B lj & 7
    const int8_t* pa[G];
#pragma unroll
    for (int w = 0; w < G; ++w)
        pa[w] = lj / R == w ? SW.w[w].X + (lj & (R - 1)) * ST + 16 * lg : SW.zero;
    const int boff = db + 16 * lg - kz - n0 - R * (lj & 7);
    // the lane's byte of the flipped elements' copies, less the index
    const int xwl = (wl & (R - 1)) * ST + kz - (wl & (R - 1));
    const bool writes = wl < 2 * R, second = (wl / R) & 1;

    auto packed_words = [&]() -> int {            // word wl of the packed sequence
        uint32_t bits[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint32_t v = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i0 = kz & 3;
                const int kap = 16 * (wl < W ? wl : 0) + 4 * q + kz - i0;
                const uint32_t d = *(const uint32_t*)(S.X + (c * R + i0) * ST + (kap < ROW ? kap : ROW));
                const uint32_t one = d & ~(d >> 7) & 0x01010101u;
                v |= ((one * 0x08040201u) >> 24) << (4 * (3 - q));
            }
            bits[c] = v;
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

    int E = A.E[j], bestE = A.bestE[j], bestT = A.bestT[j];
    const int tenure = A.tenure[j];
    const int thr = A.e_max >= 0 ? A.e_max : INT_MIN;
    const int64_t wid = A.walker_begin + j;
    int pend = pending_level(A);
    int rare = max(max(pend, thr), bestE - 1);
    int32_t* const traj = A.traj ? A.traj + j * A.steps_total : nullptr;

    // The sum over the walkers of A_w B_w, both classes.
    auto products = [&](v4i (&h)[2], bool high) {
        h[0] = h[1] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < G; ++w) {
            const int8_t* const pb = (high ? SW.w[w].DH : SW.w[w].D) + boff;
#pragma unroll
            for (int m = 0; m < KB; ++m) {
                const v4i b = {*(const int*)(pb + 64 * m), *(const int*)(pb + 64 * m + 4), *(const int*)(pb + 64 * m + 8),
                               *(const int*)(pb + 64 * m + 12)};
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    h[c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(*(const v4i*)(pa[w] + c * R * ST + 64 * m), b, h[c], 0,
                                                                 0, 0);
            }
        }
    };
    for (int t = t0 + 1; t <= t1; ++t) {
        v4i H2[2], H;
        products(H2, false);
#pragma unroll
        for (int r = 0; r < 4; ++r) H[r] = cl ? H2[1][r] : H2[0][r];
        const int xs = *(const int*)(S.X + xso);
        const int* pe = (const int*)(S.X + xeo);
        const int e0 = pe[0], e1 = pe[1], e2 = pe[2];
        const int cd0 = *(const int*)(S.D + co01), cd1 = *(const int*)(S.D + co23);
        const v4i tb = *(const v4i*)(S.T + toff);
        if (wide) {
            v4i Hh2[2];
            products(Hh2, true);
            const int ch0 = *(const int*)(S.DH + co01), ch1 = *(const int*)(S.DH + co23);
            int gw[4];
            gw[0] = __builtin_amdgcn_sdot4(ch0, cwA, 0, false);
            gw[1] = __builtin_amdgcn_sdot4(ch0, cwB, 0, false);
            gw[2] = __builtin_amdgcn_sdot4(ch1, cwA, 0, false);
            gw[3] = __builtin_amdgcn_sdot4(ch1, cwB, 0, false);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int s = (int)((uint32_t)xs << (24 - 8 * r)) >> 24;
                H[r] += 256 * (cl ? Hh2[1][r] : Hh2[0][r]) + s * 128 * gw[r];
            }
        }
        int v[4];
        v[0] = __builtin_amdgcn_sdot4(e0, w40, H[0], false);
        v[1] = __builtin_amdgcn_sdot4(e0, w43, H[1], false);
        v[2] = __builtin_amdgcn_sdot4(e1, w42, H[2], false);
        v[3] = __builtin_amdgcn_sdot4(e2, w41, H[3], false);
        int kmin = INT_MAX;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int s = (int)((uint32_t)xs << (24 - 8 * r)) >> 24;
            int d = (labs_mul_i24(s, v[r]) << sgs[r]) + Y[r];
            d = __builtin_amdgcn_sdot4(r < 2 ? cd0 : cd1, r & 1 ? cwB : cwA, d, false);
            kmin = min(kmin, tb[r] < t ? (d << 8) + az[r] : INT_MAX);
        }
        kmin = group_min<G>(kmin);
        if (live && kmin == INT_MAX) {
            halted = t;
            live = false;
        }
        if (!__ballot(live)) break;
        // ---- the flipped pair: class cs, indices n and nbs.  Lanes without a live walker (the
        // last wave's that no walker is left for; a tenure below the free positions never
        // halts one) go along on the zero behind class 0's last element, index k + 1, which
        // changes neither C nor Y; with an element in its place their C grew until the whole
        // wave multiplied the high bytes too (8,193 walkers at L = 201 2.44 us a step, now
        // 2.13; 4,097 at L = 101 1.28, now 1.01).
        const int z = live ? kmin & 511 : 2 * (k + 1), n = z >> 1, cs = z & 1;
        const int q = n - n0, nbs = k - n - cs;
        const bool cen = n == nbs;
        const int row0 = cs * R * ST;
        const int sa = S.X[row0 + n + kz];
        const int sb = ((k - cs) & 1) ? -sa : sa;
        if (live) E += 8 * (kmin >> 9);
        int8_t* const xw = S.X + (row0 + xwl + (second ? nbs : n));
        lds_order();
        if (writes && live) *xw = 0;
        if (wl == 0 && live) S.T[8 * R * cs + q] = t + tenure;
        lds_order();
        int yd[2][2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int s0 = 2 * n0 - (e ? nbs : n) + kz, off = 2 * (n1 - n0) + (s0 & ~(R - 1));
            const bool in = off >= -4 && off < ROW && cl == cs;
            const int* y = (const int*)(S.X + (in ? row0 + (s0 & (R - 1)) * ST + off : ROW));
            yd[e][0] = y[0];
            yd[e][1] = y[1];
        }
        {
            const int uf = n + kz + 1, ub = n + kz - 4;
            const short mul = (short)(cen ? 2 * sa : 4 * sa);
            const v2s mul2 = {mul, mul};
            const uint32_t f = *(const uint32_t*)(S.X + row0 + (uf & 3) * ST + min((uf & ~3) + 4 * wl, ROW));
            const uint32_t b = *(const uint32_t*)(S.X + row0 + (ub & 3) * ST + max((ub & ~3) - 4 * wl, 0));
            const v2s u01 = __builtin_bit_cast(v2s, __builtin_amdgcn_perm(f, f, 0x010C000Cu)) +
                            __builtin_bit_cast(v2s, __builtin_amdgcn_perm(b, b, 0x020C030Cu));
            const v2s u23 = __builtin_bit_cast(v2s, __builtin_amdgcn_perm(f, f, 0x030C020Cu)) +
                            __builtin_bit_cast(v2s, __builtin_amdgcn_perm(b, b, 0x000C010Cu));
            c01 += (u01 >> 8) * mul2;
            c23 += (u23 >> 8) * mul2;
        }
        lds_order();
        if (writes && live) *xw = (int8_t)(second ? -sb : -sa);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int wgt = (e ? (cen ? 0 : -16 * sb) : -16 * sa) & 0xFF;
            Y[0] = __builtin_amdgcn_sdot4(yd[e][0], wgt, Y[0], false);
            Y[1] = __builtin_amdgcn_sdot4(yd[e][0], wgt << 16, Y[1], false);
            Y[2] = __builtin_amdgcn_sdot4(yd[e][1], wgt, Y[2], false);
            Y[3] = __builtin_amdgcn_sdot4(yd[e][1], wgt << 16, Y[3], false);
        }
        if ((t & 3) == 0) wide = need_wide();
        store_c(wide);
        lds_order();
        if (traj && live && wl == 0) traj[t - 1] = E;
        const bool look = live && E <= rare;
        if (!__ballot(look)) continue;
        const int word = packed_words(), before = __shfl(word, lane - 1, 64);
        if (!look) continue;
        if (E < bestE) {
            bestE = E;
            bestT = t;
            vbest = word;
        }
        if (E <= pend) {
            const unsigned long long now = __builtin_amdgcn_s_memrealtime();
            pend = -1;
            for (int l = 0; l < A.n_levels; ++l) {
                const int lv = A.level_E[l];
                if (E > lv) pend = max(pend, lv);
                else if (wl == 0) atomicMin(&A.hit_ticks[l], now);
            }
        }
        if (E <= thr) {
            uint32_t slot = 0;
            if (wl == 0) slot = atomicAdd(A.st_count, 1u);
            slot = (uint32_t)__shfl((int)slot, lane & ~(LW - 1), 64);
            if (slot < A.st_cap && wl < W + 3) {
                uint32_t u;
                if (wl == 0) u = (uint32_t)E;
                else if (wl <= W) u = (uint32_t)before;
                else if (wl == W + 1) u = (uint32_t)wid;
                else u = (uint32_t)t;
                A.rec[(int64_t)wl * A.rec_stride + slot] = u;
            }
        }
        rare = max(max(pend, thr), bestE - 1);
    }
    if (!exists) return;
    if (halted && traj)
        for (int t = max(halted, t0 + 1) + wl; t <= t1; t += LW) traj[t - 1] = -1;
    const int word = packed_words();
    if (wl < W) {
        A.seq[j * W + wl] = (uint32_t)word;
        A.bestSeq[j * W + wl] = (uint32_t)vbest;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int n = n1 + r, x = 2 * n + 1 + cl;
        if (n >= 0 && x > p && x <= k + 1) A.tabu[j * nf + x - p - 1] = S.T[toff + r];
    }
    if (wl == 0) {
        A.E[j] = E;
        A.bestE[j] = bestE;
        A.bestT[j] = bestT;
        A.halted[j] = halted;
    }
}

}  // namespace walkimpl

// Walkers a wave for this length, 1: the walk of walk.hip.  Four (two) walkers need their
// lags and indices to fit 16 (32) lanes of four.  A step of a wave takes 1.8 times as long
// for four or two walkers as for one, and alone 0.9 to 1.4 us in place of 0.7, so it pays
// only where the waves are many (us a step, one walker a wave / this):
//   L = 101 (4):  2,048 0.83/0.99,  4,096 1.17/0.99,  16,384 3.45/1.64,  65,536 12.6/5.6
//   L = 127 (4):  4,096 1.19/1.50,  8,192 2.02/1.67,  16,384 3.54/2.17,  65,536 13.0/7.8
//   L = 201 (2):  4,096 1.19/1.18,  8,192 1.99/1.67,  16,384 3.56/3.11,  65,536 13.1/11.2
int walk_group(int L, int p, int64_t n) {
    const int k = (L - 1) / 2, range = (k >> 1) - walkimpl::first_index(k, p) + 1;
    if (k <= 63 && range <= 32 && n >= (k + 12 <= 64 ? 4096 : 8192)) return 4;
    if (k + 12 <= 128 && range <= 64 && n >= 8192) return 2;
    return 1;
}

labs_status launch_walk_group(const WalkArgs& A, int G, hipStream_t st) {
    const bool one = A.k + 12 <= 64;               // a class row in 64 bytes
    const dim3 grid((unsigned)((A.n + G - 1) / G)), block(64);
    if (G == 4 && one) hipLaunchKernelGGL((walkimpl::k_walk_group<1, 4>), grid, block, 0, st, A);
    else if (G == 4) hipLaunchKernelGGL((walkimpl::k_walk_group<2, 4>), grid, block, 0, st, A);
    else if (one) hipLaunchKernelGGL((walkimpl::k_walk_group<1, 2>), grid, block, 0, st, A);
    else hipLaunchKernelGGL((walkimpl::k_walk_group<2, 2>), grid, block, 0, st, A);
    LABS_LAUNCHED("k_walk_group");
    return LABS_OK;
}

}  // namespace labsdev
