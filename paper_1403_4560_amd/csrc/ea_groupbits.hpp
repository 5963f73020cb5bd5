// ea_groupbits.hpp -- the group engine's form for +-1 couplings: walkers as
// bits.  Any even L <= 16.
//
// Layout: one 32-bit word holds one site of up to 32 walkers of a chain (a
// "set": bit j of set s is walker s WS + j, set iff the spin is -1),
// [2 parities][sets][N/2 sites].  A site's bonds are six bits shared by every
// walker, so a bond is unsatisfied in the walkers where (s ^ neighbour ^ bond)
// is 1, and the count c of unsatisfied bonds, dE <= 0 (c >= k_s) and the
// class e of the acceptance table (c, or 7 - c for s = +1: see ea_bits.hip)
// are formed for the whole set at once, bit-sliced.  The neighbour arithmetic
// works for any L.  Each (site, walker) still draws its own Philox word:
// counter (h >> 2, 2n + p, (t << 1) | r, sample), word h & 3, as in every
// engine; a work item is (set, four consecutive sublattice sites), one Philox
// call per walker.
//
// Bound: VALU issue, Philox above all.  Its first two rounds mix only the
// site group with the walker's slot by xor, so the products of either side
// are made once: per item for the sites, once per sweep for the walkers (the
// table PW); what is left is eight rounds and two xors, 34 operations instead
// of 40 for four attempts.  In issue cycles of a wave (multiply-add 4.8; xors,
// shifts right, ands and binary32 adds and products from vector registers
// 2.5; others, and anything with a scalar operand, 4.4) an octet of walkers
// takes 1510 for 32 attempts, the field of a set 430 and the tallies 360.
// Against int8 words of four walkers per site (one bond-spin product and count
// per quad), sweep kernel attempts/ns: L = 10 x 56 temperatures 909 -> 1599
// (256 samples), L = 12 x 16 852 -> 1468 (512), L = 14 x 32 723 -> 1463 (256),
// L = 6 x 56 649 -> 1021 (1024); few chains are bound by the latency of a
// sweep: L = 6 x 56, 64 samples 6.7 -> 5.4 us.
//
// Sites are stored by position within their group of four ((h & 3) N/8 + h /
// 4), so that the lanes of a wave, which take consecutive groups, read
// consecutive words.
#pragma once

#include "ea_bitops.hpp"
#include "ea_device.hpp"
#include "ea_group.hpp"
#include "ea_item.hpp"
#include "ea_types.hpp"

namespace ea {

// Numbers of 0 .. 2^n - 1 per bit position (walker), one word per digit.
template <int NA, int NB>
__device__ __forceinline__ void add_planes(uint32_t (&a)[NA], const uint32_t (&b)[NB])
{
    static_assert(NA >= NB, "room for the sum");
    uint32_t c = a[0] & b[0];
    a[0] ^= b[0];
#pragma unroll
    for (int i = 1; i < NA; ++i) {
        if (i < NB) {
            const uint32_t t = maj3(a[i], b[i], c);
            a[i] = xor3(a[i], b[i], c);
            c = t;
        } else {
            const uint32_t t = a[i] & c;
            a[i] ^= c;
            c = t;
        }
    }
}

// The number of set words among four.
__device__ __forceinline__ void count4(const uint32_t (&x)[4], uint32_t (&n)[3])
{
    const uint32_t s = xor3(x[0], x[1], x[2]), c = maj3(x[0], x[1], x[2]), k = s & x[3];
    n[0] = s ^ x[3];
    n[1] = c ^ k;
    n[2] = c & k;
}

// Sums over the 16 lanes of a row: every lane gives 16-bit columns (bit i of
// either half), lane i receives the columns i as bits (a 16 x 16 transposition
// of both halves by four exchanges).
struct RowTranspose {
    uint32_t amt[4], mask[4];  // per step 8, 4, 2, 1

    __device__ __forceinline__ void init(int lane)
    {
        constexpr uint32_t lo[4] = {0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int m = 8 >> k;
            const bool up = lane & m;
            amt[k] = up ? m : 32 - m;
            mask[k] = up ? lo[k] : ~lo[k];
        }
    }
    template <int K>
    __device__ __forceinline__ uint32_t step(uint32_t x, uint32_t t) const
    {
        const uint32_t r = __builtin_amdgcn_alignbit(t, t, amt[K]);
        return __builtin_amdgcn_bitop3_b32(mask[K], r, x, 0xCA);  // mask ? r : x
    }
    __device__ __forceinline__ uint32_t operator()(uint32_t x) const
    {
        x = step<0>(x, (uint32_t)row_rotate<8>((int)x));
        // lanes i and i ^ 4: rotation by 4 in the upper quads of each eight, by 12 in the lower
        int t = __builtin_amdgcn_update_dpp(0, (int)x, 0x120 + 4, 0xF, 0xA, false);
        t = __builtin_amdgcn_update_dpp(t, (int)x, 0x120 + 12, 0xF, 0x5, false);
        x = step<1>(x, (uint32_t)t);
        x = step<2>(x, (uint32_t)quad_xor<2>((int)x));
        return step<3>(x, (uint32_t)quad_xor<1>((int)x));
    }
};

// Row totals of a digit-plane number, the rows' lanes holding sets of WS
// walkers: lo for walker i = lane mod 16 (WS <= 8: mod 8, in two lanes whose
// values add), hi for walker 16 + i (WS > 16).  Planes are packed to fill the
// transposition: one per word for WS > 16, two for WS > 8, four for WS <= 8.
// HALVES (WS <= 8): the row's first eight lanes hold one set, lo, the others
// another, hi.
template <bool HALVES, int NP>
__device__ __forceinline__ void row_totals(const RowTranspose &tr, const uint32_t (&p)[NP], int WS, int lane, int &lo,
                                           int &hi)
{
    lo = hi = 0;
    if (WS > 16) {
#pragma unroll
        for (int k = NP - 1; k >= 0; --k) {
            const uint32_t x = tr(p[k]);
            lo = 2 * lo + __builtin_popcount(x & 0xFFFFu);
            hi = 2 * hi + __builtin_popcount(x >> 16);
        }
    } else if (WS > 8) {
#pragma unroll
        for (int k = (NP - 1) / 2; k >= 0; --k) {
            const uint32_t x = tr(2 * k + 1 < NP ? p[2 * k] | p[2 * k + 1] << 16 : p[2 * k]);
            lo = 4 * lo + __builtin_popcount(x & 0xFFFFu) + 2 * __builtin_popcount(x >> 16);
        }
    } else {
        // columns 0 .. 7: planes 0 and 2 of a word, columns 8 .. 15: planes 1 and 3
#pragma unroll
        for (int k = (NP - 1) / 4; k >= 0; --k) {
            uint32_t v = p[4 * k];
            if (4 * k + 1 < NP) v |= p[4 * k + 1] << 8;
            if (4 * k + 2 < NP) v |= p[4 * k + 2] << 16;
            if (4 * k + 3 < NP) v |= p[4 * k + 3] << 24;
            const uint32_t x = tr(v);
            if constexpr (HALVES) {
                lo = 16 * lo + __builtin_popcount(x & 0xFFu) + 4 * __builtin_popcount(x & 0xFF0000u);
                hi = 16 * hi + __builtin_popcount(x & 0xFF00u) + 4 * __builtin_popcount(x >> 24);
            } else {
                lo = 16 * lo + __builtin_popcount(x & 0xFFFFu) + 4 * __builtin_popcount(x >> 16);
            }
        }
        lo <<= (lane & 15) >> 3;
        hi <<= (lane & 15) >> 3;
    }
}

// Adds the totals of flips, down spins and unsatisfied bonds of the sets that
// a wave's lanes hold to their LDS cells.  A wave of one set (TPS >= 64) first
// folds its four rows: swapping halves of the wave between the flips and the
// down spins leaves one quantity in each half, whose two parts are then added
// (half the additions of summing both everywhere), and likewise the rows
// between those and the unsatisfied bonds; the transpositions then run over 6
// planes, not 13.  EIGHT: a set may be eight lanes wide.
template <bool EIGHT, int PF, int PU>
__device__ __forceinline__ void add_totals(uint32_t (&fl)[PF], uint32_t (&nd)[PF],
                                           uint32_t (&un)[PU], int lane, int TPS, int WS, int s, int nT,
                                           const int32_t *sow, int32_t *flips, int32_t *ND, int32_t *U)
{
    static_assert(PU == PF + 1, "digits of the folded sums");
    RowTranspose tr;
    tr.init(lane);
    const int i = WS > 8 ? lane & 15 : lane & 7, w = s * WS + i;
    const bool ok = i < WS && w < nT, ok2 = 16 + i < WS && w + 16 < nT;
    if (TPS >= 64) {
        uint32_t x[PU] = {}, z[PU + 1] = {};
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const auto r = __builtin_amdgcn_permlane32_swap(fl[k], nd[k], false, false);
            x[k] = r[0];
            nd[k] = r[1];
        }
        add_planes(x, nd);  // flips in lanes 0 .. 31, down spins in the others
#pragma unroll
        for (int k = 0; k < PU; ++k) {
            const auto r = __builtin_amdgcn_permlane16_swap(x[k], un[k], false, false);
            z[k] = r[0];
            un[k] = r[1];
        }
        add_planes(z, un);  // rows: flips, unsatisfied bonds, down spins, unsatisfied bonds
        int lo, hi;
        row_totals<false>(tr, z, WS, lane, lo, hi);
        const int row = lane >> 4;
        int32_t *cell = row == 0 ? flips : row == 2 ? ND : U;
        if (ok) atomicAdd(&cell[row == 0 ? sow[w] : w], lo);
        if (ok2) atomicAdd(&cell[row == 0 ? sow[w + 16] : w + 16], hi);
        return;
    }
    int f0, f1, d0, d1, u0, u1;
    const auto add = [&](int w, int f, int d, int u) {
        atomicAdd(&flips[sow[w]], f);
        atomicAdd(&ND[w], d);
        atomicAdd(&U[w], u);
    };
    if constexpr (EIGHT) {
        if (TPS == 8) {
            row_totals<true>(tr, fl, WS, lane, f0, f1);
            row_totals<true>(tr, nd, WS, lane, d0, d1);
            row_totals<true>(tr, un, WS, lane, u0, u1);
            const int v = (s & ~1) * WS + i;  // the row's first set is even
            if (i < WS && v < nT) add(v, f0, d0, u0);
            if (i < WS && v + WS < nT) add(v + WS, f1, d1, u1);
            return;
        }
    }
    row_totals<false>(tr, fl, WS, lane, f0, f1);
    row_totals<false>(tr, nd, WS, lane, d0, d1);
    row_totals<false>(tr, un, WS, lane, u0, u1);
    if (ok) add(w, f0, d0, u0);
    if (ok2) add(w + 16, f1, d1, u1);
}

// The spreading tables: entry v of table k holds, in bytes 0 .. 7, 4 << k for
// the set bits of v.  One copy per workgroup, at an LDS address known to the
// compiler (the host counts them beside the frames: SPREAD_BYTES).
__device__ __forceinline__ uint2 *spread_tables()
{
    __shared__ uint2 tab[SPREAD_BYTES / sizeof(uint2)];
    return tab;
}

// What a chain's sweep needs of the walkers' slots: the Philox state words that
// depend on the slot alone (rounds 0 and 1), and the LDS address of the slot's
// threshold table.
struct GroupBitsItem {
    uint32_t *SW;         // [2][NS][N/2]
    const uint8_t *JB;    // [2][N/2] bonds +x, -x, +y, -y, +z, -z in bits 0 .. 5
    const uint4 *NB;      // neighbour words as byte offsets (group_nbrs order)
    uint32_t pw;          // LDS address of PW[parity][walker]
    uint32_t pws;         // bytes of one parity's table
    int NS, WS;
    uint32_t kb0[3], kb1[3];
};

// Four walkers (bytes 0 .. 3 of the class words Q of the four sites): their
// Philox words and accept bits, shifted into F from the lowest walker up (so that
// the walkers end up in reverse order).
// The scheduling barriers keep the order written: every LDS load ahead of the
// rounds that hide it, and the four calls side by side, round by round.  Left
// to itself the compiler orders by register pressure, one walker after the
// other and each threshold waited for where it is used: 2500 cycles a quad
// instead of 1800 with one wave per SIMD.
__device__ __forceinline__ void group_bits_quad(const uint4 (&w)[4], const uint32_t Q[4], const uint4 pg,
                                                const RoundKeys &key, uint32_t F[4])
{
    uint32_t thr[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) thr[j][k] = lds_load(w[j].w + ((Q[k] >> (8 * j)) & 0xFFu));
    u32x4 c[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = PhiloxSlot{w[j].x, w[j].y, w[j].z}.start(pg);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j) c[j] = philox_round(c[j], key.a[k], key.b[k]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        F[0] = shift_in_less(F[0], c[j].x, thr[j][0]);
        F[1] = shift_in_less(F[1], c[j].y, thr[j][1]);
        F[2] = shift_in_less(F[2], c[j].z, thr[j][2]);
        F[3] = shift_in_less(F[3], c[j].w, thr[j][3]);
    }
}

__device__ __forceinline__ void load_walkers(uint32_t pw, uint4 (&w)[4])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = lds_load4(pw + 16 * j);
}

// Metropolis update of item (set s, sites 4 g4 .. 4 g4 + 3) of parity P.  F:
// flipped sites; Sn: spins after the update; V (P = 1): digits of the count of
// unsatisfied bonds after the update.
template <int L, int P>
__device__ __forceinline__ void group_bits_item(const SweepArgs &A, const SampleDev &d, const GroupBitsItem &G, const RoundKeys &key,
                                                int s, int g4, uint32_t valid, uint32_t F[4], uint32_t Sn[4],
                                                uint32_t V[4][3])
{
    constexpr int HALF = L * L * L / 2, G4 = HALF / 4;
    uint32_t *Sp = G.SW + (P * G.NS + s) * HALF + g4;
    const char *So = (const char *)(G.SW + ((1 - P) * G.NS + s) * HALF);
    // (scheduling barriers: every load of a stage is issued before the stage
    // that uses them, so a wave waits three times here, not at each load)
    const uint32_t jb = *(const uint32_t *)(G.JB + P * HALF + 4 * g4);
    uint4 te[4];
    uint32_t nb[4][6], E[4][3], D[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) te[k] = G.NB[k * G4 + g4];
#pragma unroll
    for (int k = 0; k < 4; ++k) Sn[k] = Sp[k * G4];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t tx = P ? te[k].w : te[k].z;
        const uint32_t off[6] = {tx & 0xFFFFu,      tx >> 16,      te[k].x & 0xFFFFu,
                                 te[k].x >> 16,     te[k].y & 0xFFFFu, te[k].y >> 16};
#pragma unroll
        for (int b = 0; b < 6; ++b) nb[k][b] = *(const uint32_t *)(So + off[b]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t sv = Sn[k];
        uint32_t u[6];
#pragma unroll
        for (int b = 0; b < 6; ++b) u[b] = xor3(sv, nb[k][b], (uint32_t)__builtin_amdgcn_sbfe((int)jb, 8 * k + b, 1));
        const uint32_t a1 = xor3(u[0], u[1], u[2]), b1 = maj3(u[0], u[1], u[2]);
        const uint32_t a2 = xor3(u[3], u[4], u[5]), b2 = maj3(u[3], u[4], u[5]);
        const uint32_t C0 = a1 ^ a2, kk = a1 & a2;
        const uint32_t C1 = xor3(b1, b2, kk), C2 = maj3(b1, b2, kk);
        // dE <= 0 iff c >= k_s: no borrow out of c - k_s
        const uint32_t K0 = sel(G.kb0[0], G.kb1[0], sv), K1 = sel(G.kb0[1], G.kb1[1], sv),
                       K2 = sel(G.kb0[2], G.kb1[2], sv);
        const uint32_t w0 = ~C0 & K0;
        const uint32_t w1 = maj3(~C1, K1, w0);
        D[k] = ~maj3(~C2, K2, w1);
        E[k][0] = ~(C0 ^ sv);
        E[k][1] = ~(C1 ^ sv);
        E[k][2] = ~(C2 ^ sv);
        F[k] = 0;
    }
    // the site group's part of Philox rounds 0 and 1
    const uint4 pg = philox_group((uint32_t)g4, d.sample_id, A.key1);
    uint32_t pw = G.pw + P * G.pws + 16 * (s * G.WS);
    const uint32_t sp = lds_addr(spread_tables());
#pragma unroll 1
    for (int at = 0; at < G.WS; at += 8, pw += 128) {
        uint4 w[4];
        uint32_t Ql[4], Qh[4];
        load_walkers(pw, w);
        uint2 t[4][3];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int b = 0; b < 3; ++b) t[k][b] = lds_load2(sp + 2048 * b + 8 * __builtin_amdgcn_ubfe(E[k][b], at, 8));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            Ql[k] = xor3(t[k][0].x, t[k][1].x, t[k][2].x);
            Qh[k] = xor3(t[k][0].y, t[k][1].y, t[k][2].y);
        }
        group_bits_quad(w, Ql, pg, key, F);
        if (at + 4 < G.WS) {
            load_walkers(pw + 64, w);
            group_bits_quad(w, Qh, pg, key, F);
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t f = ((__builtin_bitreverse32(F[k]) >> (32 - G.WS)) | D[k]) & valid;
        if constexpr (P == 1) {
            // c of the site after the update: c, or 6 - c where it flipped (no walker: 0)
            const uint32_t C0 = ~(E[k][0] ^ Sn[k]), C1 = ~(E[k][1] ^ Sn[k]), C2 = ~(E[k][2] ^ Sn[k]);
            const uint32_t t = C1 & C0;
            V[k][0] = C0 & valid;
            V[k][1] = ((f & ~(C1 ^ C0)) | (~f & C1)) & valid;
            V[k][2] = ((f & ~(C2 | t)) | (~f & C2)) & valid;
        }
        F[k] = f;
        Sn[k] ^= f;
        Sp[k * G4] = Sn[k];
    }
}

// A thread's share of a sweep (up to REP site groups of its set per
// half-sweep) and the walkers' totals of it.
template <int L, int REP>
__device__ __forceinline__ void group_bits_sweep(const SweepArgs &A, const SampleDev &d, const GroupBitsItem &G,
                                                 const RoundKeys &key, int s, int TPS, const Team &tm,
                                                 const ItemLds &I, int32_t *U, int32_t *ND)
{
    constexpr int G4 = L * L * L / 8;
    // sums of 8 REP flips and down spins and of 24 REP unsatisfied bonds
    constexpr int PF = REP == 1 ? 4 : 7, PU = REP == 1 ? 5 : 8;
    static_assert(REP == 1 || REP == 8, "digits of the sums");
    uint32_t fl[PF] = {}, nd[PF] = {}, un[PU] = {};
    const bool on = s < G.NS;
    uint32_t F[4], Sn[4], V[4][3], n[3];
    // the thread's first site group and the walkers of its set, formed here in
    // either half-sweep (held across the sweep, they spill)
    int gs;
    uint32_t valid;
    const auto share = [&] {
        asm volatile("" : "+v"(s));
        gs = tm.tid() - s * TPS;
        const int bits = on ? min(G.WS, d.n_T - s * G.WS) : 0;
        valid = bits >= 32 ? ~0u : (1u << bits) - 1u;
    };
    share();
    if (on) {
#pragma unroll 1
        for (int g4 = gs; g4 < G4; g4 += TPS) {
            group_bits_item<L, 0>(A, d, G, key, s, g4, valid, F, Sn, V);
            if constexpr (REP == 1) {
                count4(F, n);
                fl[0] = n[0], fl[1] = n[1], fl[2] = n[2];
                count4(Sn, n);
                nd[0] = n[0], nd[1] = n[1], nd[2] = n[2];
                break;
            } else {
                count4(F, n);
                add_planes(fl, n);
                count4(Sn, n);
                add_planes(nd, n);
            }
        }
    }
    __syncthreads();
    share();
    if (on) {
#pragma unroll 1
        for (int g4 = gs; g4 < G4; g4 += TPS) {
            group_bits_item<L, 1>(A, d, G, key, s, g4, valid, F, Sn, V);
            count4(F, n);
            add_planes(fl, n);
            count4(Sn, n);
            add_planes(nd, n);
            uint32_t a[4] = {V[0][0], V[0][1], V[0][2], 0}, b[4] = {V[2][0], V[2][1], V[2][2], 0};
            add_planes(a, V[1]);
            add_planes(b, V[3]);
            if constexpr (REP == 1) {
                for (int k = 0; k < 4; ++k) un[k] = a[k];
                add_planes(un, b);
                break;
            } else {
                add_planes(un, a);
                add_planes(un, b);
            }
        }
    }
    // (TPS is 16, 32 or whole waves, so a row holds one set, or 8 and it holds two;
    // idle lanes hold zeros)
    add_totals<G4 <= 8>(fl, nd, un, tm.tid() & 63, TPS, G.WS, s, d.n_T, I.sow, I.fl, ND, U);
}

template <int L>
__device__ __forceinline__ void run_group_bits_item(const SweepArgs &A, const SampleDev &d, int r, char *smem,
                                                    const Team tm)
{
    constexpr int N = L * L * L, HALF = N / 2, G4 = HALF / 4, HL = L / 2;
    const int nT = d.n_T;
    const int T = tm.T, tid = tm.tid();
    const GroupBitsLdsOff o = group_bits_lds_offsets(L, nT);
    const GroupSets gsz = group_sets(L, nT, T);
    const int NS = gsz.NS, WS = gsz.WS;
    uint32_t *SW = (uint32_t *)(smem + o.spins);
    uint8_t *JB = (uint8_t *)(smem + o.J);
    uint4 *NB = (uint4 *)(smem + o.nb);
    uint4 *PW = (uint4 *)(smem + o.pw);
    uint32_t *TH = (uint32_t *)(smem + o.th);
    int32_t *U = (int32_t *)(smem + o.U), *ND = (int32_t *)(smem + o.ND);
    ItemLds I{};
    I.was = (int32_t *)(smem + o.was);
    I.sow = (int32_t *)(smem + o.sow);
    I.fl = (int32_t *)(smem + o.fl);
    I.sw = (int32_t *)(smem + o.sw);
    I.b64 = (double *)(smem + o.b64);

    const size_t sbase = (size_t)d.spin_off + (size_t)r * nT * N;
    const int gi = 2 * d.slot_off + r * nT;
    // spins: int8 [walker][parity][N/2] -> bits, four sites of a set per step
    for (int i = tid; i < 2 * NS * G4; i += T) {
        const int g = i % G4, ps = i / G4, p = ps / NS, s = ps - p * NS;
        const int8_t *src = A.spins + sbase + (size_t)s * WS * N + p * HALF + 4 * g;
        const int n = min(WS, nT - s * WS);
        uint32_t w[4] = {};
        for (int j = 0; j < n; j += 4) {
            uint32_t v[4];  // (four loads in flight; past the last walker, walker j again)
            for (int b = 0; b < 4; ++b) v[b] = *(const uint32_t *)(src + (size_t)(j + b < n ? j + b : j) * N);
            for (int b = 0; b < 4; ++b)
                for (int k = 0; k < 4; ++k) w[k] |= (j + b < n ? (v[b] >> (8 * k + 7)) & 1u : 0u) << (j + b);
        }
        for (int k = 0; k < 4; ++k) SW[ps * HALF + k * G4 + g] = w[k];
    }
    const int8_t *Jg = (const int8_t *)A.J + d.J_off;
    for (int h = tid; h < HALF; h += T) {
        int nb[2][6];
        group_nbrs<L>(0, h, nb[0]);
        group_nbrs<L>(1, h, nb[1]);
        const auto at = [](int n) { return (uint32_t)(4 * ((n & 3) * G4 + (n >> 2))); };
        NB[(h & 3) * G4 + (h >> 2)] =
            make_uint4(at(nb[0][2]) | at(nb[0][3]) << 16, at(nb[0][4]) | at(nb[0][5]) << 16,
                       at(nb[0][0]) | at(nb[0][1]) << 16, at(nb[1][0]) | at(nb[1][1]) << 16);
        for (int p = 0; p < 2; ++p) {
            uint32_t b = 0;
            for (int dd = 0; dd < 3; ++dd) {
                b |= (uint32_t)(Jg[(p * 3 + dd) * HALF + h] < 0) << (2 * dd);
                b |= (uint32_t)(Jg[((1 - p) * 3 + dd) * HALF + nb[p][2 * dd + 1]] < 0) << (2 * dd + 1);
            }
            JB[p * HALF + h] = (uint8_t)b;
        }
    }
    // k_s and the slots' tables by class e, the spreading table: as in ea_bits.hip
    int k0 = 7, k1 = 7;
    for (int c = 6; c >= 0; --c) {
        if ((d.down_mask >> (7 + 6 - c)) & 1u) k0 = c;
        if ((d.down_mask >> c) & 1u) k1 = c;
    }
    for (int i = tid; i < nT * 8; i += T) {
        const int t = i >> 3, e = i & 7;
        const size_t row = ((size_t)d.slot_off + t) * 14;
        TH[i] = e < k1 ? A.lut[row + e] : (e >= 1 && 7 - e < k0) ? A.lut[row + 7 + e - 1] : 0u;
    }
    uint2 *SP = spread_tables();  // (every team writes the same)
    for (int v = tid; v < 256; v += T) {
        uint32_t lo = 0, hi = 0;
        for (int k = 0; k < 4; ++k) {
            lo |= ((v >> k) & 1u) * 4u << (8 * k);
            hi |= ((v >> (k + 4)) & 1u) * 4u << (8 * k);
        }
        for (int k = 0; k < 3; ++k) SP[256 * k + v] = make_uint2(lo << k, hi << k);
    }
    for (int i = tid; i < nT; i += T) {
        I.was[i] = A.was[gi + i];
        I.sow[A.was[gi + i]] = i;  // kept by the exchange from here on
        I.fl[i] = 0;
        I.sw[i] = 0;
        U[i] = 0;
        ND[i] = 0;
        I.b64[i] = A.beta[d.slot_off + i];
    }
    GroupBitsItem G;
    G.SW = SW;
    G.JB = JB;
    G.NB = NB;
    G.pw = lds_addr(PW);
    G.pws = 16 * MAX_T;
    G.NS = NS;
    G.WS = WS;
    for (int i = 0; i < 3; ++i) {
        G.kb0[i] = ((k0 >> i) & 1) ? ~0u : 0u;
        G.kb1[i] = ((k1 >> i) & 1) ? ~0u : 0u;
    }
    const int64_t n0 = A.state[0];
    __syncthreads();
    // the row of PW of the walker at slot tid for sweep n, by the first wave
    // (from n_T on: the padding of the last set, whose bits are never used;
    // whole sets never reach past 64 walkers)
    const auto slot_words = [&](int64_t n, int w) {
        const int t = tm.tid();
        const uint32_t th = lds_addr(TH + 8 * min(t, nT - 1));
        const uint32_t c2 = (PURPOSE_METROPOLIS << 28) | ((uint32_t)t << 1) | (uint32_t)r;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            PhiloxSlot ps;
            ps.init((uint32_t)(2 * n + p), c2, A.key0, A.key1);
            PW[p * MAX_T + w] = make_uint4(ps.x, ps.y, ps.z, th);
        }
    };
    if (tm.wave == 0) slot_words(n0, tid < nT ? I.was[tid] : tid);
    __syncthreads();

    const int TPS = gsz.TPS;
    const int s = tid / TPS;
    RoundKeys key;
    key.init(A.key0, A.key1);
    const double hd = (double)d.h32;
    int64_t next_meas = next_measurement(n0, A.measure_every, A.measure_start);
    int64_t f = 0;  // frame of the next measurement within this chunk
    // every bond has one odd end: E_J = (unsatisfied) - (satisfied) = 2 U - 3 N
    const auto energy = [&](int w) { return (double)(2 * U[w] - 3 * N) - hd * (double)(N - 2 * ND[w]); };
    for (int it = 0; it < A.K; ++it) {
        const int64_t n = n0 + it;
        if (TPS >= G4) group_bits_sweep<L, 1>(A, d, G, key, s, TPS, tm, I, U, ND);
        else group_bits_sweep<L, 8>(A, d, G, key, s, TPS, tm, I, U, ND);
        __syncthreads();
        if (tm.wave == 0) {
            const int w = exchange_slots(A, d, r, n, I, tm.tid(), key, energy);
            slot_words(n + 1, w);
        }
        const int64_t done = n + 1;
        const bool meas = done == next_meas, last = it + 1 == A.K;
        if (!meas && !last) {
            // (U and ND: read by the exchange above, cleared by the same wave)
            const int ti = tm.tid();
            if (ti < 64 && ti < nT) U[ti] = ND[ti] = 0;
            __syncthreads();
            continue;
        }
        __syncthreads();
        if (meas) {
            // snapshot in slot order: one (set, row) per step
            next_meas += A.measure_every;
            uint32_t *dst = A.frames + f * A.frame_words + d.frame_off + (size_t)r * nT * L * L;
            const int ti = tm.tid();
            for (int i = ti; !tm.ghost && i < NS * L * L; i += T) {
                const int ss = i / (L * L), row = i - ss * (L * L);
                const int e = ((row % L) + row / L) & 1;  // parity of the even x
                uint32_t w[L];
#pragma unroll
                for (int x = 0; x < L; ++x) {
                    const int h = row * HL + x / 2, p = (x & 1) ? 1 - e : e;
                    w[x] = SW[(p * NS + ss) * HALF + (h & 3) * G4 + (h >> 2)];
                }
                for (int j = 0; j < WS && ss * WS + j < nT; ++j) {
                    uint32_t b = 0;
#pragma unroll
                    for (int x = 0; x < L; ++x) {
                        b = __builtin_amdgcn_alignbit(w[x], b, 1);
                        w[x] >>= 1;
                    }
                    dst[I.sow[ss * WS + j] * L * L + row] = b >> (32 - L);
                }
            }
            for (int t = ti; !tm.ghost && t < nT; t += T) A.frameE[f * 2 * A.total_slots + gi + t] = energy(I.was[t]);
            ++f;
            __syncthreads();  // the next sweep changes the spins read here
        }
        if (!last) {
            const int ti = tm.tid();
            for (int w = ti; w < nT; w += T) U[w] = ND[w] = 0;
            // (tallied again only after the next half-sweep's barrier)
        }
    }
    const int te = tm.tid();
    for (int i = te; !tm.ghost && i < 2 * NS * G4; i += T) {
        const int g = i % G4, ps = i / G4, p = ps / NS, ss = ps - p * NS;
        uint32_t w[4];
        for (int k = 0; k < 4; ++k) w[k] = SW[ps * HALF + k * G4 + g];
        for (int j = 0; j < WS && ss * WS + j < nT; ++j) {
            uint32_t v = 0;
            for (int k = 0; k < 4; ++k) v |= (((w[k] >> j) & 1u) ? 0xFFu : 0x01u) << (8 * k);
            *(uint32_t *)(A.spins + sbase + (size_t)(ss * WS + j) * N + p * HALF + 4 * g) = v;
        }
    }
    for (int i = te; !tm.ghost && i < nT; i += T) {
        A.was[gi + i] = I.was[i];
        A.EJ[gi + i] = 2 * U[i] - 3 * N;
        A.M[gi + i] = N - 2 * ND[i];
        A.flips[gi + i] += I.fl[i];
        A.swaps[gi + i] += I.sw[i];
    }
    __syncthreads();
}

}  // namespace ea
