// ea_hbm.hip -- HBM-resident tier: chains too large for LDS (L = 24, and L = 32
// with Gaussian couplings or long ladders), and few large chains of the row,
// one-bit and (quad_sweep_kernel) group engines (spread_slots in ea_host.cpp).
//
// Spins stay in HBM in the sublattice layout.  A sweep is one launch with one
// workgroup per slot: the spins (N bytes) of the slot's walker are loaded into
// LDS, both half-sweeps run there (a barrier between them replaces a launch),
// and the spins go back.  The replica exchange of the sweep before is decided
// at the start of the launch, by the workgroups of both slots of a pair alike
// from the energies that launch left, and the snapshot of that sweep, if one is
// due, is taken from the spins just loaded, before they change.  What one
// workgroup writes and another reads (the map; energies and magnetisations, by
// slot between the sweeps of a chunk) alternates between two buffers from
// launch to launch.  After a chunk's last sweep hbm_exchange_kernel decides the
// exchange that is left and writes the maps, and energies and magnetisations by
// walker, and hbm_snapshot_kernel takes the last snapshot if due.
//
// Bound: few chains, the launch and its chain of loads (map and energies, then
// spins, then couplings: about 12 us a sweep); many, VALU issue and the
// couplings from L2 (blocks are dealt to XCDs so that a sample's walkers share
// one).  Per sweep as four launches (two half-sweeps over spins in HBM,
// exchange, snapshot) and now, 50 sweeps a call: L = 24 Gaussian, 16 temperatures, 1 / 8 /
// 64 samples 17.3 / 21.7 / 75.8 us and 11.8 / 13.6 / 67.8; +-1, 8 / 64 samples
// 20.4 / 67.7 and 12.2 / 55.5; L = 32 Gaussian, 32 temperatures, 2 / 16 samples
// 22.9 / 77.5 and 19.0 / 69.5.  Bonds of the next word loaded a word ahead: 110
// registers for 80, 4190 us for 3392 at 64 samples.
#include <type_traits>

#include "ea_device.hpp"
#include "ea_group.hpp"
#include "ea_item.hpp"
#include "ea_types.hpp"
#include "ea_update.hpp"

namespace ea {

__device__ __forceinline__ int xcd_block(int b, int nb)
{
    const int nb8 = nb & ~7;
    return b < nb8 ? (b & 7) * (nb8 >> 3) + (b >> 3) : b;
}

// The same for +-1 couplings (int8x4 bond words Ja..Jzn): a bond-spin product
// byte n ^ J is 0x00 for +1 and 0xFE for -1, so per byte c = number of -1
// products and S_J = 6 - 2c.  Acceptance uses the slot's threshold table
// thr[a*7 + b] (a = (s_i+1)/2, b = (S_J+6)/2): accept iff dE <= 0 (bit a*7+b of
// down_mask, set on the host from 2 s (S_J + h) <= 0) or w < thr.  S_u = S_J.
__device__ __forceinline__ uint32_t update_word_pm1(uint32_t Sv, uint32_t Xa, uint32_t Xs, uint32_t Yp, uint32_t Ym,
                                                    uint32_t Zp, uint32_t Zm, uint32_t Ja, uint32_t Js, uint32_t Jy,
                                                    uint32_t Jyn, uint32_t Jz, uint32_t Jzn, const u32x4 rw,
                                                    const uint32_t *thr, uint32_t down_mask, int Sus[4])
{
    constexpr uint32_t LOW = 0x01010101u;
    const uint32_t cnt = (((Xa ^ Ja) >> 1) & LOW) + (((Xs ^ Js) >> 1) & LOW) + (((Yp ^ Jy) >> 1) & LOW) +
                         (((Ym ^ Jyn) >> 1) & LOW) + (((Zp ^ Jz) >> 1) & LOW) + (((Zm ^ Jzn) >> 1) & LOW);
    const uint32_t words[4] = {rw.x, rw.y, rw.z, rw.w};
    uint32_t fm = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int sh = 8 * i;
        const int b = 6 - (int)((cnt >> sh) & 0xFFu);               // (S_J + 6) / 2
        const int m = __builtin_amdgcn_sbfe((int)Sv, sh + 7, 1);  // 0: s_i = +1, -1: s_i = -1
        const int idx = (m + 1) * 7 + b;
        const bool accept = ((down_mask >> idx) & 1u) | (words[i] < thr[idx]);
        fm |= accept ? 0xFEu << sh : 0u;
        Sus[i] = 2 * b - 6;
    }
    return fm;
}

struct HbmTally {
    int accE = 0;  // second half: sum of (S_u + hgrid) XOR m' over the thread's sites
    int nd = 0;    // down spins after the update, both halves
    int nd1 = 0;   // of the second half
    int bf = 0;    // set bits of the flip masks (7 per flipped byte)
};

// What a sweep needs of the walker's slot.
struct HbmSlot {
    PhiloxSlot ps;
    float ka, kb, b2, h32;
    const uint32_t *thr;
};

// Word i of the rows with y + z = EPS + P (mod 2) of sublattice P (one class of
// rows: eps = (y + z + P) & 1 is the same for all its words, see ea_row.hpp for
// the x neighbours): its word index and those of its neighbours.
template <int L, int P, int EPS>
struct HbmWord {
    static constexpr int WPR = L / 8, HL = L / 2, WORDS = L * L / 2 * WPR;
    int row, k, g, g_x, g_yp, g_ym, g_zp, g_zm;
    __device__ __forceinline__ explicit HbmWord(int i)
    {
        const int rr = i / WPR, z = rr / HL, y = 2 * (rr - z * HL) + ((z + EPS + P) & 1);
        k = i - rr * WPR;
        const int kx = EPS ? (k + 1 == WPR ? 0 : k + 1) : (k == 0 ? WPR - 1 : k - 1);
        row = y + L * z;
        g = row * WPR + k;
        g_x = row * WPR + kx;
        g_yp = y + 1 == L ? g - (L - 1) * WPR : g + WPR;
        g_ym = y == 0 ? g + (L - 1) * WPR : g - WPR;
        g_zp = z + 1 == L ? g - (L - 1) * L * WPR : g + L * WPR;
        g_zm = z == 0 ? g + (L - 1) * L * WPR : g - L * WPR;
    }
};

// The bonds of a word: own +x, +y, +z, the other
// sublattice's +x at the same index, the -y and -z neighbours' +y and +z, and
// the element before the word (Gaussian) or the word before it (+-1).
template <int JK>
struct HbmBonds {
    typedef typename std::conditional<JK == 0, int4, uint32_t>::type V;
    V x, y, z, v, ym, zm;
    uint32_t e;

    template <int L, int P, int EPS>
    __device__ __forceinline__ void load(const SweepArgs &A, const SampleDev &d, const HbmWord<L, P, EPS> &w)
    {
        constexpr int HALF = L * L * L / 2;
        const V *J = (const V *)(JK == 0 ? (const char *)(A.Ju + d.J_off) : (const char *)A.J + d.J_off);
        const V *Jp = J + P * 3 * (HALF / 4), *Jo = J + (1 - P) * 3 * (HALF / 4);
        x = Jp[w.g];
        y = Jp[HALF / 4 + w.g];
        z = Jp[2 * (HALF / 4) + w.g];
        v = Jo[w.g];
        ym = Jo[HALF / 4 + w.g_ym];
        zm = Jo[2 * (HALF / 4) + w.g_zm];
        if constexpr (!EPS) {
            if constexpr (JK == 0) e = (uint32_t)((const int *)Jo)[4 * w.g_x + 3];
            else e = Jo[w.g_x];
        }
    }
};

// The words of one class; S: the walker's spins in LDS.
template <int L, int JK, int P, int EPS>
__device__ __forceinline__ void hbm_class(const SweepArgs &A, const SampleDev &d, uint8_t *S, const HbmSlot &sl,
                                          const RoundKeys &key, HbmTally &ty)
{
    constexpr int N = L * L * L, HALF = N / 2;
    typedef HbmWord<L, P, EPS> Word;
    uint8_t *own = S + P * HALF;
    const uint8_t *oth = S + (1 - P) * HALF;
#pragma unroll 1
    for (int i = threadIdx.x; i < Word::WORDS; i += hbm_threads(L)) {
        const Word w(i);
        HbmBonds<JK> b;
        b.template load<L, P, EPS>(A, d, w);
        const uint32_t Sv = *(const uint32_t *)(own + 4 * w.g);
        const uint32_t Xa = *(const uint32_t *)(oth + 4 * w.g);
        const uint32_t Xo = *(const uint32_t *)(oth + 4 * w.g_x);
        const uint32_t Yp = *(const uint32_t *)(oth + 4 * w.g_yp);
        const uint32_t Ym = *(const uint32_t *)(oth + 4 * w.g_ym);
        const uint32_t Zp = *(const uint32_t *)(oth + 4 * w.g_zp);
        const uint32_t Zm = *(const uint32_t *)(oth + 4 * w.g_zm);
        const u32x4 rw = sl.ps.call(philox_group((uint32_t)w.g, d.sample_id, A.key1), key);
        const uint32_t Xs = __builtin_amdgcn_perm(Xa, Xo, EPS ? 0x00070605u : 0x06050403u);
        uint32_t fm;
        int Sus[4];
        if constexpr (JK == 0) {
            // bonds to the aligned x neighbour (x + 1 if eps = 0, else x - 1) and the shifted one
            int Ja[4], Js[4];
            if constexpr (EPS) {
                Ja[0] = b.v.x; Ja[1] = b.v.y; Ja[2] = b.v.z; Ja[3] = b.v.w;
                Js[0] = b.x.x; Js[1] = b.x.y; Js[2] = b.x.z; Js[3] = b.x.w;
            } else {
                Ja[0] = b.x.x; Ja[1] = b.x.y; Ja[2] = b.x.z; Ja[3] = b.x.w;
                Js[0] = (int)b.e; Js[1] = b.v.x; Js[2] = b.v.y; Js[3] = b.v.z;
            }
            const int Jy[4] = {b.y.x, b.y.y, b.y.z, b.y.w}, Jyn[4] = {b.ym.x, b.ym.y, b.ym.z, b.ym.w};
            const int Jz[4] = {b.z.x, b.z.y, b.z.z, b.z.w}, Jzn[4] = {b.zm.x, b.zm.y, b.zm.z, b.zm.w};
            const float kav[4] = {sl.ka, sl.ka, sl.ka, sl.ka}, kbv[4] = {sl.kb, sl.kb, sl.kb, sl.kb};
            fm = update_word_gauss(Sv, Xa, Xs, Yp, Ym, Zp, Zm, Ja, Js, Jy, Jyn, Jz, Jzn, rw, kav, kbv,
                                         [&](int) { return sl.b2; }, sl.h32, d.hgrid, Sus) &
                 0xFEFEFEFEu;
        } else {
            const uint32_t Ja = EPS ? b.v : b.x, Js = EPS ? b.x : __builtin_amdgcn_perm(b.v, b.e, 0x06050403u);
            fm = update_word_pm1(Sv, Xa, Xs, Yp, Ym, Zp, Zm, Ja, Js, b.y, b.ym, b.z, b.zm, rw, sl.thr, d.down_mask, Sus);
        }
        const uint32_t Sn = Sv ^ fm;
        *(uint32_t *)(own + 4 * w.g) = Sn;
        ty.bf += __builtin_popcount(fm);
        const int nd = __builtin_popcount(Sn & 0x80808080u);
        ty.nd += nd;
        if constexpr (P == 1) {
            tally_final(Sv, fm, Sus, ty.accE);
            ty.nd1 += nd;
        }
    }
}

// Snapshot rows of one walker (bit x of row (y, z) set iff the spin is -1): a
// word of sublattice p holds every other x of its row, from x = 8 k +
// ((p + y + z) & 1).
__device__ __forceinline__ void hbm_rows(const uint32_t *S, int L, uint32_t *dst, int first, int step)
{
    const int wpr = L / 8;
    for (int row = first; row < L * L; row += step) {
        const int yz = ((row % L) + row / L) & 1;
        uint32_t bits = 0;
        if (L & 7) {
            const int8_t *Sb = (const int8_t *)S;
            for (int x = 0; x < L; ++x)
                bits |= (uint32_t)(Sb[((x + yz) & 1) * (L * L * L / 2) + ((x + L * row) >> 1)] < 0) << x;
            dst[row] = bits;
            continue;
        }
        for (int k = 0; k < wpr; ++k) {
            // signs at bits 7, 15, 23, 31 to bits 0, 2, 4, 6
            const uint32_t even = (((S[row * wpr + k] >> 7) & 0x01010101u) * 0x01041040u) >> 24 & 0x55u;
            const uint32_t odd = (((S[(L * L + row) * wpr + k] >> 7) & 0x01010101u) * 0x01041040u) >> 24 & 0x55u;
            bits |= (even << yz | odd << (1 - yz)) << (8 * k);
        }
        dst[row] = bits;
    }
}

// Whether a measurement is due after done sweeps, and its frame in this chunk.
__device__ __forceinline__ bool hbm_due(const SweepArgs &A, int64_t done, int64_t &f)
{
    if (A.measure_every <= 0 || done <= A.measure_start) return false;
    const int64_t x = done - A.measure_start;  // (a 64-bit division takes about 0.6 us of a lone wave)
    if (x >> 31 == 0 ? (uint32_t)x % (uint32_t)A.measure_every != 0 : x % A.measure_every != 0) return false;
    f = measurements_upto(done, A.measure_every, A.measure_start) -
        measurements_upto(A.state[0], A.measure_every, A.measure_start) - 1;
    return true;
}

// Slot t's walker in a sweep, after the exchange that follows the sweep before
// (the first sweep of a chunk finds it done), and its energy then: first all
// loads, so that a caller can do other work while they are on the way, then the
// decision.
struct SlotWalker {
    int w, wo, lo;
    bool pair;
    int64_t ej, ejo;
    int32_t m, mo;
    double bt, bo, E;

    __device__ __forceinline__ void load(const SweepArgs &A, const SampleDev &d, int64_t n, int gi, int t)
    {
        w = A.was[gi + t];
        E = 0.0;
        if (A.it > 0) {
            const bool odd = (n - 1) & 1;
            lo = odd ? (t - 1) | 1 : t & ~1;
            pair = lo >= 0 && lo + 1 < d.n_T;
            const int to = !pair ? t : t == lo ? t + 1 : t - 1;
            wo = A.was[gi + to];
            ej = A.EJ[gi + t];
            ejo = A.EJ[gi + to];
            m = A.M[gi + t];
            mo = A.M[gi + to];
            bt = A.beta[d.slot_off + t];
            bo = A.beta[d.slot_off + to];
        }
    }

    // count: this thread counts the swap of the pair (one thread per slot)
    template <int JK>
    __device__ __forceinline__ void decide(const SweepArgs &A, const SampleDev &d, int r, int64_t n, int gi, int t,
                                           bool count)
    {
        if (A.it > 0) {
            const double unit = JK == 0 ? 0x1p-18 : 1.0, hd = (double)d.h32;
            const double Eo = (double)ejo * unit - hd * (double)mo;
            E = (double)ej * unit - hd * (double)m;
            const double D = t == lo ? (bt - bo) * (E - Eo) : (bo - bt) * (Eo - E);
            const u32x4 q = philox4x32_10(0u, (uint32_t)(n - 1),
                                          (PURPOSE_EXCHANGE << 28) | ((uint32_t)lo << 1) | (uint32_t)r, d.sample_id,
                                          A.key0, A.key1);
            if (pair && exchange_accept(q.x, q.y, D)) {
                if (t == lo && count) atomicAdd((unsigned long long *)&A.swaps[gi + lo], 1ull);
                w = wo;
                E = Eo;
            }
        }
    }
};

template <int L, int JK, int VAR>
__global__ void __launch_bounds__(hbm_threads(L)) hbm_sweep_kernel(SweepArgs A)
{
    constexpr int N = L * L * L, T = hbm_threads(L), W = T / 64;
    __shared__ __attribute__((aligned(16))) uint8_t S[N];
    __shared__ long long se[W];
    __shared__ int sc[2][W];
    __shared__ uint32_t thr[14];
    const int wi = xcd_block(blockIdx.x, gridDim.x);
    const int code = A.walkers[wi];
    const SampleDev d = sample_of_item(A.samples, code >> 7);
    const int r = (code >> 6) & 1, t = code & 63, tid = threadIdx.x;
    const int nT = d.n_T, gi = 2 * d.slot_off + r * nT;
    const int64_t n = A.state[0] + A.it;
    const float b32 = A.beta32[d.slot_off + t];
    SlotWalker sw;
    sw.load(A, d, n, gi, t);
    sw.decide<JK>(A, d, r, n, gi, t, tid == 0);
    const int w = sw.w;
    const double Et = sw.E;
    uint4 *glob = (uint4 *)(A.spins + d.spin_off + ((size_t)r * nT + w) * N);
    constexpr int CHUNKS = N / 16, PER = (CHUNKS + T - 1) / T;
    static_assert(PER <= 4);
    // all of the spins on the way at once
    const auto chunk = [&](int k) { return glob[min(k * T + tid, CHUNKS - 1)]; };
    const uint4 v0 = chunk(0), v1 = PER > 1 ? chunk(1) : v0, v2 = PER > 2 ? chunk(2) : v0, v3 = PER > 3 ? chunk(3) : v0;
    if (tid == 0) A.was_next[gi + t] = w;
    if (JK == 1 && tid < 14) thr[tid] = A.lut[((size_t)d.slot_off + t) * 14 + tid];
    const auto keep = [&](int k, const uint4 v) {
        if (k < PER && k * T + tid < CHUNKS) ((uint4 *)S)[k * T + tid] = v;
    };
    keep(0, v0);
    keep(1, v1);
    keep(2, v2);
    keep(3, v3);
    __syncthreads();
    int64_t f;
    if (A.it > 0 && hbm_due(A, n, f)) {
        hbm_rows((const uint32_t *)S, L, A.frames + f * A.frame_words + d.frame_off + ((size_t)r * nT + t) * L * L, tid, T);
        if (tid == 0) A.frameE[f * 2 * A.total_slots + gi + t] = Et;
        __syncthreads();
    }
    HbmSlot sl;
    const float cp = two_beta_log2e(b32);
    sl.ka = cp * 0x1p-18f;
    sl.kb = cp * (d.h32 - (float)d.hgrid * 0x1p-18f);
    sl.b2 = 2.0f * b32;
    sl.h32 = d.h32;
    sl.thr = thr;
    const uint32_t c2 = (PURPOSE_METROPOLIS << 28) | ((uint32_t)t << 1) | (uint32_t)r;
    RoundKeys key;
    key.init(A.key0, A.key1);
    HbmTally ty;
    sl.ps.init((uint32_t)(2 * n), c2, A.key0, A.key1);
    hbm_class<L, JK, 0, 0>(A, d, S, sl, key, ty);
    hbm_class<L, JK, 0, 1>(A, d, S, sl, key, ty);
    __syncthreads();
    sl.ps.init((uint32_t)(2 * n + 1), c2, A.key0, A.key1);
    hbm_class<L, JK, 1, 0>(A, d, S, sl, key, ty);
    hbm_class<L, JK, 1, 1>(A, d, S, sl, key, ty);
    // E_J = -(sum of s' S_u over the odd sites): accE + nd1 sums s' (S_u +
    // hgrid), less hgrid sum s' (a thread has at most 32 odd sites,
    // L = 32: 32 x 12 2^21 < 2^31)
    const long long e = wave_sum_i64((long long)ty.accE + (1 + 2 * (long long)d.hgrid * (JK == 0)) * ty.nd1);
    // set bits of the flip masks (at most 7 x 4096 sites a wave) and down spins
    const int s2 = wave_sum_i32(ty.bf + (ty.nd << 16)), fl = s2 & 0xFFFF, nd = s2 >> 16;
    if ((tid & 63) == 0) {
        se[tid >> 6] = e;
        sc[0][tid >> 6] = fl;
        sc[1][tid >> 6] = nd;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (k * T + tid < CHUNKS) glob[k * T + tid] = ((const uint4 *)S)[k * T + tid];
    if (tid == 0) {
        long long E = 0;
        int bf = 0, down = 0;
        for (int k = 0; k < W; ++k) {
            E += se[k];
            bf += sc[0][k];
            down += sc[1][k];
        }
        A.EJ_next[gi + t] = (JK == 0 ? (long long)d.hgrid * (N / 2) : 0) - E;
        A.M_next[gi + t] = N - 2 * down;
        atomicAdd((unsigned long long *)&A.flips[gi + t], (unsigned long long)(bf / 7));
    }
}

// The exchange after a chunk's last sweep, one wave per (sample, chain): reads
// the buffers that the last sweep wrote, leaves all of them in the first ones.
__global__ void __launch_bounds__(64) hbm_exchange_kernel(SweepArgs A)
{
    const int code = A.items[blockIdx.x];
    const SampleDev d = A.samples[code >> 1];
    const int r = code & 1, t = threadIdx.x;
    const int nT = d.n_T, gi = 2 * d.slot_off + r * nT;
    const int64_t n = A.state[0] + A.it;
    __shared__ int32_t was[MAX_T], sow[MAX_T], sw[MAX_T];
    __shared__ double b64[MAX_T], E[MAX_T];
    int64_t ej = 0;
    int32_t m = 0;
    if (t < nT) {
        was[t] = A.was[gi + t];
        sw[t] = 0;
        b64[t] = A.beta[d.slot_off + t];
        ej = A.EJ[gi + t];
        m = A.M[gi + t];
        E[was[t]] = (double)ej * (A.jkind == 0 ? 0x1p-18 : 1.0) - (double)d.h32 * (double)m;
    }
    __syncthreads();
    if (t < nT) sow[was[t]] = t;
    __syncthreads();
    ItemLds I{};
    I.was = was;
    I.sow = sow;
    I.sw = sw;
    I.b64 = b64;
    RoundKeys key;
    key.init(A.key0, A.key1);
    const int w0 = t < nT ? was[t] : t, w = exchange_slots(A, d, r, n, I, t, key, [&](int ww) { return E[ww]; });
    __syncthreads();
    if (t < nT) {
        A.was_next[gi + t] = w;
        A.EJ_next[gi + w0] = ej;
        A.M_next[gi + w0] = m;
        A.swaps[gi + t] += sw[t];
        int64_t f;
        if (hbm_due(A, n + 1, f)) A.frameE[f * 2 * A.total_slots + gi + t] = E[w];
    }
}

// Snapshot of one (sample, chain, slot) after a chunk's last sweep, when a
// measurement is due (the launch returns at once otherwise).
__global__ void __launch_bounds__(256) hbm_snapshot_kernel(SweepArgs A)
{
    int64_t f;
    if (!hbm_due(A, A.state[0] + A.it + 1, f)) return;
    const int code = A.walkers[blockIdx.x];
    const SampleDev d = A.samples[code >> 7];
    const int r = (code >> 6) & 1, nT = d.n_T, L = d.L;
    const size_t base = d.spin_off + (size_t)r * nT * L * L * L;
    for (int t = code & 63; t < min((code & 63) + A.per, nT); ++t) {
        const uint32_t *Sw = (const uint32_t *)(A.spins + base + (size_t)A.was[2 * d.slot_off + r * nT + t] * L * L * L);
        hbm_rows(Sw, L, A.frames + f * A.frame_words + d.frame_off + ((size_t)r * nT + t) * L * L, threadIdx.x, blockDim.x);
    }
}

// Few chains of the group engine (Gaussian couplings, L = 12 and 14): the same
// form with a workgroup per four consecutive slots, whose walkers are brought
// into the group engine's words (a word: one site of the four) in LDS; its
// update and neighbour table, one site group per thread and half-sweep.
// Bound: as above; the table and the couplings are formed while the map and
// the energies are on the way.
// At 16 samples x 21 temperatures, L = 14, a sweep takes 12.3 us (21.3 by the
// group engine, a workgroup per chain), half of it the two half-sweeps; forming
// the table after the exchange's loads came back took 13.0.
// Bytes i of four words to word i: rows and columns of a 4 x 4 byte matrix.
__device__ __forceinline__ void transpose_bytes(uint32_t a[4])
{
    const uint32_t p = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u), q = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u);
    const uint32_t u = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u), v = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
    a[0] = __builtin_amdgcn_perm(q, p, 0x05040100u);
    a[1] = __builtin_amdgcn_perm(q, p, 0x07060302u);
    a[2] = __builtin_amdgcn_perm(v, u, 0x05040100u);
    a[3] = __builtin_amdgcn_perm(v, u, 0x07060302u);
}

template <int L>
__global__ void __launch_bounds__(quad_threads(L), 4) quad_sweep_kernel(SweepArgs A)
{
    constexpr int N = L * L * L, HALF = N / 2, PS = HALF + 1, G4 = HALF / 4, T = quad_threads(L), W = T / 64;
    static_assert(T >= G4, "a thread takes one site group of a half-sweep");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint4 *NB = (uint4 *)smem;
    int *Jl = (int *)(NB + HALF);
    uint32_t *SG = (uint32_t *)(Jl + 3 * N);
    __shared__ long long se[4][W];
    __shared__ int sc[4][W];
    __shared__ float b32[4];
    const int code = A.walkers[xcd_block(blockIdx.x, gridDim.x)];
    const SampleDev d = sample_of_item(A.samples, code >> 7);
    const int r = (code >> 6) & 1, t0 = code & 63, tid = threadIdx.x;
    const int nT = d.n_T, gi = 2 * d.slot_off + r * nT;
    const int64_t n = A.state[0] + A.it;
    // lane i mod 4 decides slot t0 + i (beyond the ladder: its last slot, and
    // the result is not used)
    const int own = min(t0 + (tid & 3), nT - 1);
    const bool real = t0 + (tid & 3) < nT;
    SlotWalker sw;
    sw.load(A, d, n, gi, own);
    const float b = A.beta32[d.slot_off + own];
    constexpr int JQ = 3 * N / 4, JPER = (JQ + T - 1) / T;
    const float4 *src = (const float4 *)((const float *)A.J + d.J_off);  // J_off is a multiple of 4
    float4 v[JPER];
#pragma unroll
    for (int k = 0; k < JPER; ++k) v[k] = src[min(k * T + tid, JQ - 1)];
    __builtin_amdgcn_sched_barrier(0);
    for (int h = tid; h < HALF; h += T) NB[(h & 3) * G4 + (h >> 2)] = nbr_entry<L>(h);
    sw.decide<0>(A, d, r, n, gi, own, real && tid < 4);
    if (tid < 4) {
        b32[tid] = b;
        if (real) A.was_next[gi + own] = sw.w;
    }
    // couplings as exact int32 multiples of 2^-18
#pragma unroll
    for (int k = 0; k < JPER; ++k)
        if (k * T + tid < JQ)
            ((int4 *)Jl)[k * T + tid] = make_int4((int)(v[k].x * 262144.0f), (int)(v[k].y * 262144.0f),
                                                  (int)(v[k].z * 262144.0f), (int)(v[k].w * 262144.0f));
    // spins: four sites of each walker, to four words (padding walkers: +1)
    uint32_t *glob[4], valid = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int w = __builtin_amdgcn_readlane(sw.w, i);
        glob[i] = (uint32_t *)(A.spins + d.spin_off + ((size_t)r * nT + w) * N);
        valid |= (t0 + i < nT ? 0xFEu : 0u) << (8 * i);
    }
    uint32_t in[2][4];
    const int st = min(tid, G4 - 1);
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) in[p][i] = glob[i][p * G4 + st];
#pragma unroll
    for (int p = 0; p < 2; ++p)
        if (tid < G4) {
            uint32_t a[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = t0 + i < nT ? in[p][i] : 0x01010101u;
            transpose_bytes(a);
#pragma unroll
            for (int k = 0; k < 4; ++k) SG[p * PS + 4 * tid + k] = a[k];
        }
    __syncthreads();
    int64_t f;
    if (A.it > 0 && hbm_due(A, n, f)) {
        uint32_t *dst = A.frames + f * A.frame_words + d.frame_off + ((size_t)r * nT + t0) * L * L;
        for (int i = tid; i < 4 * L * L; i += T) {
            const int k = i / (L * L), row = i - k * (L * L), e = ((row % L) + row / L) & 1;
            if (t0 + k >= nT) break;
            uint32_t bits = 0;
            for (int x = 0; x < L; ++x)
                bits |= (SG[((x + e) & 1) * PS + row * (L / 2) + (x >> 1)] >> (8 * k + 7) & 1u) << x;
            dst[i] = bits;
        }
        if (tid < 4 && real) A.frameE[f * 2 * A.total_slots + gi + own] = sw.E;
        __syncthreads();
    }
    GroupLane ln;
    int ts[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        ts[i] = min(t0 + i, nT - 1);
        const float cp = two_beta_log2e(b32[i]);
        ln.ka[i] = cp * 0x1p-18f;
        ln.kb[i] = cp * (d.h32 - (float)d.hgrid * 0x1p-18f);
        ln.t[i] = i;
    }
    ln.flip = valid;
    ln.one = (valid >> 1) & 0x01010101u;
    ln.h32 = d.h32;
    RoundKeys key;
    key.init(A.key0, A.key1);
    GroupTally ty;
    const auto slot_words = [&](int p) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            ln.ps[i].init((uint32_t)(2 * n + p), (PURPOSE_METROPOLIS << 28) | ((uint32_t)ts[i] << 1) | (uint32_t)r, A.key0,
                          A.key1);
    };
    slot_words(0);
    if (tid < G4) group_item<L, 0>(A, d, SG, Jl, b32, NB, 1, 0, tid, key, ln, ty);
    __syncthreads();
    slot_words(1);
    if (tid < G4) group_item<L, 1>(A, d, SG, Jl, b32, NB, 1, 0, tid, key, ln, ty);
    // back to four sites of each walker (the odd ones are the thread's own, the
    // even ones have the barrier)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int k = 0; k < 4; ++k) in[p][k] = SG[p * PS + 4 * st + k];
        transpose_bytes(in[p]);
    }
    // a thread's (S_u + hgrid) XOR m' over four sites is at most 48 2^21 + 4, a
    // row of sixteen below 2^31; down spins and flips of a wave at most 512 each
    const int hg1 = 2 * d.hgrid + 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e16 = group_sum_dpp<16>(ty.accE[i]);
        const int nd1 = (int)(ty.nd1 >> (8 * i)) & 0xFF;
        const int c = wave_sum_i32((nd1 + ((int)(ty.nd0 >> (8 * i)) & 0xFF)) |
                                   ((int)(ty.flips >> (8 * i)) & 0xFF) << 16);
        const int nd = wave_sum_i32(nd1);
        const long long e = (long long)__builtin_amdgcn_readlane(e16, 0) + __builtin_amdgcn_readlane(e16, 16) +
                            __builtin_amdgcn_readlane(e16, 32) + __builtin_amdgcn_readlane(e16, 48);
        if ((tid & 63) == 0) {
            se[i][tid >> 6] = e + (long long)hg1 * nd;
            sc[i][tid >> 6] = c;
        }
    }
    __syncthreads();
    // (stores after the last barrier, which would wait for them)
    if (tid < G4) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (t0 + i < nT) glob[i][p * G4 + tid] = in[p][i];
    }
    if (tid < 4 && real) {
        long long E = -(long long)d.hgrid * HALF;
        int c = 0;
        for (int k = 0; k < W; ++k) {
            E += se[tid][k];
            c += sc[tid][k];
        }
        A.EJ_next[gi + own] = -E;
        A.M_next[gi + own] = N - 2 * (c & 0xFFFF);
        atomicAdd((unsigned long long *)&A.flips[gi + own], (unsigned long long)(c >> 16));
    }
}

template __global__ void quad_sweep_kernel<12>(SweepArgs);
template __global__ void quad_sweep_kernel<14>(SweepArgs);

#define EA_HBM(Lv)                                                   \
    template __global__ void hbm_sweep_kernel<Lv, 0, 0>(SweepArgs); \
    template __global__ void hbm_sweep_kernel<Lv, 1, 0>(SweepArgs); \
    template __global__ void hbm_sweep_kernel<Lv, 0, 1>(SweepArgs); \
    template __global__ void hbm_sweep_kernel<Lv, 1, 1>(SweepArgs);
EA_HBM(8)
EA_HBM(16)
EA_HBM(24)
EA_HBM(32)
#undef EA_HBM

}  // namespace ea
