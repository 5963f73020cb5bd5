// ea_kernels.hip -- gfx950 kernels of the Edwards-Anderson Monte Carlo engine.
//
// LDS-resident tier (L <= 16).  One workgroup owns one (sample, chain) work
// item for a chunk of K sweeps: the chain's n_T walkers (int8 spins) and the
// sample's couplings are loaded into LDS once, then every sweep of the chunk --
// two checkerboard half-sweeps of Metropolis updates (Methods: single-spin-flip
// Monte Carlo), the exact energy bookkeeping, the replica-exchange pass
// (Methods: parallel tempering) and, when due, a snapshot of the chain in slot
// order for the overlap measurement -- runs out of LDS.  Spins and maps go back
// to HBM once per chunk.
//
// The two chains of a sample only meet in the overlap q_i = s_i^a s_i^b
// (eq. 2), so they are independent work items; the measurement kernel
// combines their snapshots after the chunk.
//
// Two half-sweep engines share that frame here:
//  * row engine (L = 8, 16; Gaussian couplings): a thread owns one walker and
//    one (x-word, y) column and walks z; it works on 4 sites at once (one int8x4
//    word = one Philox call), keeps couplings as integer 2^-18 units and the
//    walker's energy/flip tallies in registers for the whole sweep;
//  * site engine (any even L <= 16, either coupling kind; chains too small for
//    the group engine): a thread takes a 4-site group of any walker and updates
//    its sites one by one.  Outside the batch launch the tiny kernel takes its
//    place up to 1024 odd sites (L = 2, and L = 4 with up to 32 temperatures).
// The group engine (ea_group.hip: one word = one site of four walkers) and the
// one-bit engine (ea_bits.hip: +-1 couplings) use the same frame with their
// own LDS layouts.  This file also holds the overlap measurement and the setup
// and check kernels (HBM-resident tier: ea_hbm.hip; finalize: ea_finalize.hip).
#include <type_traits>

#include "ea_device.hpp"
#include "ea_item.hpp"
#include "ea_row.hpp"
#include "ea_types.hpp"
#include "ea_update.hpp"

namespace ea {

// One kernel per (engine, L, coupling kind).  VAR only separates the symbol
// of the one-sample-per-launch comparator from the batched launch in
// profiles; the code is identical.
template <int L, int JK, int VAR>
__global__ void __launch_bounds__(1024) site_sweep_kernel(SweepArgs A)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    for (int item = blockIdx.x; item < A.n_items; item += gridDim.x) {
        const int code = A.items[item];
        run_item<L, JK, false>(A, A.samples[code >> 1], code & 1, smem, whole_block(), (int)threadIdx.x);
    }
}

// Tiny chains (L = 2 or 4, at most 1024 odd sites over the ladder): a lane per
// (walker, site pair), which keeps its even and its odd site's spin, couplings
// and neighbour addresses in registers for the whole chunk; only neighbour
// spins are read from LDS.  A walker's lanes lie in one wave, so energy, down
// spins and flips are a lane reduction and two counts of a ballot, once a
// sweep, and every walker decides its own exchange from the energies of its
// slot and the other's: two barriers a sweep.
//
// The exchange's random words are drawn ahead of time, a thread per (sweep,
// pair), so a sweep only reads them.
//
// Bound: one wave's chain of instructions, about 2100 cycles a sweep at few
// chains (a half-sweep 500, energies and a barrier 450, the exchange 500).
// 100 sweeps, by the site engine in workgroups of 1024 threads and now: L = 4,
// 8 temperatures, 16 / 512 / 4096 samples 424 / 1639 / 13024 us and 99 / 184 /
// 1112; +-1 16 / 4096 samples 376 / 11582 and 93 / 1098; L = 2, 16 temperatures,
// 4096 samples 9240 and 311.  Every sweep's words drawn in it, the exact test
// for every site and exchange tables in global memory: 108 / 224 / 1430, 100 /
// 1227, 385.
template <int L, int JK, int VAR>
__global__ void __launch_bounds__(1024) tiny_sweep_kernel(SweepArgs A)
{
    constexpr int N = L * L * L, HALF = N / 2, HL = L / 2;
    __shared__ int8_t S[2 * 1024];
    __shared__ double Es[2][MAX_T], db[MAX_T];  // db: of beta, slots t and t + 1
    __shared__ float beta[MAX_T];
    __shared__ int32_t map[MAX_T], fl[MAX_T], sw[MAX_T];
    extern __shared__ uint2 ex[];  // [2][threads]
    __shared__ uint32_t lut[JK == 1 ? 14 * MAX_T : 1];
    const int code = A.items[blockIdx.x];
    const SampleDev d = sample_of_item(A.samples, code >> 1);
    const int r = code & 1, nT = d.n_T, gi = 2 * d.slot_off + r * nT;
    const int tid = threadIdx.x, w = tid / HALF, h = tid % HALF;
    const bool on = w < nT;
    for (int i = tid; i < nT; i += blockDim.x) {
        map[A.was[gi + i]] = i;
        fl[i] = 0;
        sw[i] = 0;
        db[i] = A.beta[d.slot_off + i] - A.beta[d.slot_off + min(i + 1, nT - 1)];
        beta[i] = A.beta32[d.slot_off + i];
    }
    if (JK == 1)
        for (int i = tid; i < 14 * nT; i += blockDim.x) lut[i] = A.lut[(size_t)d.slot_off * 14 + i];

    // the lane's two sites (sublattice index h): spin, neighbours in LDS, bonds
    // in the order x+, x-, y+, y-, z+, z-
    const int row = h / HL, j = h - row * HL, y = row % L, z = row / L;
    typedef typename std::conditional<JK == 0, float, int>::type Bond;
    int8_t *glob = A.spins + d.spin_off + (size_t)r * nT * N + (size_t)w * N;
    int s[2], nb[2][6];
    Bond J[2][6];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int x = 2 * j + ((y + z + p) & 1);
        const int xp = x + 1 == L ? 0 : x + 1, xm = x == 0 ? L - 1 : x - 1;
        const int yp = y + 1 == L ? 0 : y + 1, ym = y == 0 ? L - 1 : y - 1;
        const int zp = z + 1 == L ? 0 : z + 1, zm = z == 0 ? L - 1 : z - 1;
        const int q[6] = {(xp + L * row) >> 1,           (xm + L * row) >> 1,           (x + L * (yp + L * z)) >> 1,
                          (x + L * (ym + L * z)) >> 1,   (x + L * (y + L * zp)) >> 1,   (x + L * (y + L * zm)) >> 1};
        s[p] = on ? glob[p * HALF + h] : 0;
        if (on) S[w * N + p * HALF + h] = (int8_t)s[p];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            nb[p][k] = (on ? w * N : 0) + (1 - p) * HALF + q[k];
            // a bond is stored with the site at its lower end along the axis
            const int e = (k & 1) ? ((1 - p) * 3 + k / 2) * HALF + q[k] : (p * 3 + k / 2) * HALF + h;
            if constexpr (JK == 0) J[p][k] = ((const float *)A.J)[d.J_off + e];
            else J[p][k] = ((const int8_t *)A.J)[d.J_off + e];
        }
    }
    __syncthreads();
    int t = on ? map[w] : 0;
    // the walker's lanes within the wave
    const int lane = tid & 63;
    const uint64_t lanes = (HALF >= 64 ? ~0ull : (1ull << HALF) - 1) << (lane / HALF * HALF);
    const bool lead = on && h == HALF - 1;
    const double unit = JK == 0 ? 0x1p-18 : 1.0, hd = (double)d.h32;
    const int64_t n0 = A.state[0];
    int64_t next_meas = next_measurement(n0, A.measure_every, A.measure_start), f = 0;
    RoundKeys key;
    key.init(A.key0, A.key1);
    const uint4 pg = philox_group((uint32_t)(h >> 2), d.sample_id, A.key1);
    float b32 = beta[t], c2l = two_beta_log2e(b32);
    int ej = 0, down = 0;
    // The exchange's random words: a thread each for (sweep, pair), ahead of
    // time for as many sweeps as the threads give, into either half of ex in turn
    const int pairs = nT / 2 > 0 ? nT / 2 : 1, ahead = (int)blockDim.x / pairs, my = tid / pairs;
    const auto draw = [&](int64_t first, int half) {
        const int64_t n = first + my;
        const int lo = 2 * (tid - my * pairs) + (int)(n & 1);
        const u32x4 q = philox4x32_10(0u, (uint32_t)n, (PURPOSE_EXCHANGE << 28) | ((uint32_t)lo << 1) | (uint32_t)r,
                                      d.sample_id, A.key0, A.key1);
        ex[half * blockDim.x + tid] = make_uint2(q.x, q.y);
    };
    int half = 0, use = 0;  // of the sweep at hand
    draw(n0, 0);
    for (int it = 0; it < A.K; ++it) {
        const int64_t n = n0 + it;
        const uint32_t c2 = (PURPOSE_METROPOLIS << 28) | ((uint32_t)t << 1) | (uint32_t)r;
        int flips = 0;
        down = 0;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            int v[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) v[k] = S[nb[p][k]];
            PhiloxSlot ps;
            ps.init((uint32_t)(2 * n + p), c2, A.key0, A.key1);
            const u32x4 rw = ps.call(pg, key);
            const uint32_t word = (h & 2) ? ((h & 1) ? rw.w : rw.z) : ((h & 1) ? rw.y : rw.x);
            const int si = s[p];
            bool accept;
            int units;
            if constexpr (JK == 0) {
                // exact: every partial sum is a multiple of 2^-18 below 2^6
                float SJ = J[p][0] * (float)v[0];
#pragma unroll
                for (int k = 1; k < 6; ++k) SJ = SJ + J[p][k] * (float)v[k];
                // the binary32 estimate decides where it is safe (accept_gap; y
                // is c' times the exact -s_i f), as in the word engines
                const float sf = (float)si * (SJ + d.h32), g = accept_gap(c2l * -sf, (float)word);
                accept = g < 0.0f;
                if (__builtin_amdgcn_ballot_w64(__builtin_fabsf(g) <= ACCEPT_MARGIN) != 0) {
                    const float dE = 2.0f * sf;
                    accept = (dE <= 0.0f) | (u24_of(word) < exp_ea32(-(b32 * dE)));
                }
                units = (int)(SJ * 262144.0f);
            } else {
                units = 0;
#pragma unroll
                for (int k = 0; k < 6; ++k) units += J[p][k] * v[k];
                const float fi = (float)units + d.h32;  // its sign is exact
                accept = (si * fi <= 0.0f) | (word < lut[(t * 2 + ((si + 1) >> 1)) * 7 + ((units + 6) >> 1)]);
            }
            accept = accept && on;
            if (accept) {
                s[p] = -si;
                S[w * N + p * HALF + h] = (int8_t)-si;
            }
            flips += __popcll(__ballot(accept) & lanes);
            down += __popcll(__ballot(s[p] < 0) & lanes);
            // minus the walker's E_J: every bond joins one even and one odd
            // site, and the even spins change no more (at most 32 x 6 2^21)
            if (p == 1) {
                ej = s[1] * units;
                if constexpr (HALF == 4) ej = group_sum_dpp<4>(ej);
                else {
                    ej = group_sum_dpp<16>(ej);
                    const auto rows = __builtin_amdgcn_permlane16_swap(ej, ej, false, false);
                    ej = (int)(rows[0] + rows[1]);  // rows 0 and 1, 2 and 3
                }
            }
            if (p == 0) __syncthreads();
        }
        if (use + 1 == ahead) draw(n + 1, half ^ 1);
        const double E = (double)-ej * unit - hd * (double)(N - 2 * down);
        if (lead) {
            Es[it & 1][t] = E;
            atomicAdd(&fl[t], flips);
        }
        __syncthreads();
        // exchange of slots lo and lo + 1: each walker decides for itself
        const bool odd = n & 1;
        const int lo = odd ? (t - 1) | 1 : t & ~1, other = t == lo ? t + 1 : t - 1;
        const bool pair = on && lo >= 0 && lo + 1 < nT;
        const int to = pair ? other : t;
        const double Eo = Es[it & 1][to], dE = t == lo ? E - Eo : Eo - E;
        const uint2 q = ex[half * blockDim.x + use * pairs + (pair ? lo >> 1 : 0)];
        if (++use == ahead) {
            use = 0;
            half ^= 1;
        }
        if (exchange_accept(q.x, q.y, db[pair ? lo : 0] * dE) && pair) {
            if (t == lo && lead) atomicAdd(&sw[lo], 1);
            t = other;
            b32 = beta[t];
            c2l = two_beta_log2e(b32);
        }
        if (n + 1 == next_meas) {
            next_meas += A.measure_every;
            if (lead) {
                map[t] = w;
                A.frameE[f * 2 * A.total_slots + gi + t] = E;
            }
            __syncthreads();
            uint32_t *dst = A.frames + f * A.frame_words + d.frame_off + (size_t)r * nT * L * L;
            for (int i = tid; i < nT * L * L; i += blockDim.x) {
                const int ts = i / (L * L);
                dst[i] = pack_row_lds<L>(S + map[ts] * N, i - ts * (L * L));
            }
            ++f;
            __syncthreads();
        }
    }
    if (on) {
        glob[h] = (int8_t)s[0];
        glob[HALF + h] = (int8_t)s[1];
    }
    if (lead) {
        A.was[gi + t] = w;
        if (A.K > 0) {
            A.EJ[gi + w] = -ej;
            A.M[gi + w] = N - 2 * down;
        }
    }
    __syncthreads();
    for (int i = tid; i < nT; i += blockDim.x) {
        A.flips[gi + i] += fl[i];
        A.swaps[gi + i] += sw[i];
    }
}

// L = 8 chains are small (two waves for 16 walkers), so their workgroups are
// held to 128 VGPRs to keep four waves per SIMD resident.
template <int L, int VAR, bool TAB, bool SPLIT>
__global__ void __launch_bounds__(ROW_MAX_THREADS, L == 8 ? 4 : 1) row_sweep_kernel(SweepArgs A)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int code = A.items[blockIdx.x];
    const Team tm = whole_block();
    run_item<L, 0, true, TAB, SPLIT>(A, sample_of_item(A.samples, code >> 1), code & 1, smem, tm, tm.tid());
}

#define EA_SITE(Lv)                                               \
    template __global__ void site_sweep_kernel<Lv, 0, 0>(SweepArgs); \
    template __global__ void site_sweep_kernel<Lv, 1, 0>(SweepArgs); \
    template __global__ void site_sweep_kernel<Lv, 0, 1>(SweepArgs); \
    template __global__ void site_sweep_kernel<Lv, 1, 1>(SweepArgs);
EA_SITE(2)
EA_SITE(4)
EA_SITE(6)
EA_SITE(8)
EA_SITE(10)
EA_SITE(12)
EA_SITE(14)
EA_SITE(16)
#undef EA_SITE
#define EA_TINY(Lv)                                               \
    template __global__ void tiny_sweep_kernel<Lv, 0, 0>(SweepArgs); \
    template __global__ void tiny_sweep_kernel<Lv, 1, 0>(SweepArgs); \
    template __global__ void tiny_sweep_kernel<Lv, 0, 1>(SweepArgs); \
    template __global__ void tiny_sweep_kernel<Lv, 1, 1>(SweepArgs);
EA_TINY(2)
EA_TINY(4)
#undef EA_TINY
#define EA_ROW(Lv, TABv)                                                    \
    template __global__ void row_sweep_kernel<Lv, 0, TABv, false>(SweepArgs); \
    template __global__ void row_sweep_kernel<Lv, 1, TABv, false>(SweepArgs); \
    template __global__ void row_sweep_kernel<Lv, 0, TABv, true>(SweepArgs);  \
    template __global__ void row_sweep_kernel<Lv, 1, TABv, true>(SweepArgs);
EA_ROW(8, true)
EA_ROW(16, true)
EA_ROW(16, false)
#undef EA_ROW

// ---------------------------------------------------------------------------
// Overlap measurement (eq. 2).  One wave per (sample, slot).  For each snapshot
// frame of the chunk: the overlap bits e = NOT(a XOR b) of the two chains'
// rows mark q_i = +1; the column counts
//   C[x][y] = #{z : e(x,y,z)},  D[x][z] = #{y : e(x,y,z)},  R[y][z] = #{x : e}
// give the count of q_i = +1 in every plane of the nine wave vectors
// k_f = (2 pi / L) u_f (each plane c = u_f . r mod L holds L^2 sites), so the
// plane sums are P_f[c] = 2 count - L^2 and
// q(k_f) = sum_c P_f[c] e^{2 pi i c / L} / N (summed in c order), added to the
// binary64 accumulators of the slot in time order.
//
// A wave may take F frames side by side, one per group of G = 64 / F lanes,
// each group at least 2 L lanes wide: the frames' counts and Fourier sums are
// independent, and their accumulation stays one frame after the other.
//
// C and D come from bit-sliced vertical counters: lane y of a group (C) adds
// the rows (y, z) over z, lane D0 + z (D) the rows (y, z) over y (D0 = L
// with frames side by side, else 32), one 32-bit word per step into six bit
// planes, and then reads the L column counts off the planes.  Tables in LDS
// use a row stride of L + 1 words, so that the strided reads of the plane
// sums fall in distinct banks.
template <int L, int D0>
__device__ __forceinline__ void column_counts(const uint32_t *eqr, int lane, int *C, int *D)
{
    constexpr int LP = L + 1;
    static_assert(D0 >= L && D0 + L <= 64, "C and D lanes apart");
    const bool isC = lane < L, isD = lane >= D0 && lane < D0 + L;
    if (!isC && !isD) return;
    const int u = isC ? lane : lane - D0;
    uint32_t c0 = 0, c1 = 0, c2 = 0, c3 = 0, c4 = 0, c5 = 0;
#pragma unroll 4
    for (int v = 0; v < L; ++v) {
        const uint32_t w = eqr[isC ? u + LP * v : v + LP * u];
        uint32_t k = c0 & w;
        c0 ^= w;
        uint32_t k2 = c1 & k;
        c1 ^= k;
        k = c2 & k2;
        c2 ^= k2;
        k2 = c3 & k;
        c3 ^= k;
        k = c4 & k2;
        c4 ^= k2;
        c5 |= k;  // counts reach at most L <= 32
    }
    int *dst = isC ? C : D;
#pragma unroll
    for (int x = 0; x < L; ++x) {
        const int cnt = (int)(((c0 >> x) & 1u) | (((c1 >> x) & 1u) << 1) | (((c2 >> x) & 1u) << 2) |
                              (((c3 >> x) & 1u) << 3) | (((c4 >> x) & 1u) << 4) | (((c5 >> x) & 1u) << 5));
        dst[x * LP + u] = cnt;
    }
}

// Frames measured side by side by one wave: as many as groups of 2 L lanes
// fit, at most two (four groups of 16 lanes, at L <= 8, measured no faster
// than one).
template <int L>
constexpr int meas_frames()
{
    return 2 * L <= 32 ? 2 : 1;
}

// LDS of one slot's measurement (per frame group g: the tables of its frame).
template <int L, int F>
struct MeasLds {
    static_assert(F >= 1 && 2 * L * F <= 64, "a group of 2 L lanes per frame");
    static constexpr int LP = L + 1, G = 64 / F;
    static constexpr int GC = G / L;  // chunks of v per plane count
    double accs[NACC];
    double re_f[F][NPLANE], im_f[F][NPLANE];
    double Ea[F], Eb[F];
    double cst[L], snt[L];  // cos and sin of 2 pi c / L
    uint32_t eqr[F][L * LP];
    int C[F][L * LP], D[F][L * LP], R[F][L * LP];
    int P[F][NPLANE][L];
    int part[F][NPLANE][GC][L];
};

// The measurement of slot A.slots[slot_index] by one wave, with its LDS at buf.
template <int L, int F>
__device__ __forceinline__ void measure_slot(const MeasureArgs &A, int slot_index, char *buf)
{
    constexpr int L2 = L * L, LP = L + 1;
    constexpr uint32_t mask = L == 32 ? 0xFFFFFFFFu : ((1u << L) - 1u);
    using M = MeasLds<L, F>;
    constexpr int G = M::G, GC = M::GC;
    M &S = *reinterpret_cast<M *>(buf);
    auto &accs = S.accs;
    const int gs = A.slots[slot_index];
    const int s = A.slot_sample[gs];
    const SampleDev d = A.samples[s];
    const int t = gs - d.slot_off;
    const int tid = threadIdx.x, T = blockDim.x;
    const int g = tid / G, lt = tid - g * G;  // frame group, lane within it
    int64_t nf;
    if (A.explicit_frames > 0) {
        nf = A.explicit_frames;
    } else {
        const int64_t n0 = A.state[0];
        nf = measurements_upto(n0 + A.K, A.measure_every, A.measure_start) -
             measurements_upto(n0, A.measure_every, A.measure_start);
    }
    if (nf <= 0) return;
    for (int i = tid; i < NACC; i += T) accs[i] = A.acc[(size_t)gs * NACC + i];
    for (int c = tid; c < L; c += T) {
        S.cst[c] = A.costab[(size_t)L * MAX_L + c];
        S.snt[c] = A.sintab[(size_t)L * MAX_L + c];
    }
    constexpr double Nd = (double)(L2 * L);
    for (int64_t f0 = 0; f0 < nf; f0 += F) {
        const int64_t f = f0 + g;
        const bool live = f < nf;  // the last batch may hold fewer than F frames
        uint32_t *eqr = S.eqr[g];
        int *C = S.C[g], *D = S.D[g], *R = S.R[g];
        double Ea = 0.0, Eb = 0.0;  // one frame per wave: the accumulating lane's own
        if (live) {
            const uint32_t *ra = A.frames + f * A.frame_words + d.frame_off + (size_t)t * L2;
            const uint32_t *rb = ra + (size_t)d.n_T * L2;
            if (lt == NPLANE) {  // the frame's two energies, loaded early (used by the accumulation)
                const double *E = A.frameE + f * 2 * A.total_slots + 2 * (size_t)d.slot_off;
                Ea = E[t];
                Eb = E[d.n_T + t];
                if constexpr (F > 1) {
                    S.Ea[g] = Ea;
                    S.Eb[g] = Eb;
                }
            }
            for (int i = lt; i < L2; i += G) {
                const uint32_t e = ~(ra[i] ^ rb[i]) & mask;
                const int y = i % L, z = i / L;
                eqr[y + LP * z] = e;
                R[y + LP * z] = __builtin_popcount(e);
            }
        }
        __syncthreads();
        if (live) column_counts<L, F == 1 ? 32 : L>(eqr, lt, C, D);  // C[x][y] at x*LP + y, D[x][z] at x*LP + z
        __syncthreads();
        // plane counts: lane (c, chunk) sums v = chunk, chunk + GC, ... of
        // every family (no divergence: the family loop is unrolled), then
        // (family, c) tasks add the GC chunk partials (integers: any order)
        if (live && lt < L * GC) {
            const int c = lt % L, chunk = lt / L;
#pragma unroll
            for (int fam = 0; fam < NPLANE; ++fam) {
                int cnt = 0;
                for (int v = chunk; v < L; v += GC) {
                    const int cm = c - v < 0 ? c - v + L : c - v;    // c - v mod L
                    const int cp = c + v >= L ? c + v - L : c + v;   // c + v mod L
                    const int vm = v - c < 0 ? v - c + L : v - c;    // v - c mod L
                    if (fam == 0) cnt += C[c * LP + v];        // x = c
                    else if (fam == 1) cnt += C[v * LP + c];   // y = c
                    else if (fam == 2) cnt += D[v * LP + c];   // z = c
                    else if (fam == 3) cnt += C[cm * LP + v];  // x + y = c
                    else if (fam == 4) cnt += C[cp * LP + v];  // x - y = c
                    else if (fam == 5) cnt += D[cm * LP + v];  // x + z = c
                    else if (fam == 6) cnt += D[cp * LP + v];  // x - z = c
                    else if (fam == 7) cnt += R[v + LP * cm];  // y + z = c
                    else cnt += R[v + LP * vm];                // y - z = c
                }
                S.part[g][fam][chunk][c] = cnt;
            }
        }
        __syncthreads();
        if (live) {
            for (int task = lt; task < NPLANE * L; task += G) {
                const int fam = task / L, c = task - fam * L;
                int cnt = 0;
                for (int k = 0; k < GC; ++k) cnt += S.part[g][fam][k][c];
                S.P[g][fam][c] = 2 * cnt - L2;
            }
        }
        __syncthreads();
        if (live && lt < NPLANE) {
            double re = 0.0, im = 0.0;
            for (int c = 0; c < L; ++c) {
                re += (double)S.P[g][lt][c] * S.cst[c];
                im += (double)S.P[g][lt][c] * S.snt[c];
            }
            S.re_f[g][lt] = re / Nd;
            S.im_f[g][lt] = im / Nd;
        }
        __syncthreads();
        // the batch's frames into the accumulators, in time order
        const int nb = F == 1 ? 1 : nf - f0 < F ? (int)(nf - f0) : F;
        if (tid < NPLANE) {
            for (int k = 0; k < nb; ++k) {
                const double re = S.re_f[k][tid], im = S.im_f[k][tid];
                accs[5 + 3 * tid] += re;
                accs[6 + 3 * tid] += im;
                accs[7 + 3 * tid] += re * re + im * im;
            }
        } else if (tid == NPLANE) {
            for (int k = 0; k < nb; ++k) {
                int S0 = 0;
                for (int c = 0; c < L; ++c) S0 += S.P[k][0][c];
                const double q0 = (double)S0 / Nd;
                accs[0] += 1.0;
                accs[1] += q0;
                accs[2] += q0 * q0;
                accs[3] += (q0 * q0) * q0;
                accs[4] += (q0 * q0) * (q0 * q0);
                const double ea = F == 1 ? Ea : S.Ea[k], eb = F == 1 ? Eb : S.Eb[k];
                accs[32] += ea;
                accs[33] += ea * ea;
                accs[34] += eb;
                accs[35] += eb * eb;
            }
        }
        __syncthreads();
    }
    for (int i = tid; i < NACC; i += T) A.acc[(size_t)gs * NACC + i] = accs[i];
}

template <int L>
__global__ void __launch_bounds__(64) measure_kernel(MeasureArgs A)
{
    __shared__ __attribute__((aligned(16))) char buf[sizeof(MeasLds<L, meas_frames<L>()>)];
    measure_slot<L, meas_frames<L>()>(A, blockIdx.x, buf);
}

#define EA_MEAS(Lv) template __global__ void measure_kernel<Lv>(MeasureArgs);
EA_MEAS(2)
EA_MEAS(4)
EA_MEAS(6)
EA_MEAS(8)
EA_MEAS(10)
EA_MEAS(12)
EA_MEAS(14)
EA_MEAS(16)
EA_MEAS(24)
EA_MEAS(32)
#undef EA_MEAS

// Neighbouring binary32 values (by bit pattern; -0 and +0 step to the
// smallest subnormals, infinities stay).
__device__ __forceinline__ float float_up(float v)
{
    if (v == __builtin_inff()) return v;
    if (v == 0.0f) return __uint_as_float(1u);
    const uint32_t b = __float_as_uint(v);
    return __uint_as_float(v > 0.0f ? b + 1u : b - 1u);
}
__device__ __forceinline__ float float_down(float v) { return -float_up(-v); }

// Exhaustive check of the acceptance gap used by the row, group and HBM
// engines, in binary64, with M = ACCEPT_MARGIN.  One thread per binary32 bit
// pattern v (NaNs excluded by the launch):
// (1) the hardware exponential is monotone: 2^v <= 2^(next binary32 above v);
// (2) for x = v: every exponent y the engines can form for x lies within a
//     relative 2^-21 of z = x log2(e) plus an absolute 2^-20 (the roundings of
//     both forms in update_word_gauss: at most about 5 2^-24 relative, plus
//     2 beta32 log2(e) 2^-19 2^-24 < 2^-20 from the field remainder's constant
//     of the folded form for beta32 <= 2^20); with yl, yh the binary32 values just
//     outside that interval and A = 2^y 2^32 at both ends (exact here),
//     T = exp_ea32(x) 2^32 (0 below -86):
//       x <= 0:  T - (M - 384) <= A(yl)  and  A(yh) <= T + (M - 128)
//       x > 0:   A(yl) >= 2^32 - M + 384   (dE < 0: the exact test accepts)
// Also records the largest |A / T - 1| at the two ends over [-86, 0].
__global__ void exp_bracket_kernel(uint32_t first_bits, uint32_t count, unsigned long long *violations,
                                   unsigned int *max_dev_bits)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float v = __uint_as_float(first_bits + i);
    bool ok = true;
    if (v != __builtin_inff() && !(__builtin_amdgcn_exp2f(v) <= __builtin_amdgcn_exp2f(float_up(v)))) ok = false;

    const double TWO32 = 4294967296.0, M = ACCEPT_MARGIN;
    const double z = (double)v * (double)__uint_as_float(0x3FB8AA3Bu);  // exact: 24 x 24 bits
    const double B = 0x1p-21, D = 0x1p-20;
    const double zl = (z <= 0.0 ? z * (1.0 + B) : z * (1.0 - B)) - D;
    const double zh = (z <= 0.0 ? z * (1.0 - B) : z * (1.0 + B)) + D;
    float yl = (float)zl, yh = (float)zh;
    if ((double)yl > zl) yl = float_down(yl);
    if ((double)yh < zh) yh = float_up(yh);
    const double Al = (double)__builtin_amdgcn_exp2f(yl) * TWO32;
    const double Ah = (double)__builtin_amdgcn_exp2f(yh) * TWO32;
    if (v > 0.0f) {
        ok = ok && Al >= TWO32 - M + 384.0;
    } else {
        const double T = v >= -86.0f ? (double)exp_ea32(v) * TWO32 : 0.0;
        ok = ok && Al >= T - (M - 384.0) && Ah <= T + (M - 128.0);
        if (v >= -86.0f) {
            const float dev = (float)(fmax(fabs(Al - T), fabs(Ah - T)) / T);
            atomicMax(max_dev_bits, __float_as_uint(dev));
        }
    }
    if (!ok) atomicAdd(violations, 1ull);
}

// The replica-exchange shortcut (exchange_accept in ea_device.hpp), one
// thread per binary32 bit pattern y from -0 down to -58: the hardware
// exponential lies within a relative 2^-22 of 2^y (binary64 exp2 as the
// reference) and exp_ea64(y) within 2^-49 of e^y (binary64 exp, itself within
// an ulp); records the largest |2^y (hardware) / 2^y - 1|.  With D = 1.5 y
// (down to -87, past the cut at -40) it also compares the decision itself
// with u < exp_ea64(D) for uniforms on the 2^-53 grid at distances k (2^-17
// exp_ea64(D) + 2^-24) (k = -6 .. 6) from exp_ea64(D), both sides of the
// margin, and for u = 0 and u = 1 - 2^-53, each with the random words' unused
// low bits clear and set; and that D = -1.5 y >= 0 accepts the same uniforms.
__global__ void exchange_bracket_kernel(uint32_t first_bits, uint32_t count, unsigned long long *violations,
                                        unsigned long long *max_dev_bits)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float y = __uint_as_float(first_bits + i);
    const double dev = fabs((double)__builtin_amdgcn_exp2f(y) / exp2((double)y) - 1.0);
    bool ok = dev <= 0x1p-22 && fabs(exp_ea64((double)y) / exp((double)y) - 1.0) <= 0x1p-49;
    if (y < 0.0f) {
        const double D = 1.5 * (double)y, E = exp_ea64(D);
        const auto decides = [&](double u) {
            const uint64_t n = (uint64_t)(u * 0x1p53);
            const uint32_t w0 = (uint32_t)(n >> 26) << 5, w1 = (uint32_t)(n & 0x3FFFFFFu) << 6;
            return exchange_accept(w0, w1, D) == (u < E) && exchange_accept(w0 | 31u, w1 | 63u, D) == (u < E) &&
                   exchange_accept(w0 | 31u, w1 | 63u, -D);
        };
        ok = ok && decides(0.0) && decides(1.0 - 0x1p-53);
        for (int k = -6; k <= 6; ++k)
            ok = ok && decides(fmax(0.0, fmin(floor((E + k * (E * 0x1p-17 + 0x1p-24)) * 0x1p53) * 0x1p-53,
                                              1.0 - 0x1p-53)));
    }
    atomicMax(max_dev_bits, (unsigned long long)__double_as_longlong(dev));
    if (!ok) atomicAdd(violations, 1ull);
}

__global__ void advance_kernel(int64_t *state, int64_t k)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) state[0] += k;
}

// ---------------------------------------------------------------------------
// From-scratch energies E_J (exact integer units) and magnetisations, one
// walker of a (sample, chain) per workgroup (blockIdx.y = walker); used to
// verify the incremental bookkeeping and to rebuild the state after
// ea_write_state.  (One workgroup for all walkers of a chain, in turn, took
// 262 us at 64 samples x 24 temperatures of L = 16, 3443 us at 128 x 32 of
// L = 32: too few workgroups, and a barrier per walker.  Now 24 and 367 us.)
template <int JK>
__global__ void __launch_bounds__(256) energy_kernel(const SampleDev *samples, const int32_t *items,
                                                    const int8_t *spins, const void *J, int64_t *EJ_out,
                                                    int32_t *M_out)
{
    __shared__ long long se[4];
    __shared__ int sm[4];
    const int code = items[blockIdx.x], w = blockIdx.y;
    const SampleDev d = samples[code >> 1];
    if (w >= d.n_T) return;
    const int r = code & 1;
    const int L = d.L, N = L * L * L, HALF = N / 2, HL = L / 2;
    const int tid = threadIdx.x;
    const int8_t *Sw = spins + d.spin_off + ((size_t)r * d.n_T + w) * N;
    const float *Jf = (const float *)J + d.J_off;
    const int8_t *Ji = (const int8_t *)J + d.J_off;
    long long e = 0;
    int m = 0;
    // sublattice index h of both parities: the bonds +x, +y, +z of either site
    // end at the other parity's sites of the same or the next row
    for (int h = tid; h < HALF; h += 256) {
        const int row = h / HL, j = h - row * HL, z = row / L, y = row - z * L;
        const int yn = y + 1 == L ? h - (L - 1) * HL : h + HL;
        const int zn = z + 1 == L ? h - (L - 1) * L * HL : h + L * HL;
        const int jn = j + 1 == HL ? h - (HL - 1) : h + 1;
        for (int p = 0; p < 2; ++p) {
            const int8_t *So = Sw + (1 - p) * HALF;
            const int si = Sw[p * HALF + h], xn = ((y + z + p) & 1) ? jn : h;
            const int nb[3] = {So[xn], So[yn], So[zn]};
            int c = 0;
            for (int dd = 0; dd < 3; ++dd) {
                const int i = (p * 3 + dd) * HALF + h;
                c += (JK == 0 ? (int)(Jf[i] * 262144.0f) : (int)Ji[i]) * nb[dd];  // |.| < 3 2^21
            }
            e -= (long long)(c * si);
            m += si;
        }
    }
    e = wave_sum_i64(e);
    m = wave_sum_i32(m);
    if ((tid & 63) == 0) {
        se[tid >> 6] = e;
        sm[tid >> 6] = m;
    }
    __syncthreads();
    if (tid == 0) {
        const size_t gi = 2 * (size_t)d.slot_off + (size_t)r * d.n_T + w;
        EJ_out[gi] = se[0] + se[1] + se[2] + se[3];
        M_out[gi] = sm[0] + sm[1] + sm[2] + sm[3];
    }
}

template __global__ void energy_kernel<0>(const SampleDev *, const int32_t *, const int8_t *, const void *,
                                          int64_t *, int32_t *);
template __global__ void energy_kernel<1>(const SampleDev *, const int32_t *, const int8_t *, const void *,
                                          int64_t *, int32_t *);

// The sublattice-split layout against the caller's natural order (i = x + L (y
// + L z), slot by slot).  Sites 2h and 2h + 1 share the sublattice index h: the
// even x of row (y, z) is of parity (y + z) & 1, the odd x of the other.
//
// One workgroup per (sample, chain, slot): row first + blockIdx.x of the
// [S][2][n_T] table, whose spins start base bytes into the caller's array;
// four sublattice indices (8 natural bytes) per thread step, a whole number of
// them for every even L.  On the host, one byte at a time, the two directions
// took more than 40 ms each for 12.6 MB; here a pass over the memory, 12 and 10
// us (2.1 and 2.5 TB/s).  Bound: HBM.
template <bool TO_NATURAL>
__global__ void __launch_bounds__(256) split_spins_kernel(const SampleDev *samples, const int32_t *slot_sample,
                                                         const int32_t *was, int64_t first, int64_t base,
                                                         int8_t *natural, int8_t *spins)
{
    const int64_t row = first + blockIdx.x;
    const SampleDev d = samples[slot_sample[row >> 1]];
    const int L = d.L, HL = L / 2, N = L * L * L, HALF = N / 2;
    const int k = (int)(row - 2 * (int64_t)d.slot_off), r = k >= d.n_T;
    uint2 *nat = (uint2 *)(natural + (d.spin_off + (int64_t)k * N - base));
    uint32_t *S0 = (uint32_t *)(spins + d.spin_off + ((int64_t)r * d.n_T + was[row]) * N), *S1 = S0 + HALF / 4;
    for (int i = threadIdx.x; i < HALF / 4; i += blockDim.x) {
        uint32_t odd = 0;  // 0xFF in the bytes of rows whose even x is of parity 1
        for (int b = 0; b < 4; ++b) {
            const int rr = (4 * i + b) / HL;
            odd |= ((rr + rr / L) & 1 ? 0xFFu : 0u) << (8 * b);  // L is even: rr = y modulo 2
        }
        if constexpr (TO_NATURAL) {
            const uint32_t a = S0[i], c = S1[i];
            const uint32_t ev = (a & ~odd) | (c & odd), od = (c & ~odd) | (a & odd);
            nat[i] = make_uint2(__builtin_amdgcn_perm(od, ev, 0x05010400u), __builtin_amdgcn_perm(od, ev, 0x07030602u));
        } else {
            const uint2 v = nat[i];
            const uint32_t ev = __builtin_amdgcn_perm(v.y, v.x, 0x06040200u);
            const uint32_t od = __builtin_amdgcn_perm(v.y, v.x, 0x07050301u);
            S0[i] = (ev & ~odd) | (od & odd);
            S1[i] = (od & ~odd) | (ev & odd);
        }
    }
}

template __global__ void split_spins_kernel<true>(const SampleDev *, const int32_t *, const int32_t *, int64_t, int64_t,
                                                  int8_t *, int8_t *);
template __global__ void split_spins_kernel<false>(const SampleDev *, const int32_t *, const int32_t *, int64_t,
                                                   int64_t, int8_t *, int8_t *);

// The same for couplings [3][N] (blockIdx.y = direction), samples first +
// blockIdx.x; Ju (may be NULL) receives them as multiples of 2^-18.
template <class T>
__global__ void __launch_bounds__(256) split_couplings_kernel(const SampleDev *samples, int first, int64_t base,
                                                             const T *natural, T *J, int32_t *Ju)
{
    const SampleDev d = samples[first + blockIdx.x];
    const int L = d.L, HL = L / 2, N = L * L * L, HALF = N / 2, dd = blockIdx.y;
    const T *nat = natural + (d.J_off - base) + (int64_t)dd * N;
    for (int h = threadIdx.x; h < HALF; h += blockDim.x) {
        const int rr = h / HL, p = (rr + rr / L) & 1;
        const int64_t even = d.J_off + (p * 3 + dd) * HALF + h, odd = d.J_off + ((1 - p) * 3 + dd) * HALF + h;
        J[even] = nat[2 * h];
        J[odd] = nat[2 * h + 1];
        if (Ju) {
            Ju[even] = (int32_t)((float)nat[2 * h] * 262144.0f);
            Ju[odd] = (int32_t)((float)nat[2 * h + 1] * 262144.0f);
        }
    }
}

template __global__ void split_couplings_kernel<float>(const SampleDev *, int, int64_t, const float *, float *,
                                                       int32_t *);
template __global__ void split_couplings_kernel<int8_t>(const SampleDev *, int, int64_t, const int8_t *, int8_t *,
                                                        int32_t *);

// Snapshot of the current state (slot order, bit rows) into frame 0, for an
// immediate measurement.  One workgroup per (sample, chain).
__global__ void __launch_bounds__(256) snapshot_kernel(const SampleDev *samples, const int32_t *items,
                                                      const int8_t *spins, const int32_t *was,
                                                      const int64_t *EJ, const int32_t *M, int jkind,
                                                      uint32_t *frame, double *frameE)
{
    const int code = items[blockIdx.x];
    const SampleDev d = samples[code >> 1];
    const int r = code & 1;
    const int L = d.L, L2 = L * L, N = L2 * L, HALF = N / 2;
    const size_t sbase = (size_t)d.spin_off + (size_t)r * d.n_T * N;
    const int gi = 2 * d.slot_off + r * d.n_T;
    uint32_t *dst = frame + d.frame_off + (size_t)r * d.n_T * L2;
    for (int i = threadIdx.x; i < d.n_T * L2; i += blockDim.x) {
        const int t = i / L2, row = i - t * L2;
        const int8_t *Sw = spins + sbase + (size_t)was[gi + t] * N;
        const int yz = (row % L) + row / L;
        uint32_t bits = 0;
        for (int x = 0; x < L; ++x) {
            const int p = (x + yz) & 1;
            bits |= (uint32_t)(Sw[p * HALF + ((x + L * row) >> 1)] < 0) << x;
        }
        dst[i] = bits;
    }
    const double unit = jkind == 0 ? 0x1p-18 : 1.0;
    for (int t = threadIdx.x; t < d.n_T; t += blockDim.x) {
        const int w = was[gi + t];
        frameE[gi + t] = (double)EJ[gi + w] * unit - (double)d.h32 * (double)M[gi + w];
    }
}

}  // namespace ea
