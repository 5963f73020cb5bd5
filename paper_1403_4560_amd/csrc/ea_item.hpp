// ea_item.hpp -- device helpers shared by the LDS-resident engines: block
// copies, wave and lane-group sums, the LDS frame of one (sample, chain) work
// item and the replica-exchange pass over it.
#pragma once

#include "ea_device.hpp"
#include "ea_types.hpp"

namespace ea {

// The threads that run one work item: the whole workgroup, or one of the
// equal, wave-aligned teams a batch workgroup is split into (each team with
// its own LDS region; every team passes the same barriers).  A ghost team
// computes like a real one on a copy of a real item but writes nothing to
// global memory (it fills a batch unit that has fewer items than teams).
struct Team {
    int T;       // threads in the team
    bool ghost;
    int wave;    // index within the team of this wave's first thread

    // This thread's index within the team, formed where it is called: what
    // follows from it is then not hoisted out of a sweep loop and kept across
    // it, in the end in scratch memory.  A kernel that uses any pays for it at
    // every launch and wave: one sweep a call at two chains a compute unit took
    // 40.2 us with 80 bytes and takes 32.7 without (L = 12 x 8 temperatures),
    // +-1 couplings at L = 10 x 56 60.8 and 54.1 (200 bytes).
    __device__ __forceinline__ int tid() const
    {
        int lane;
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
        return wave + lane;
    }
};

// Team index of a workgroup split into teams of T threads (whole waves).
__device__ __forceinline__ Team make_team(int team, int T, bool ghost)
{
    return Team{T, ghost, (__builtin_amdgcn_readfirstlane((int)threadIdx.x) & ~63) - team * T};
}

__device__ __forceinline__ Team whole_block()
{
    return Team{(int)blockDim.x, false, __builtin_amdgcn_readfirstlane((int)threadIdx.x) & ~63};
}

// Byte copy by T threads, 16 bytes at a time when both ends allow it; four
// copies in flight per thread.
__device__ __forceinline__ void block_copy(void *__restrict__ dst, const void *__restrict__ src, size_t bytes,
                                           int T, int tid)
{
    if ((((uintptr_t)dst | (uintptr_t)src | bytes) & 15) == 0) {
        int4 *__restrict__ d = (int4 *)dst;
        const int4 *__restrict__ s = (const int4 *)src;
        const size_t n = bytes / 16;
        size_t i = tid;
        for (; i + 3 * (size_t)T < n; i += 4 * (size_t)T) {
            const int4 a = s[i], b = s[i + T], c = s[i + 2 * T], e = s[i + 3 * T];
            d[i] = a;
            d[i + T] = b;
            d[i + 2 * T] = c;
            d[i + 3 * T] = e;
        }
        for (; i < n; i += T) d[i] = s[i];
    } else {
        int8_t *d = (int8_t *)dst;
        const int8_t *s = (const int8_t *)src;
        for (size_t i = tid; i < bytes; i += T) d[i] = s[i];
    }
}

// count walkers of bytes each (a multiple of 8) from consecutive blocks at
// glob to blocks lstride bytes apart at lds (to_lds), or back, in 8-byte words.
__device__ __forceinline__ void copy_walkers(int8_t *lds, size_t lstride, int8_t *glob, int count, size_t bytes,
                                             bool to_lds, uint32_t T, uint32_t tid)
{
    const uint32_t per = (uint32_t)bytes / 8, total = per * (uint32_t)count;
    for (uint32_t i = tid; i < total; i += T) {
        const uint32_t w = i / per, j = i - w * per;
        uint2 *l = (uint2 *)(lds + w * lstride) + j;
        uint2 *g = (uint2 *)(glob + w * bytes) + j;
        if (to_lds) *l = *g;
        else *g = *l;
    }
}

// Pointers into the dynamic LDS of one work item.
struct ItemLds {
    int8_t *S;
    void *J;
    int32_t *was, *sow, *M, *dM, *fl, *sw;
    long long *EJ, *dEJ;
    uint32_t *lut;
    float *b32;
    double *b64;
    uint4 *ph;  // row engine: the site groups' Philox words (philox_group)
};

// The descriptor of a workgroup's sample, read into scalar registers: the
// item code is the same for every lane, and descriptors are read-only during a
// launch, so the read may go through the scalar cache.
__device__ __forceinline__ SampleDev sample_of_item(const SampleDev *samples, int idx)
{
    typedef const __attribute__((address_space(4))) uint32_t *ConstWords;
    static_assert(sizeof(SampleDev) % 4 == 0, "descriptor is read in 32-bit words");
    const ConstWords src = (ConstWords)(samples + __builtin_amdgcn_readfirstlane(idx));
    uint32_t w[sizeof(SampleDev) / 4];
#pragma unroll
    for (int k = 0; k < (int)(sizeof(SampleDev) / 4); ++k) w[k] = src[k];
    SampleDev d;
    __builtin_memcpy(&d, w, sizeof d);
    return d;
}

__device__ __forceinline__ ItemLds item_lds(char *smem, int L, int nT, int jkind)
{
    const LdsOff o = lds_offsets(L, nT, jkind);
    ItemLds p;
    p.S = (int8_t *)(smem + o.spins);
    p.J = (void *)(smem + o.J);
    p.was = (int32_t *)(smem + o.was);
    p.sow = (int32_t *)(smem + o.sow);
    p.M = (int32_t *)(smem + o.M);
    p.dM = (int32_t *)(smem + o.dM);
    p.fl = (int32_t *)(smem + o.fl);
    p.sw = (int32_t *)(smem + o.sw);
    p.EJ = (long long *)(smem + o.EJ);
    p.dEJ = (long long *)(smem + o.dEJ);
    p.lut = (uint32_t *)(smem + o.lut);
    p.b32 = (float *)(smem + o.b32);
    p.b64 = (double *)(smem + o.b64);
    p.ph = (uint4 *)(smem + o.ph);
    return p;
}

// v of the lane K places along in the same row of 16 lanes (rotation).
template <int K>
__device__ __forceinline__ int row_rotate(int v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x120 + K, 0xF, 0xF, true);
}

template <int K>
__device__ __forceinline__ long long row_rotate(long long v)
{
    // (the halves as a register pair: assembled with shifts and ors, the
    // compiler adds the halves into a sum one at a time)
    typedef int int2v __attribute__((ext_vector_type(2)));
    int2v h = __builtin_bit_cast(int2v, v);
    h.x = row_rotate<K>(h.x);
    h.y = row_rotate<K>(h.y);
    return __builtin_bit_cast(long long, h);
}

// v of lane (this lane XOR K) within its aligned group of four (K = 1 or 2).
template <int K>
__device__ __forceinline__ int quad_xor(int v)
{
    static_assert(K == 1 || K == 2, "quad permutation");
    return __builtin_amdgcn_mov_dpp(v, K == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true);
}

template <int K>
__device__ __forceinline__ long long quad_xor(long long v)
{
    typedef int int2v __attribute__((ext_vector_type(2)));
    int2v h = __builtin_bit_cast(int2v, v);
    h.x = quad_xor<K>(h.x);
    h.y = quad_xor<K>(h.y);
    return __builtin_bit_cast(long long, h);
}

// Sum over aligned groups of W = 4 or 16 consecutive lanes, every lane of the
// group active (DPP: permutations within four lanes, rotations within a row).
template <int W, class V>
__device__ __forceinline__ V group_sum_dpp(V v)
{
    static_assert(W == 4 || W == 16, "group of four lanes or a row");
    if constexpr (W == 4) {
        v += quad_xor<1>(v);
        v += quad_xor<2>(v);
    } else {
        v += row_rotate<8>(v);
        v += row_rotate<4>(v);
        v += row_rotate<2>(v);
        v += row_rotate<1>(v);
    }
    return v;
}

// Sums over a wave, every lane of it active: within the rows by rotations, then
// one lane of each row by scalar adds (a shuffle through LDS for each of the
// six steps took about a third of the HBM tier's end of sweep).
__device__ __forceinline__ int wave_sum_i32(int v)
{
    v = group_sum_dpp<16>(v);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
           __builtin_amdgcn_readlane(v, 48);
}

__device__ __forceinline__ long long wave_sum_i64(long long v)
{
    v = group_sum_dpp<16>(v);
    const auto row = [&](int lane) {
        const uint32_t lo = __builtin_amdgcn_readlane((int)(unsigned long long)v, lane);
        const uint32_t hi = __builtin_amdgcn_readlane((int)((unsigned long long)v >> 32), lane);
        return (long long)((unsigned long long)hi << 32 | lo);
    };
    return row(0) + row(16) + row(32) + row(48);
}

// Sum of v over the lanes of this lane's row of 16 whose index agrees with
// this lane's modulo S (S = 1, 2, 4, 8 or 16, uniform): rotations by S, 2S,
// .., 8.  Every lane of the wave must be active.
template <class V>
__device__ __forceinline__ V row_residue_sum(V v, int S)
{
    if (S <= 1) v += row_rotate<1>(v);
    if (S <= 2) v += row_rotate<2>(v);
    if (S <= 4) v += row_rotate<4>(v);
    if (S <= 8) v += row_rotate<8>(v);
    return v;
}

// v of the other lane of a pair of neighbouring lanes: (0, 1), (2, 3), .. or,
// with odd set, (1, 2), (3, 4), ..
__device__ __forceinline__ int pair_other(int v, int lane, bool odd)
{
    const int a = quad_xor<1>(v);
    const int l = __builtin_amdgcn_mov_dpp(v, 0x130, 0xF, 0xF, true);  // of lane + 1
    const int r = __builtin_amdgcn_mov_dpp(v, 0x138, 0xF, 0xF, true);  // of lane - 1
    return !odd ? a : (lane & 1) ? l : r;
}

// Replica exchange of neighbouring slots (t, t+1), t = n&1, n&1 + 2, ..., after
// sweep n (Methods: parallel tempering; even-odd pairs alternate with the sweep
// parity).  D = (beta_t - beta_{t+1}) (E_t - E_{t+1}) in binary64, E_w =
// energy(w); accepted iff D >= 0 or u53 < exp_ea64(D) (decided by
// exchange_accept), u53 from the exchange counter (0, n, (1 << 28) | (t << 1)
// | r, sample).  Swaps walker labels only, in both maps (was: slot -> walker,
// sow: walker -> slot), so the sweep that follows reads its temperatures
// without rebuilding sow.
//
// By one whole wave, lane t for slot t: both lanes of a pair form its decision
// from the same operands, and the slots' walkers and energies cross between
// the lanes in registers.  A lone wave's chain that the others wait for, so it
// has no branch before the decision (lanes without a slot or a pair read those
// at hand) and the random words, with the round keys that the caller holds in
// vector registers (VKEYS), run while the loads are on the way: 1600 cycles of a
// sweep before; us a sweep, before and now: L = 6 x 16 temperatures 4.12 and 3.97,
// L = 8 x 16 4.08 and 3.87, L = 10 x 16 5.67 and 5.47 (few chains), +-1 L = 8 x 56
// 5.66 and 5.53.  Not for the one-bit engine at L = 32, whose words take 2 % longer
// with the keys live here (113.6 and 116.1).  Nothing is kept between sweeps: held
// in registers, it would be spilled.  Returns the walker now at slot t (t itself
// from n_T on).
template <bool VKEYS = true, class Energy>
__device__ __forceinline__ int exchange_slots(const SweepArgs &A, const SampleDev &d, int r, int64_t n, const ItemLds &I,
                                              int t, const RoundKeys &key, Energy energy)
{
    const int nT = d.n_T;
    const bool odd = n & 1;
    const int lo = odd ? (t - 1) | 1 : t & ~1;  // the pair's lower slot
    const bool pair = lo >= 0 && lo + 1 < nT;
    const int lc = pair ? lo : 0;
    int w = I.was[min(t, nT - 1)];
    const double b0 = I.b64[lc], b1 = I.b64[min(lc + 1, nT - 1)];
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t c2 = (PURPOSE_EXCHANGE << 28) | ((uint32_t)lo << 1) | (uint32_t)r;
    u32x4 q;
    double E;
    if constexpr (VKEYS) {
        PhiloxSlot ps;
        ps.init((uint32_t)n, c2, A.key0, A.key1);
        q = ps.start(philox_group(0u, d.sample_id, A.key1));
#pragma unroll
        for (int k = 0; k < 3; ++k) q = philox_round(q, key.a[k], key.b[k]);
        __builtin_amdgcn_sched_barrier(0);
        E = energy(w);
#pragma unroll
        for (int k = 3; k < 8; ++k) q = philox_round(q, key.a[k], key.b[k]);
    } else {
        E = energy(w);
        q = philox4x32_10(0u, (uint32_t)n, c2, d.sample_id, A.key0, A.key1);
    }
    typedef int int2v __attribute__((ext_vector_type(2)));
    int2v e = __builtin_bit_cast(int2v, E);
    e.x = pair_other(e.x, t, odd);
    e.y = pair_other(e.y, t, odd);
    const double Eo = __builtin_bit_cast(double, e);
    const int wo = pair_other(w, t, odd);
    const double D = (b0 - b1) * (t == lo ? E - Eo : Eo - E);
    if (pair && exchange_accept(q.x, q.y, D)) {
        w = wo;
        if (t == lo) atomicAdd(&I.sw[t], 1);
        I.was[t] = w;
        I.sow[w] = t;
    }
    return t < nT ? w : t;
}

}  // namespace ea
