// ea_finalize.hip -- disorder averages and jackknife errors of the observables
// of eqs. 3-6 on the device, from the per-slot accumulators of the selected
// samples of one system, with exact sums over samples (ea_exact.hpp).
#include "ea_exact.hpp"
#include "ea_types.hpp"

namespace ea {

// Observables of eqs. 3-6 from disorder-averaged thermal means D[36] (column
// order of the accumulators), each formula evaluated in the order written,
// one rounding per binary64 operation.  two_sin = 2 sin(pi/L) (host libm).
__device__ __forceinline__ void observables_of(const double *D, int L, double two_sin, double *o)
{
    const double N = (double)L * L * L;
    const double q1 = D[1], q2 = D[2], q3 = D[3], q4 = D[4], Q = q1;
    const double c2 = q2 - 2.0 * Q * q1 + Q * Q;
    const double c4 = q4 - 4.0 * Q * q3 + 6.0 * Q * Q * q2 - 4.0 * Q * Q * Q * q1 + Q * Q * Q * Q;
    double chi[NPLANE];
    for (int f = 0; f < NPLANE; ++f) {
        const double re = D[5 + 3 * f], im = D[6 + 3 * f];
        chi[f] = N * (D[7 + 3 * f] - (re * re + im * im));
    }
    const double chi0 = N * (q2 - q1 * q1);
    const double chik = (chi[0] + chi[1] + chi[2]) / 3.0;
    const double chik2 = (chi[3] + chi[4] + chi[5] + chi[6] + chi[7] + chi[8]) / 6.0;
    o[0] = q1;
    o[1] = chi0;
    o[2] = chik;
    o[3] = chik2;
    o[4] = 0.5 * (3.0 - c4 / (c2 * c2));
    o[5] = sqrt(chi0 / chik - 1.0) / two_sin;
    o[6] = chik / chik2;
    o[7] = chi0 / chik;
    o[8] = D[32];
    o[9] = D[34];
}

constexpr int NOBS_VAL = 10;  // observables per slot (the count column aside)

// Disorder averages (eqs. 3-6) and leave-one-sample-out jackknife errors
// (Methods, last paragraph) per temperature slot over S selected samples of
// one system, in three launches; off[i] is sample i's first slot (NULL: every
// sample of an ensemble of one system, off[i] = i nT).
//  1. finalize_sums_kernel, column j of slot t: exact sum over samples of the
//     thermal mean acc[j] / acc[0], its digits kept in cols[t][j] with the
//     column's window; D[j] = (rounded sum) / S.
//  2. finalize_values_kernel: the observables of D (the central values), and
//     for replicate s D_s[j] = (rounded exact sum less sample s's value) /
//     (S - 1) and its observables O_s, kept in rep[t][k][s] (10 nT S doubles).
//  3. finalize_errors_kernel, observable k of slot t: exact sums over s of
//     O_s give the replicate mean Obar = (rounded sum) / S, then exact sums of
//     (O_s - Obar)^2 give err = sqrt((S-1)/S * rounded sum).
// Bound: latency (dependent binary64 divisions, LDS chains); the accumulators
// are read twice (14 MB at 2048 samples x 24 slots, 3 us of HBM time).  One
// workgroup a slot, its columns summed serially by 36 lanes into limb arrays
// in scratch memory, had left most of the chip idle: 7492 us at 2048 samples x
// 24 slots, 493 us at 64 x 56.  Split by column, by (sample, column) and by
// observable, with only a sum's window of limbs carried and rounded: 29 + 34 +
// 22 us and 9 + 16 + 17 us.
__device__ __forceinline__ size_t slot_of(const int32_t *off, int i, int nT, int t)
{
    return (size_t)(off ? off[i] : i * nT) + t;
}

// Lowest and highest limb of a set of values over a workgroup (LDS, start
// values XL and -1) and the counts of its non-finite ones.
struct Window {
    int imin, imax, spec[3];
};

__device__ __forceinline__ void window_clear(Window &w)
{
    w.imin = XL;
    w.imax = -1;
    w.spec[0] = w.spec[1] = w.spec[2] = 0;
}

// Notes x; true if it is finite and not zero (it then has digits to add).
__device__ __forceinline__ bool window_note(double x, int &imin, int &imax, Window &w)
{
    const int c = exact_class(x);
    if (c >= 0) {
        atomicAdd(&w.spec[c], 1);
        return false;
    }
    const int i = exact_limb(x);
    if (i < 0) return false;
    imin = min(imin, i);
    imax = max(imax, i);
    return true;
}

__device__ __forceinline__ void window_join(Window &w, int imin, int imax)
{
    if (imax < 0) return;
    atomicMin(&w.imin, imin);
    atomicMax(&w.imax, imax);
}

// Digits lo .. hi of a set's sum (zeros when it holds no nonzero value).
__device__ __forceinline__ void window_range(const Window &w, int &lo, int &hi)
{
    lo = w.imax < 0 ? 0 : w.imin;
    hi = w.imax < 0 ? XWIN : w.imax + XWIN;
}

// One workgroup takes FIN_SUM_COLS neighbouring columns of a slot.  A wave's lanes
// hold 16 samples of each column, and each of them adds into a copy of the
// limbs of its own, because the values of one column fall on the same limbs.
constexpr int SUM_COPIES = 16;

__global__ void __launch_bounds__(256) finalize_sums_kernel(const int32_t *off, int S, int nT, const double *acc,
                                                            FinColumn *cols)
{
    static_assert(NACC % FIN_SUM_COLS == 0, "whole column groups");
    __shared__ unsigned long long lim[FIN_SUM_COLS][XL][SUM_COPIES];
    __shared__ long long sum[FIN_SUM_COLS][XL];
    __shared__ Window win[FIN_SUM_COLS];
    const int t = blockIdx.y, tid = threadIdx.x;
    const int c = tid % FIN_SUM_COLS, j = blockIdx.x * FIN_SUM_COLS + c;
    const int first = tid / FIN_SUM_COLS, step = 256 / FIN_SUM_COLS, copy = first % SUM_COPIES;
    if (tid < FIN_SUM_COLS) window_clear(win[tid]);
    for (int i = tid; i < FIN_SUM_COLS * XL * SUM_COPIES; i += 256) (&lim[0][0][0])[i] = 0ull;
    __syncthreads();
    int imin = XL, imax = -1;
    for (int i = first; i < S; i += step) {
        const double *a = acc + slot_of(off, i, nT, t) * NACC;
        const double m = a[j] / a[0];
        if (window_note(m, imin, imax, win[c])) exact_add_atomic(&lim[c][0][copy], m, SUM_COPIES);
    }
    window_join(win[c], imin, imax);
    __syncthreads();
    for (int k = 0; k < FIN_SUM_COLS; ++k) {
        int lo, hi;
        window_range(win[k], lo, hi);
        for (int i = tid / SUM_COPIES; i <= hi - lo; i += 256 / SUM_COPIES) {
            long long v = (long long)lim[k][lo + i][tid % SUM_COPIES];
            for (int m = SUM_COPIES / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m);
            if (tid % SUM_COPIES == 0) sum[k][lo + i] = v;
        }
    }
    __syncthreads();
    if (tid < FIN_SUM_COLS) {
        FinColumn &o = cols[(size_t)t * NACC + j];
        const Window &w = win[c];
        int lo, hi;
        window_range(w, lo, hi);
        exact_carry(sum[c], o.dig, lo, hi);
        o.lo = lo;
        o.hi = hi;
        for (int k = 0; k < 3; ++k) o.spec[k] = w.spec[k];
        double v;
        if (!exact_special(w.spec[0], w.spec[1], w.spec[2], &v)) v = exact_round_less(o.dig, lo, hi, 0.0);
        o.D = v / (double)S;
    }
}

// One workgroup takes FIN_VAL_TILE samples of a slot: first every (sample, column)
// pair of the tile over all threads, then one thread a sample for the
// observables.  S = 0: central values only.
__global__ void __launch_bounds__(256) finalize_values_kernel(const int32_t *off, int S, int count, int nT, int L,
                                                              double two_sin, const double *acc,
                                                              const FinColumn *cols, double *rep, double *mean_out)
{
    __shared__ uint32_t dig[NACC][XL];
    __shared__ int32_t lo[NACC], hi[NACC], spec[NACC][3];
    __shared__ double Ds[FIN_VAL_TILE][NACC + 1];
    const int t = blockIdx.y, tid = threadIdx.x;
    const int s0 = blockIdx.x * FIN_VAL_TILE, n = min(FIN_VAL_TILE, S - s0);
    const FinColumn *col = cols + (size_t)t * NACC;
    if (n > 0) {
        if (tid < NACC) {
            lo[tid] = col[tid].lo;
            hi[tid] = col[tid].hi;
            for (int k = 0; k < 3; ++k) spec[tid][k] = col[tid].spec[k];
        }
        for (int i = tid; i < NACC * XL; i += 256) {
            const int j = i / XL, k = i - j * XL;
            if (k >= col[j].lo && k <= col[j].hi) dig[j][k] = col[j].dig[k];
        }
        __syncthreads();
        for (int i = tid; i < n * NACC; i += 256) {
            const int s = i / NACC, j = i - s * NACC;
            const double *a = acc + slot_of(off, s0 + s, nT, t) * NACC;
            const double m = a[j] / a[0];
            const int c = exact_class(m);
            double v;
            if (!exact_special(spec[j][0] - (c == 0), spec[j][1] - (c == 1), spec[j][2] - (c == 2), &v))
                v = exact_round_less(dig[j], lo[j], hi[j], c < 0 ? m : 0.0);
            Ds[s][j] = v / (double)(S - 1);
        }
        __syncthreads();
        if (tid < n) {
            double o[NOBS_VAL];
            observables_of(Ds[tid], L, two_sin, o);
            for (int k = 0; k < NOBS_VAL; ++k) rep[((size_t)t * NOBS_VAL + k) * S + s0 + tid] = o[k];
        }
    }
    if (blockIdx.x == 0 && tid == 64) {
        double D[NACC], o[NOBS_VAL];
        for (int j = 0; j < NACC; ++j) D[j] = col[j].D;
        observables_of(D, L, two_sin, o);
        for (int k = 0; k < NOBS_VAL; ++k) mean_out[(size_t)t * (NOBS_VAL + 1) + k] = o[k];
        mean_out[(size_t)t * (NOBS_VAL + 1) + NOBS_VAL] = (double)count;
    }
}

// One workgroup takes one observable of a slot; each lane adds into a copy of
// the limbs of its own.
__global__ void __launch_bounds__(256) finalize_errors_kernel(int S, const double *rep, double *err_out)
{
    __shared__ unsigned long long lim[XL][64];
    __shared__ long long sum[XL];
    __shared__ uint32_t dig[XL];
    __shared__ Window win;
    __shared__ double obar;
    const int k = blockIdx.x, t = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const double *o = rep + ((size_t)t * NOBS_VAL + k) * S;
    for (int pass = 0; pass < 2; ++pass) {
        const double ob = pass ? obar : 0.0;
        if (tid == 0) window_clear(win);
        for (int i = tid; i < XL * 64; i += 256) (&lim[0][0])[i] = 0ull;
        __syncthreads();
        int imin = XL, imax = -1, lo, hi;
        for (int i = tid; i < S; i += 256) {
            const double dv = o[i] - ob, x = pass ? dv * dv : o[i];
            if (window_note(x, imin, imax, win)) exact_add_atomic(&lim[0][lane], x, 64);
        }
        window_join(win, imin, imax);
        __syncthreads();
        window_range(win, lo, hi);
        for (int i = lo + (tid >> 6); i <= hi; i += 4) {
            long long v = (long long)lim[i][lane];
            for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
            if (lane == 0) sum[i] = v;
        }
        __syncthreads();
        if (tid == 0) {
            double v;
            exact_carry(sum, dig, lo, hi);
            if (!exact_special(win.spec[0], win.spec[1], win.spec[2], &v)) v = exact_round_less(dig, lo, hi, 0.0);
            if (pass == 0) obar = v / (double)S;
            else err_out[(size_t)t * (NOBS_VAL + 1) + k] = sqrt((double)(S - 1) / (double)S * v);
            if (pass == 1 && k == 0) err_out[(size_t)t * (NOBS_VAL + 1) + NOBS_VAL] = 0.0;
        }
        __syncthreads();
    }
}

}  // namespace ea
