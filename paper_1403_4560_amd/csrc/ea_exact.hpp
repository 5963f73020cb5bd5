// ea_exact.hpp -- exact sums of binary64 values, rounded once.
//
// The disorder average of eqs. 3-6 (the overline: an average over the
// realizations of one model at one field and one temperature ladder) is taken
// as the exact sum of the per-sample thermal means rounded once to binary64
// (nearest, ties to even) and then divided by the sample count; a
// leave-one-sample-out replicate of the jackknife (Methods, last paragraph) is
// the exact sum of the other samples' values, rounded once, divided by the
// count less one.  No result then depends on the order in which threads or
// atomics visit the samples.
//
// Representation.  Every finite binary64 is an integer multiple of 2^-1074.
// An exact sum is XL signed 64-bit limbs, limb k weighing 2^(32k) such units.
// A value adds its 53-bit significand, cut into three 32-bit digits, to three
// consecutive limbs, so each limb grows by less than 2^32 per value: fewer
// than 2^30 values can never overflow a limb, and the additions commute (plain
// integer adds, or integer atomics in LDS).  Carrying the limbs that a set of
// values touches (a few of the XL, as values of one kind span a few binades)
// leaves a two's complement number of 32-bit digits.  Non-finite
// values are counted apart (NaN, +inf, -inf) and decide the result as IEEE
// addition would: any NaN, or +inf together with -inf, gives NaN; otherwise an
// infinity wins.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ea_types.hpp"

namespace ea {

struct ExactDigits {
    int i;               // lowest limb touched
    int64_t d0, d1, d2;  // signed digits for limbs i, i+1, i+2
};

// The three digits of a finite x (negated when neg).  x = 0 gives zeros.
__device__ __forceinline__ ExactDigits exact_digits(double x, bool neg)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const int be = (int)((b >> 52) & 0x7ff);
    const uint64_t frac = b & ((1ull << 52) - 1);
    const uint64_t m = be ? (frac | (1ull << 52)) : frac;  // x = m 2^(o - 1074)
    const int o = be ? be - 1 : 0;
    const int sh = o & 31;
    const uint64_t lo = m << sh;                       // bits 0..63 of m 2^sh
    const uint64_t hi = sh ? (m >> (64 - sh)) : 0ull;  // bits 64..84
    ExactDigits r;
    r.i = o >> 5;
    r.d0 = (int64_t)(lo & 0xffffffffull);
    r.d1 = (int64_t)(lo >> 32);
    r.d2 = (int64_t)hi;
    if (neg != ((b >> 63) != 0)) {
        r.d0 = -r.d0;
        r.d1 = -r.d1;
        r.d2 = -r.d2;
    }
    return r;
}

// The lowest limb a finite x touches, or -1 for a zero (which touches none).
__device__ __forceinline__ int exact_limb(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const int be = (int)((b >> 52) & 0x7ff);
    if ((b << 1) == 0) return -1;
    return (be ? be - 1 : 0) >> 5;
}

// lim[k stride] += digit k of x, on limbs shared by a workgroup (LDS), by
// integer atomics.
__device__ __forceinline__ void exact_add_atomic(unsigned long long *lim, double x, int stride)
{
    const ExactDigits g = exact_digits(x, false);
    lim += g.i * stride;
    atomicAdd(lim, (unsigned long long)g.d0);
    atomicAdd(lim + stride, (unsigned long long)g.d1);
    atomicAdd(lim + 2 * stride, (unsigned long long)g.d2);
}

// A sum's window: values whose lowest limbs lie in [imin, imax] have a sum
// that is a two's complement number of the digits imin .. imax + 3 (fewer than
// 2^30 values of magnitude below 2^(32 (imax + 3)); digit imax + 3 is the
// signed top).
constexpr int XWIN = 3;

// Carry limbs lo .. hi (already summed over their copies) into digits, the top
// one in two's complement.
__device__ __forceinline__ void exact_carry(const long long *lim, uint32_t *dig, int lo, int hi)
{
    int64_t carry = 0;
    for (int k = lo; k <= hi; ++k) {
        const int64_t v = lim[k] + carry;
        dig[k] = (uint32_t)v;
        carry = v >> 32;  // arithmetic shift: floor division by 2^32
    }
}

// The leading digits of a magnitude whose digits arrive from the lowest up:
// the highest nonzero digit, the two below it, and whether any lower bit is set.
struct LeadingDigits {
    uint32_t w0 = 0, w1 = 0, w2 = 0, p1 = 0, p2 = 0;
    bool sticky = false, low = false;
    int top = -1;

    __device__ __forceinline__ void push(uint32_t v, int k)
    {
        const bool nz = v != 0;
        w0 = nz ? v : w0;
        w1 = nz ? p1 : w1;
        w2 = nz ? p2 : w2;
        sticky = nz ? low : sticky;
        top = nz ? k : top;
        low |= p2 != 0;
        p2 = p1;
        p1 = v;
    }

    // The magnitude rounded once to binary64 (nearest, ties to even).
    __device__ __forceinline__ double round() const
    {
        if (top < 0) return 0.0;
        const uint64_t hi = (uint64_t)w0 << 32 | w1;
        const int lz = __builtin_clz(w0);
        const int b = 32 * top + 32 - lz;  // bit length
        if (b <= 53)  // exact: subnormal, or normal with at most 53 bits
            return ldexp((double)(top >= 1 ? hi : (uint64_t)w0), -1074);
        // T: the 64 bits from the leading one down; the rest decides ties
        const uint64_t T = lz ? hi << lz | w2 >> (32 - lz) : hi;
        const bool more = sticky || (uint32_t)(w2 << lz) != 0;
        uint64_t mant = T >> 11;
        const uint64_t rest = T & 0x7ff;
        if ((rest & 0x400) && ((rest & 0x3ff) || more || (mant & 1))) ++mant;
        int e = b - 53;
        if (mant == (1ull << 53)) {
            mant >>= 1;
            ++e;
        }
        return ldexp((double)mant, e - 1074);  // exact, or overflow to infinity
    }
};

// The sum held by digits lo .. hi less x (finite; 0 takes nothing away),
// rounded once to binary64 (an exact zero is +0).  The digits are read twice,
// for the sign of the difference and then for its magnitude, so that no digit
// array is kept in registers.
__device__ __forceinline__ double exact_round_less(const uint32_t *dig, int lo, int hi, double x)
{
    const ExactDigits g = exact_digits(x, true);
    const auto digit = [&](int k) {
        const int64_t t = k == hi ? (int64_t)(int32_t)dig[k] : (int64_t)dig[k];
        const int j = k - g.i;
        return t + (j == 0 ? g.d0 : j == 1 ? g.d1 : j == 2 ? g.d2 : 0);
    };
    int64_t c = 0;
    for (int k = lo; k <= hi; ++k) c = (digit(k) + c) >> (k == hi ? 63 : 32);
    const bool neg = c < 0;
    LeadingDigits m;
    c = 0;
    for (int k = lo; k <= hi; ++k) {
        const int64_t d = digit(k), v = (neg ? -d : d) + c;
        m.push((uint32_t)v, k);
        c = v >> 32;
    }
    const double r = m.round();
    return neg ? -r : r;
}

// Result of a sum with non-finite terms (counts n_nan, n_pinf, n_ninf), or
// false when every term is finite.
__device__ __forceinline__ bool exact_special(int n_nan, int n_pinf, int n_ninf, double *out)
{
    if (n_nan || (n_pinf && n_ninf)) {
        *out = __longlong_as_double(0x7ff8000000000000ll);
        return true;
    }
    if (n_pinf) {
        *out = __longlong_as_double(0x7ff0000000000000ll);
        return true;
    }
    if (n_ninf) {
        *out = __longlong_as_double((long long)0xfff0000000000000ull);
        return true;
    }
    return false;
}

// Special-value class of x: 0 NaN, 1 +inf, 2 -inf, -1 finite.
__device__ __forceinline__ int exact_class(double x)
{
    if (x != x) return 0;
    if (x == __longlong_as_double(0x7ff0000000000000ll)) return 1;
    if (x == __longlong_as_double((long long)0xfff0000000000000ull)) return 2;
    return -1;
}

}  // namespace ea
