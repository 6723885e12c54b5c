// FP64 functions of the step kernels on the arguments a step has: the logarithm,
// sine and cosine of its 23-bit uniforms and the exponential of the hop
// probabilities.  The library's serve every argument (a Box-Muller pair takes
// 123 FP64 operations with them, here 50; a hop probability 38, here 26).
//
// Accuracy: no function may be further off than the library's.  Largest and
// root-mean-square relative errors in units of 1e-17, over every 23-bit uniform
// and x in +-50 for exp, library / here (tests/test_f64_functions.py holds them):
//   log   12.59, 4.75 / 11.14, 4.71    sine and cosine  14.84, 4.41 / 12.25, 4.28
//   exp   13.71, 4.91 / 11.50, 4.72    hop probability  28.86, 7.04 / 28.73, 6.97
// What takes them there: every sum that gives a result has its larger term exact
// (a product or table entry of few bits, the rest of it in the smaller term), so
// that the result is rounded about once, and the polynomials interpolate at the
// zeros of Chebyshev's polynomial of their interval.  With one rounded term each
// (Taylor series, 2 pi and the table entries rounded once), errors up to 2.7e-16, the
// steps were 2 to 3 % faster (8191 x 27, 1000 steps: 4.36 against 4.43 ms).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

namespace ssp {

// f in [1 + q/128, 1 + (q+1)/128): C = 1/f at the middle to 24 bits (exactly 1 and
// 1/2 at the two ends, so that the logarithm of a number just below 1 keeps its
// relative accuracy), c = 2^-31 C, hi + lo = -ln C [- ln 2 from f = sqrt 2 on], hi a
// multiple of 2^-42.
struct LogEntry {
    float c, lo;
    double hi;
};
struct Exp2Entry {
    double hi, lo;  // 2^(j/64)
};
struct alignas(16) F64Tables {
    LogEntry lg[128];
    Exp2Entry e2[64];
};
constexpr int kLogSqrt2 = 53;  // first interval taken as twice a number below 1

// (on the host, in extended precision; the kernels copy the tables to LDS)
inline void make_f64_tables(F64Tables& t)
{
    for (int q = 0; q < 128; ++q) {
        const float c = q == 0 ? 1.0f : (q == 127 ? 0.5f : (float)(1.0 / (1.0 + (q + 0.5) / 128.0)));
        const long double l = -logl((q >= kLogSqrt2 ? 2.0L : 1.0L) * (long double)c);
        const double hi = (double)(rintl(l * 0x1p42L) * 0x1p-42L);
        t.lg[q] = {c * 0x1p-31f, (float)(l - (long double)hi), hi};
    }
    for (int j = 0; j < 64; ++j) {
        const long double v = exp2l(j / 64.0L);
        const double hi = (double)v;
        t.e2[j] = {hi, (double)(v - (long double)hi)};
    }
}

// ln u for u = ((w >> 9) + 1/2) 2^-23 = m 2^-24: m = n 2^-z normalised to 32 bits,
// f = n 2^-31, r = C f - 1 (exact: 24 bits each; |r| <= 2^-8, in the first interval
// 0 <= r < 2^-7), and ln u = (E ln 2 + hi + r) + (lo + log1p(r) - r): the first sum is
// exact (multiples of 2^-47 below 2^5), the rest r^2 times a polynomial.
__host__ __device__ __forceinline__ double log_u01(const F64Tables& t, uint32_t w)
{
    const uint32_t m = (w >> 8) | 1u;
    const int z = __builtin_clz(m);
    const uint32_t n = m << z;
    const int q = (int)(n >> 24) - 128;
    const LogEntry g = t.lg[q];
    const double r = __builtin_fma((double)n, (double)g.c, -1.0);
    const double E = (double)(7 - z + (q >= kLogSqrt2 ? 1 : 0));
    double p = 1.0 / 7.0;
    p = __builtin_fma(p, r, -1.0 / 6.0);
    p = __builtin_fma(p, r, 1.0 / 5.0);
    p = __builtin_fma(p, r, -1.0 / 4.0);
    p = __builtin_fma(p, r, 1.0 / 3.0);
    p = __builtin_fma(p, r, -1.0 / 2.0);
    // ln 2 as 40 bits and the rest
    const double h = __builtin_fma(E, 0x1.62e42fefa2000p-1, g.hi) + r;
    const double l = __builtin_fma(E, 0x1.9ef35793c7673p-41, (double)g.lo);
    return h + __builtin_fma(p, r * r, l);
}

// cos and sin of 2 pi u: the nearest quarter turn is taken off in integers,
// leaving |x| <= 1/8 turn in multiples of 2^-24, so that t = x^2, x times 2 pi to
// 30 bits and 1 - 19.75 t are exact.
__host__ __device__ __forceinline__ void sincos_u01(uint32_t w, double& cs, double& sn)
{
    const int m = (int)((w >> 8) | 1u);
    const int k = (m + (1 << 21)) >> 22;
    const double x = (double)(m - (k << 22)) * 0x1p-24;
    const double t = x * x;
    double a = -0x1.6cc577dadd922p-1;
    a = __builtin_fma(a, t, 0x1.e8f036bcd3237p+1);
    a = __builtin_fma(a, t, -0x1.e3074d2614b2dp+3);
    a = __builtin_fma(a, t, 0x1.50783486facaap+5);
    a = __builtin_fma(a, t, -0x1.32d2cce62b872p+6);
    a = __builtin_fma(a, t, 0x1.466bc6775aae1p+6);
    a = __builtin_fma(a, t, -0x1.4abbce625be53p+5);
    a = __builtin_fma(a, t, 0x1.0b4611a626331p-32);  // 2 pi, beyond its leading part
    a = __builtin_fma(x, 0x1.921fb54400000p+2, x * a);
    double b = -0x1.b38340f56931fp+0;
    b = __builtin_fma(b, t, 0x1.f9cfc07738157p+2);
    b = __builtin_fma(b, t, -0x1.a6d1f0ab7905cp+4);
    b = __builtin_fma(b, t, 0x1.e1f50688302c5p+5);
    b = __builtin_fma(b, t, -0x1.55d3c7e3cbd74p+6);
    b = __builtin_fma(b, t, 0x1.03c1f081b5ac4p+6);
    b = __builtin_fma(b, t, 0x1.619b20dd10d2ep-7);  // 19.75 - 2 pi^2
    b = __builtin_fma(t, b, __builtin_fma(t, -19.75, 1.0));
    const double s0 = (k & 1) ? b : a, c0 = (k & 1) ? a : b;
    const uint64_t flip_s = (uint64_t)(uint32_t)(k & 2) << 62, flip_c = (uint64_t)(uint32_t)((k + 1) & 2) << 62;
    sn = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, s0) ^ flip_s);
    cs = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, c0) ^ flip_c);
}

// e^x = v 2^n, v in [0.99, 2], for |x| <= 700: x = (j/64 + n) ln 2 + r, |r| <= ln2/128.
__host__ __device__ __forceinline__ double exp_scaled(const F64Tables& t, double x, int& n)
{
    const double k = __builtin_rint(x * 0x1.71547652b82fep+6);
    double r = __builtin_fma(-k, 0x1.62e42fee00000p-7, x);
    r = __builtin_fma(-k, 0x1.a39ef35793c76p-39, r);
    const int N = (int)k;
    double p = 0x1.11111d8fbe766p-7;
    p = __builtin_fma(p, r, 0x1.55556b3304ec0p-5);
    p = __builtin_fma(p, r, 0x1.5555555555255p-3);
    p = __builtin_fma(p, r, 0x1.ffffffffff57fp-2);
    p = __builtin_fma(p * r, r, r);
    const Exp2Entry T = t.e2[N & 63];
    n = N >> 6;
    return T.hi + __builtin_fma(T.hi, p, T.lo);
}

}  // namespace ssp
