// FP64 functions of the step kernels on the arguments a step has: the logarithm,
// sine and cosine of its 23-bit uniforms and the exponential of the hop
// probabilities.  The library's serve every argument (a Box-Muller pair takes
// 123 FP64 operations with them, here 48; a hop probability 38, here 26).
//
// Accuracy: no function may be further off than the library's.  Largest and
// root-mean-square relative errors in units of 1e-17, over every 23-bit uniform
// and x in +-50 for exp, library / here (tests/test_f64_functions.py holds them):
//   log   12.59, 4.75 / 12.03, 4.71    sine and cosine  14.84, 4.41 / 12.25, 4.28
//   exp   13.71, 4.91 / 11.50, 4.72    hop probability  28.86, 7.04 / 28.73, 6.97
// What takes them there: every sum that gives a result has its larger term exact
// (a product or table entry of few bits, the rest of it in the smaller term), so
// that the result is rounded about once, and the polynomials interpolate at the
// zeros of Chebyshev's polynomial of their interval.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

namespace ssp {

// f in [1 + q/128, 1 + (q+1)/128): c = 2^-31 C, minus_ln = -ln C [- ln 2 from f = sqrt 2
// on], C = kLogPoints[q] 2^-24 near 1/f of the middle.
struct LogEntry {
    double c, minus_ln;
};
struct Exp2Entry {
    double hi, lo;  // 2^(j/64)
};
struct alignas(16) F64Tables {
    LogEntry lg[128];
    Exp2Entry e2[64];
};
constexpr int kLogSqrt2 = 53;  // first interval taken as twice a number below 1

// Gal's accurate table (S. Gal, "An accurate elementary mathematical library for the
// IEEE floating point standard", ACM TOMS 17, 1991): of the 24-bit numbers around 1/f of
// an interval's middle (with |r| <= 2^-8 on the interval, or within 2^-10 of it) the one
// whose logarithm is nearest to a multiple of 2^-49, within 2e-17 of the logarithms that
// it is used for, so that no second table entry has to carry the rest; 1 and 1/2 at
// the two ends, so that the logarithm of a number just below 1 keeps its relative
// accuracy.
constexpr uint32_t kLogPoints[128] = {
    0x1000000, 0x0fcd3b3, 0x0fb3148, 0x0f95b6d, 0x0f77aa7, 0x0f58b7a, 0x0f384e8, 0x0f1f52c,
    0x0f03710, 0x0ee1b0e, 0x0ec9629, 0x0eb097f, 0x0e90b9d, 0x0e7a7ab, 0x0e609b7, 0x0e45a4f,
    0x0e2c462, 0x0e112a6, 0x0df9f04, 0x0de2a92, 0x0dc89f9, 0x0daf8c5, 0x0d9bd58, 0x0d81492,
    0x0d70b67, 0x0d59e70, 0x0d41821, 0x0d2e40d, 0x0d18c1e, 0x0d02683, 0x0ced9fc, 0x0cd4c23,
    0x0cc38a1, 0x0cb1260, 0x0c9949c, 0x0c87f10, 0x0c703d2, 0x0c5d2b0, 0x0c4e750, 0x0c3a195,
    0x0c29090, 0x0c12db3, 0x0c0577f, 0x0bf0f60, 0x0be0021, 0x0bcf9e5, 0x0bbc7dc, 0x0bab395,
    0x0b9864a, 0x0b87018, 0x0b75f9d, 0x0b6753b, 0x0b5a9d8, 0x0b46ff7, 0x0b392e9, 0x0b2bf54,
    0x0b19547, 0x0b0c56a, 0x0af9944, 0x0aed66a, 0x0adac9b, 0x0acff57, 0x0ac34d0, 0x0aae434,
    0x0aa0ccb, 0x0a92df2, 0x0a85dfe, 0x0a7c276, 0x0a68be4, 0x0a5c575, 0x0a4db18, 0x0a44a5b,
    0x0a3427b, 0x0a2a651, 0x0a1e775, 0x0a11e7d, 0x0a01cfe, 0x09f5b9d, 0x09eaca2, 0x09dd0d7,
    0x09cf6a6, 0x09c2efc, 0x09b7cbb, 0x09aee4e, 0x09a4e8a, 0x0999bdf, 0x0989aaa, 0x097f43c,
    0x0978eb3, 0x0967934, 0x095fe5c, 0x0952132, 0x094814c, 0x0942768, 0x09352c0, 0x092b25d,
    0x0921da1, 0x0911212, 0x0908fac, 0x09023eb, 0x08f5fc0, 0x08e92fe, 0x08e5da6, 0x08d8804,
    0x08ce6b8, 0x08c8096, 0x08b9183, 0x08b3f91, 0x08a8ff9, 0x089f5be, 0x0894675, 0x088d0d2,
    0x08840fa, 0x087c463, 0x08712d5, 0x0867542, 0x085dd4d, 0x0856fcf, 0x0852db8, 0x0845e3b,
    0x083fef6, 0x08327d1, 0x0829f50, 0x0825a2b, 0x0820006, 0x0810a79, 0x080cc3d, 0x0800000,
};

// (on the host, in extended precision; the kernels copy the tables to LDS)
inline void make_f64_tables(F64Tables& t)
{
    for (int q = 0; q < 128; ++q) {
        const long double C = kLogPoints[q] * 0x1p-24L;
        const long double l = -logl((q >= kLogSqrt2 ? 2.0L : 1.0L) * C);
        t.lg[q] = {(double)(C * 0x1p-31L), (double)(rintl(l * 0x1p49L) * 0x1p-49L)};
    }
    for (int j = 0; j < 64; ++j) {
        const long double v = exp2l(j / 64.0L);
        const double hi = (double)v;
        t.e2[j] = {hi, (double)(v - (long double)hi)};
    }
}

// ln u for u = ((w >> 9) + 1/2) 2^-23 = m 2^-24: m = n 2^-z normalised to 32 bits,
// f = n 2^-31, r = C f - 1 (exact: 24 bits each; |r| < 0.005, in the first interval
// 0 <= r < 2^-7), and ln u = (E ln 2 - ln C + r) + (log1p(r) - r): the first sum is
// exact (multiples of 2^-49, below 2^4 where ln C counts), the rest r^2 times a polynomial.
__host__ __device__ __forceinline__ double log_u01(const F64Tables& t, uint32_t w)
{
    const uint32_t m = (w >> 8) | 1u;
    const int z = __builtin_clz(m);
    const uint32_t n = m << z;
    const int q = (int)(n >> 24) - 128;
    const LogEntry g = t.lg[q];
    const double r = __builtin_fma((double)n, g.c, -1.0);
    const double E = (double)(7 - z + (q >= kLogSqrt2 ? 1 : 0));
    double p = 1.0 / 7.0;
    p = __builtin_fma(p, r, -1.0 / 6.0);
    p = __builtin_fma(p, r, 1.0 / 5.0);
    p = __builtin_fma(p, r, -1.0 / 4.0);
    p = __builtin_fma(p, r, 1.0 / 3.0);
    p = __builtin_fma(p, r, -1.0 / 2.0);
    // ln 2 as 40 bits and the rest
    const double h = __builtin_fma(E, 0x1.62e42fefa2000p-1, g.minus_ln) + r;
    return h + __builtin_fma(p, r * r, E * 0x1.9ef35793c7673p-41);
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
