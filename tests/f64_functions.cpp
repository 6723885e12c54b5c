// Largest and root-mean-square relative errors of the step's FP64 functions, run on
// the host, against extended precision: the logarithm, sine and cosine over every
// 23-bit uniform, the exponential and the hop probability over x in +-50 and beyond.
// Test helper only; compiled by the test into a temporary directory.
#include <cstdio>
#include <random>

#include "ssp_f64.h"

struct Errors {
    double most = 0.0, squares = 0.0;
    long n = 0;
    void add(double got, long double want)
    {
        const double e = (double)fabsl(((long double)got - want) / want);
        most = e > most ? e : most;
        squares += e * e;
        ++n;
    }
    void print(const char* name) const { std::printf("%s %.6e %.6e\n", name, most, std::sqrt(squares / n)); }
};

int main()
{
    ssp::F64Tables t;
    ssp::make_f64_tables(t);
    Errors lg, sn, cs, ex, hop, far;
    const long double two_pi = 6.283185307179586476925286766559005768L;
    for (uint32_t i = 0; i < (1u << 23); ++i) {
        const uint32_t w = (i << 9) | (i & 511u);  // (the low nine bits don't count)
        const long double u = ((long double)i + 0.5L) / 8388608.0L;
        lg.add(ssp::log_u01(t, w), logl(u));
        const int k = (int)rintl(4.0L * u);
        const long double x = (u - k / 4.0L) * two_pi, s = sinl(x), c = cosl(x);
        double got_c, got_s;
        ssp::sincos_u01(w, got_c, got_s);
        const long double s4[4] = {s, c, -s, -c}, c4[4] = {c, -s, -c, s};
        sn.add(got_s, s4[k & 3]);
        cs.add(got_c, c4[k & 3]);
    }
    std::mt19937_64 g(5);
    std::uniform_real_distribution<double> wide(-50.0, 50.0), whole(-700.0, 700.0);
    std::normal_distribution<double> near(0.0, 4.0);
    for (int i = 0; i < (1 << 23); ++i) {
        const double x = i & 1 ? wide(g) : near(g);
        int n;
        const double e = std::ldexp(ssp::exp_scaled(t, x, n), n);
        ex.add(e, expl(x));
        hop.add(std::fmin(0.2 / (1.0 + e), 0.5), (long double)0.2 / (1.0L + expl(x)));
    }
    for (int i = 0; i < (1 << 16); ++i) {
        const double x = i < 2 ? (i ? 700.0 : -700.0) : whole(g);
        int n;
        const double v = ssp::exp_scaled(t, x, n);
        far.add(std::ldexp(v, n), expl(x));
    }
    lg.print("log");
    sn.print("sin");
    cs.print("cos");
    ex.print("exp");
    hop.print("hop");
    far.print("far");
    return 0;
}
