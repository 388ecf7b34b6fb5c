// Largest error of each function of csrc/math64.hpp, in units of the last place of
// the result, against 64-bit significands (long double) over the arguments the
// float64 paths have. Prints "name ulp" lines.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <random>

#include "../../paper_2012_14332_amd/csrc/math64.hpp"

using namespace abc;

static double ulps(double got, long double want)
{
    if (want == 0.0L) return got == 0.0 ? 0.0 : INFINITY;
    const double w = (double)want;
    const double step = std::nextafter(std::fabs(w), INFINITY) - std::fabs(w);
    return (double)(std::fabs((long double)got - want) / (long double)step);
}

struct Worst {
    const char* name;
    double e = 0.0;
    explicit Worst(const char* n) : name(n) {}
    void add(double got, long double want) { const double u = ulps(got, want); if (!(u <= e)) e = u; }
    ~Worst() { std::printf("%s %.4f\n", name, e); }
};

int main()
{
    static Math64 tab;
    stage_math64(tab);
    std::mt19937_64 g(1);
    std::uniform_real_distribution<double> unit(0.0, 1.0);
    const int N = 300000;
    {
        Worst w("log");
        auto one = [&](double x) { w.add(log_mid(x, tab), logl((long double)x)); };
        for (int i = 0; i < N; ++i) {
            one(((double)(g() >> 43) + 0.5) * 0x1p-21);    // the noise's uniforms
            one(((double)(g() >> 32) + 1.0) * 0x1p-32);    // the proposals'
            one(std::floor(std::exp2(31.0 * unit(g))) + 1.0);  // 1 + a count
        }
        for (int i = 1; i <= 70000; ++i) one((double)i);
        // both sides of every table interval, and of the carry at 3/2, around 1
        for (int e = -32; e <= 31; ++e)
            for (int i = 0; i <= LOG_N; ++i)
                for (int d = -2; d <= 2; ++d) {
                    const double x = host_double(host_bits(std::ldexp(1.0 + i / (double)LOG_N, e)) + (int64_t)d);
                    if (x != 1.0) one(x);
                }
    }
    {
        Worst s("sin"), c("cos");
        auto one = [&](double phi) {
            double sn, cs;
            sincos_turn(phi, sn, cs);
            s.add(sn, sinl((long double)phi));
            c.add(cs, cosl((long double)phi));
        };
        const double two_pi = 2.0 * 3.14159265358979323846;
        for (int i = 0; i < N; ++i) {
            one(two_pi * (((double)(g() >> 43) + 0.5) * 0x1p-21));
            one(6.283185307179586 * ((double)(g() >> 32) * 0x1p-32));
        }
        for (int q = 0; q < (1 << 21); q += 1 << 17)  // around the multiples of pi / 8
            for (int d = -40; d < 40; ++d)
                if (q + d >= 0) one(two_pi * (((double)(q + d) + 0.5) * 0x1p-21));
    }
    {
        Worst w("pow");
        auto one = [&](double M, float n) { w.add(pow_exp(pow_arg(M, (double)n, tab), tab), powl((long double)M, (long double)n)); };
        for (int i = 0; i < N; ++i) {
            const double M = std::floor(std::exp2(31.0 * unit(g)));
            one(M, (float)(POW_N_MAX * unit(g)));
            one(M, (float)(2.0 * unit(g)));
        }
        for (double M : {1.0, 2.0, 3.0, 127.0, 128.0, 2147483647.0})
            for (float n : {0.0f, 0x1p-149f, 0x1p-24f, 0.5f, 1.0f, 2.0f, 15.999999f, 16.0f}) one(M, n);
    }
    for (double err : {0.0, 0x1p-23, -0x1p-23}) {
        seed_error = err;
        Worst r("sqrt"), d("div"), b("divby");
        for (int i = 0; i < N / 3; ++i) {
            const double x = std::exp2(120.0 * unit(g) - 60.0), y = std::exp2(400.0 * unit(g));
            r.add(sqrt_mid(x), sqrtl((long double)x));
            d.add(div_mid(x, 1.0 + y), (long double)x / (long double)(1.0 + y));
            const double P = std::floor(std::exp2(31.0 * unit(g))) + 1.0;
            b.add(div_by(x, P, 1.0 / P), (long double)x / (long double)P);
        }
        if (sqrt_mid(0.0) != 0.0 || !std::isinf(sqrt_mid(INFINITY)) || !std::isnan(sqrt_mid(-1.0))) r.e = INFINITY;
    }
    return 0;
}
