// Host checks of rvea_variation.h.
//   spread n step   largest relative error of half_spread against long double, in
//                   units of 2^-53: all variates that are a multiple of step, and
//                   the 64 next to 0, 1/2 and 1.  The binary32 estimate is that of
//                   the device with correctly rounded log2 and exp2.
//   gap             "log(U) log(1-p) d" lines from the input, a gap each
#include <cstdio>
#include <cstdlib>

#include "rvea_variation.h"

static double error_of(uint32_t u, int n)
{
    const bool lo = u < 0x800000u;
    const uint32_t v = lo ? u : 0x1000000u - u;
    const float one = std::ldexp(1.0f, n - 25), af = (float)v * one, ninv = 1.0f / (float)n;
    const float log2 = (float)std::log2((double)std::fmax(af, one));
    const float l = std::fma(-ninv, log2, ((float)(n - 2)) * ninv - 1.0f);
    const double zh = (double)(float)std::exp2((double)l);
    const double got = n == 21 ? rvea::half_spread<21>(lo, af, zh, n) : rvea::half_spread<0>(lo, af, zh, n);
    if (u == 0) return got == 0.0 ? 0.0 : 1e300;
    const long double a = (long double)v * 0x1p-23L;
    const long double want = 0.5L * std::pow(a, (lo ? 1.0L : -1.0L) / (long double)n);
    return (double)(std::fabs((long double)got - want) / want) * 0x1p53;
}

int main(int argc, char **argv)
{
    if (argc == 2) {
        double logu, lq;
        int d;
        while (std::scanf("%la %la %d", &logu, &lq, &d) == 3)
            std::printf("%d\n", rvea::mutation_gap(logu, lq, d));
        return 0;
    }
    if (argc != 4) return 2;
    const int n = std::atoi(argv[2]);
    const uint32_t step = (uint32_t)std::atoi(argv[3]);
    double worst = 0.0;
    auto take = [&](uint32_t u) {
        const double e = error_of(u, n);
        if (!(e <= worst)) worst = e;
    };
    for (uint32_t u = 0; u < 1u << 24; u += step) take(u);
    for (uint32_t k = 0; k < 64; ++k) {
        take(k);
        take((1u << 24) - 1 - k);
        take((1u << 23) - 32 + k);
    }
    std::printf("%.6g\n", worst);
    return 0;
}
