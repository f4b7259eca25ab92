// rvea_variation.h -- binary64 arithmetic of crossover and mutation, for the
// device and for host checks of its error.
#pragma once

#include <cmath>
#include <cstdint>
#include <cstring>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define RVEA_HD __host__ __device__ __forceinline__
#else
#define RVEA_HD inline
#endif

namespace rvea {

// z^n for a positive integer n (square and multiply, n uniform); the
// default distribution index eta = 20 (n = 21) gets straight-line code
RVEA_HD double ipow(double z, int n)
{
    if (n == 21) {
        const double z2 = z * z, z4 = z2 * z2, z8 = z4 * z4, z16 = z8 * z8;
        return (z16 * z4) * z;
    }
    double r = 1.0, b = z;
    while (n) {
        if (n & 1) r *= b;
        n >>= 1;
        if (n) b *= b;
    }
    return r;
}

// a double's high word alone (20 fraction bits)
RVEA_HD double high_word(double x)
{
    uint64_t w;
    std::memcpy(&w, &x, 8);
    w &= 0xffffffff00000000ull;
    std::memcpy(&x, &w, 8);
    return x;
}

// Half of the spread factor from af = a 2^(n-2) and zh, half of a binary32
// estimate z of a^(-1/n) (lo: the branch below 1/2).  With t = a z^(n-1) and
// e = 1 - t z, in size some n 1e-7,
//   above 1/2: a^(-1/n) = z (1 - e)^(-1/n),
//   below:     a^(1/n)  = t (1 - e)^(-(n-1)/n)
// (the rounding of t enters e too and cancels but for its n-th part), each by its
// expansion.  Two terms up to n = 32: the largest error over all 2^24 variates
// with this card's estimates is 1.00 to 1.41 times 2^-53 there (a root of third
// order and its reciprocal: 1.41 to 1.88).  The third term is some n^3 1e-21, so
// beyond it is taken too: 1.38 to 1.42 times 2^-53 at n = 33 to 64, 5.98 without.
template <int NR>
RVEA_HD double half_spread(bool lo, float af, double zh, int n)
{
    double p;  // zh^(n-1)
    if (NR == 21 || n == 21) {
        const double z2 = zh * zh, z4 = z2 * z2, z8 = z4 * z4, z16 = z8 * z8;
        p = z16 * z4;
    } else {
        p = ipow(zh, n - 1);
    }
    const double th = (double)af * p;         // t / 2
    const double e4 = std::fma(-th, zh, 0.25);  // e / 4
    const double dn = (double)n;
    // coefficients of e4: 4 c1, 16 c2 and 64 c3, with s = n - 1 below 1/2 and 1
    // above: c1 = s/n, c2 = s (s + n)/(2 n^2), c3 = s (s + n)(s + 2n)/(6 n^3) (the
    // last in use needs no more than 20 bits)
    const double c1 = lo ? 4.0 * (dn - 1.0) / dn : 4.0 / dn;
    const double lo2 = 8.0 * (dn - 1.0) * (2.0 * dn - 1.0) / (dn * dn);
    const double hi2 = 8.0 * (dn + 1.0) / (dn * dn);
    double c2;
    if (NR == 0 && n > 32) {  // uniform
        const double lo3 = lo2 * (3.0 * dn - 1.0) * 4.0 / (3.0 * dn);
        const double hi3 = hi2 * (2.0 * dn + 1.0) * 4.0 / (3.0 * dn);
        c2 = std::fma(e4, lo ? high_word(lo3) : high_word(hi3), lo ? lo2 : hi2);
    } else {
        c2 = lo ? high_word(lo2) : high_word(hi2);
    }
    const double base = lo ? th : zh;
    return std::fma(base * e4, std::fma(e4, c2, c1), base);
}

// Genes between two mutation sites: floor(log U / log(1-p)), at most d.  A
// quotient, not a product with the reciprocal, whose second rounding can leave
// the floor one lower at whole numbers.
RVEA_HD int mutation_gap(double logu, double lq, int d)
{
    double q = logu / lq;
    if (!(q >= 0.0)) q = 0.0;
    q = std::floor(q);
    return q >= (double)d ? d : (int)q;
}

}  // namespace rvea
