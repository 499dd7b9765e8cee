// math_seeds.cpp -- the refined reciprocal, the quotient and the logarithm of
// mech_math.h from a seed as inexact as the hardware's (tests/test_math_seeds.py).
//
// The seed is 1/b (1 + d) with |d| up to 2^-24, which is above the 2^-24.3
// measured on the device.  One third-order step leaves d^3 = 2^-72 and the
// rounding of two fused multiply-adds, the last of them half an ulp and the other
// one e times an ulp: below 0.51 ulp of the reciprocal, but a result just above a
// power of two counts in ulps of half the size, so 1.02.  The quotient's residual step
// rounds once more: the same bound.  The logarithm's bar is the one of
// tests/test_math_accuracy.py.
#define MECH_HD_INLINE static inline
static double seed(double b);
#define MECH_RCP_SEED(b) seed(b)
#include "mech_math.h"

#include <stdio.h>
#include <random>

static std::mt19937_64 rng(11);
static double worst_seed = 0x1p-24;
static double seed(double b) {
    // the ends of the interval as often as its inside
    const double u = (double)(long long)rng() * 0x1p-63, d = worst_seed * (fabs(u) < 0.25 ? (u < 0 ? -1.0 : 1.0) : u);
    return (double)(1.0L / b * (1.0L + d));
}
static double ulps(double got, long double ref) {
    int e;
    frexp((double)ref, &e);
    return (double)(fabsl(got - ref) / ldexpl(1.0L, e - 53));
}

int main() {
    double e_rcp = 0, e_div = 0, e_log = 0;
    auto one = [&](double b) {
        e_rcp = fmax(e_rcp, ulps(mech::rcp_d(b), 1.0L / b));
        const double a = ldexp(1.0 + (double)(rng() >> 12) * 0x1p-52, (int)(rng() % 40) - 20);
        e_div = fmax(e_div, ulps(mech::fdiv(a, b), (long double)a / b));
        // the logarithm divides m - 1 by m + 1
        const double y = fabs(b);
        if (y > 1e-12 && y < 1e12 && y != 1.0) e_log = fmax(e_log, ulps(mech::log_d(y), logl((long double)y)));
    };
    for (int i = 0; i < 1000000; ++i) {
        const double m = 1.0 + (double)(rng() >> 12) * 0x1p-52;
        one(ldexp(rng() & 1 ? m : -m, (int)(rng() % 600) - 300));
        one(ldexp(m, (int)(rng() % 60) - 30));
    }
    for (int k = -300; k <= 300; ++k)
        for (double m : {1.0, 1.0 + 0x1p-52, 2.0 - 0x1p-52, 1.5, 1.0 + 0x1p-26}) one(ldexp(m, k));
    printf("rcp %.4f ulp, quotient %.4f, logarithm %.4f\n", e_rcp, e_div, e_log);
    return !(e_rcp <= 1.02 && e_div <= 1.02 && e_log <= 1.5);
}
