// math_edges.cpp -- the FP64 exponentials of mech_math.h far from and at the
// ends of the range of e^x, and the refined reciprocal's quotient
// (tests/test_math_edges.py).
#define MECH_HD_INLINE static inline
#include "mech_math.h"

#include <stdio.h>
#include <initializer_list>

int main() {
    int bad = 0;
    auto check = [&](bool ok, const char *what, double x) {
        if (!ok) {
            ++bad;
            printf("FAILED %s at %.17g\n", what, x);
        }
    };
    for (double x : {711.0, 1e3, 1e6, 1e9}) {
        check(mech::exp_d(x) == INFINITY, "exp", x);
        check(mech::exp_d(-x - 40.0) == 0.0, "exp", -x - 40.0);
        check(mech::expm1_d(x) == INFINITY, "expm1", x);
        check(mech::expm1_d(-x) == -1.0, "expm1", -x);
    }
    for (double x : {0.0, 0.34657, 0.3466, 1.0, 40.0, 709.0, 744.0, 745.0}) {
        const long double ref = expl(-(long double)x);
        // one ulp, or half the smallest number where the result is subnormal
        const double u = fmax(fabs((double)ref) * 0x1p-52, 0x1p-1074);
        check(fabsl(mech::exp_d(-x) - ref) <= 1.0L * u, "exp", -x);
        check(mech::exp_decay_d(-x) == mech::exp_d(-x), "exp_decay", -x);
    }
    for (double x : {746.0, 1e9, 1e300, (double)INFINITY}) check(mech::exp_decay_d(-x) == 0.0, "exp_decay", -x);
    check(mech::exp_d(NAN) != mech::exp_d(NAN) && mech::expm1_d(NAN) != mech::expm1_d(NAN), "NaN", NAN);
    check(mech::fdiv(1.0, 3.0) == 1.0 / 3.0 && mech::fdiv(0.0, 3.0) == 0.0, "fdiv", 3.0);
    printf("%d failed\n", bad);
    return bad != 0;
}
