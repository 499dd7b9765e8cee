// fixed_point.cpp -- the rounding of a node sum's two words to FP64
// (fx_total of mech_math.h) against 128-bit integers (tests/test_fixed_point.py).
//
// At most 2^19 contributions of |h| <= 2^43 and |l| <= 2^43 each.  Correctly
// rounded while |total| < 2^30 (97 bits); beyond it two roundings, each half an
// ulp of its result, the first at most doubled by the second's binade: 1 ulp
// and a half bound it.
#define MECH_HD_INLINE static inline
#include "mech_math.h"

#include <stdio.h>
#include <random>

typedef __int128 i128;

// (H 2^44 + L) 2^-67, rounded to nearest even; `ulp`: of the result
static double rounded(i128 t, double &ulp) {
    const bool neg = t < 0;
    unsigned __int128 m = neg ? -(unsigned __int128)t : (unsigned __int128)t;
    int bits = 0;
    while (bits < 128 && m >> bits) ++bits;
    const int drop = bits > 53 ? bits - 53 : 0;
    unsigned __int128 q = m >> drop;
    if (drop) {
        const unsigned __int128 rest = m - (q << drop), half = (unsigned __int128)1 << (drop - 1);
        if (rest > half || (rest == half && (q & 1))) ++q;
    }
    ulp = ldexp(1.0, drop - 67);
    const double x = ldexp((double)(uint64_t)q, drop - 67);
    return neg ? -x : x;
}

int main() {
    std::mt19937_64 rng(7);
    long bad = 0, n = 0;
    auto check = [&](long long H, long long L) {
        const i128 t = (i128)H * ((i128)1 << 44) + L;
        double ulp;
        const double ref = rounded(t, ulp), got = mech::fx_total(H, L);
        const bool small = fabs(ref) < 0x1p30;
        ++n;
        if (small ? got != ref : !(fabs(got - ref) <= 1.5 * ulp)) {
            if (++bad <= 10) printf("FAILED H %lld L %lld: %.17g, not %.17g\n", H, L, got, ref);
        }
    };
    for (long long H : {0ll, 1ll, -1ll, 5ll, -(1ll << 30), (1ll << 53) - 1, -(1ll << 53), (1ll << 62)})
        for (long long L : {0ll, 1ll, -1ll, 1ll << 43, -(1ll << 43), (1ll << 44) - 1, 1ll << 44, -(1ll << 44), (1ll << 53) + 1,
                            -(1ll << 53) - 1, (1ll << 62) - 1, -(1ll << 62)})
            check(H, L);
    for (int i = 0; i < 2000000; ++i) {
        const int hb = 1 + (int)(rng() % 62), lb = 1 + (int)(rng() % 62);
        const long long H = (long long)rng() >> (64 - hb), L = (long long)rng() >> (64 - lb);
        check(H, L);
        // the two words cancel but for a few bits
        if (lb > 45) check(-(L >> 44) + (long long)(rng() % 3) - 1, L);
    }
    printf("%ld sums, %ld failed\n", n, bad);
    return bad != 0;
}
