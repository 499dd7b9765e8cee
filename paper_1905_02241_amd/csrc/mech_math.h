// mech_math.h -- FP64 elementary functions of the mechanism kernels.
//
// Device code of the kernels, also compiled for the host by the accuracy test
// (tests/math_host.cpp), which defines MECH_HD_INLINE itself.
#pragma once
#include <math.h>

#ifndef MECH_HD_INLINE
#define MECH_HD_INLINE __host__ __device__ __forceinline__
#endif

namespace mech {

// e^x, e^x - 1 and ln x in FP64 for the rate and reversal-potential
// expressions.  The library versions keep their polynomial coefficients in
// about forty vector registers across the fused kernels' loops, which held
// the FP64 fused kernel at 4 waves per SIMD; these take each coefficient as
// the scalar operand of the fused multiply-add (fma_s), so the kernels fit
// in 70 to 80 (FP64) and 55 (FP32-mixed) registers, the time-fused ones in 87 to 90
// and 70.

// a b + c with c in a scalar register pair (one scalar operand is allowed per
// vector instruction).
MECH_HD_INLINE double fma_s(double a, double b, double c) {
#if defined(__HIP_DEVICE_COMPILE__)
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
#else
    return fma(a, b, c);   // host builds (the accuracy test): the same operation
#endif
}
// 1/b within about one ulp without the IEEE division sequence's scaling steps:
// the hardware reciprocal (2^-24.3 measured) and one third-order step, r <- r +
// r (e + e^2) with e = 1 - b r, whose error is e^3 (two Newton steps, which
// this replaces, take one operation more and end at the same rounding error).
// Valid for normal, finite, non-zero b.  Host builds refine 1/b, or what the
// seed's test (tests/math_seeds.cpp) puts in its place.
#if defined(__HIP_DEVICE_COMPILE__)
#define MECH_RCP_SEED(b) __builtin_amdgcn_rcp(b)
#elif !defined(MECH_RCP_SEED)
#define MECH_RCP_SEED(b) (1.0 / (b))
#endif
MECH_HD_INLINE double rcp_d(double b) {
    const double r = MECH_RCP_SEED(b), e = fma(-b, r, 1.0);
    return fma(r, fma(e, e, e), r);
}
// a/b with one residual correction of the quotient, for a/b in the normal
// range (every rate expression's).
MECH_HD_INLINE double fdiv(double a, double b) {
    const double r = rcp_d(b);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}

// Reduction after Cody and Waite: x = k ln2 + r with k = rint(x / ln2) and r
// formed by two fused multiply-adds against ln2 split into a double and its
// remainder, so |r| <= ln2/2 up to rounding.  e^r - 1 = r + r^2/2 + r^3 p(r)
// with p the polynomial of degree 9 whose error relative to e^r - 1 is smallest
// there (Remez exchange in 200 bits: 2^-61.7; degree 8 would be 2^-55.2, which
// shows in the result).  For |x| < 2^50; far below -745 and above 710 the
// exponent adjust alone gives 0 and +inf, and NaN passes.  Against long-double
// references (tests/test_math_accuracy.py): e^x within 1 ulp,
// e^x - 1 within 1.8 ulp, ln x within 1.2 ulp, sin x within 1.5 ulp.
constexpr double kLn2Hi = 0x1.62e42fefa39efp-1, kLn2Lo = 0x1.abc9e3b39803fp-56, kLog2e = 0x1.71547652b82fep+0;
MECH_HD_INLINE double em1_series(double r) {
    double p = 0x1.1ef5222fa41b6p-29;
    p = fma_s(p, r, 0x1.af5d200d2370ep-26);
    p = fma_s(p, r, 0x1.27e52b2d06e95p-22);
    p = fma_s(p, r, 0x1.71ddf95400f23p-19);
    p = fma_s(p, r, 0x1.a01a018305ca2p-16);
    p = fma_s(p, r, 0x1.a01a01af758adp-13);
    p = fma_s(p, r, 0x1.6c16c16c1cce4p-10);
    p = fma_s(p, r, 0x1.111111110f7ecp-7);
    p = fma_s(p, r, 0x1.5555555555549p-5);
    p = fma_s(p, r, 0x1.5555555555559p-3);
    p = fma(p, r, 0.5);
    return fma(r * r, p, r);
}
MECH_HD_INLINE int exp_reduce(double x, double &r) {
    const double k = rint(x * kLog2e);
    r = fma(-k, kLn2Lo, fma(-k, kLn2Hi, x));
    return (int)k;
}
MECH_HD_INLINE double exp_d(double x) {
    double r;
    const int k = exp_reduce(x, r);
    return ldexp(1.0 + em1_series(r), k);
}
// e^x for x <= 0 of any size (-inf too), for a decay over a step: 0 below -745.
// NaN gives 0 as well: the caller's other operand carries it.
MECH_HD_INLINE double exp_decay_d(double x) { return exp_d(fmax(x, -746.0)); }
// e^x - 1 = 2^k (e^r - 1) + (2^k - 1): the series alone when k = 0, so the
// result keeps its relative accuracy near x = 0; k at most 1024, where 2^k is
// +inf and the series' part still finite.
MECH_HD_INLINE double expm1_d(double x) {
    double r;
    int k = exp_reduce(x, r);
    k = k < 1024 ? k : 1024;
    return ldexp(em1_series(r), k) + (ldexp(1.0, k) - 1.0);
}
// ln x = e ln2 + ln m with x = m 2^e, m in [sqrt(1/2), sqrt(2)).  With
// f = m - 1 (exact) and s = f/(m + 1), |s| <= 0.172, ln m = 2 atanh(s) =
// 2s + s R with R = 2s^2/3 + 2s^4/5 + ... (series to s^22, tail below 2^-59
// relative), and 2s = f - s f, so ln m = f - s (f - R): the exact f carries
// the result and the rounding of the rest stays small beside it.  0 gives
// -inf, negative arguments and NaN give NaN, +inf gives +inf.
MECH_HD_INLINE double log_d(double x) {
    int e;
    double m = frexp(x, &e);
    if (m < 0x1.6a09e667f3bcdp-1) {   // sqrt(1/2)
        m += m;
        e -= 1;
    }
    const double f = m - 1.0;
    const double s = fdiv(f, m + 1.0), z = s * s;
    double p = 2.0 / 23.0;            // then 2/21 ... 2/5
    p = fma_s(p, z, 2.0 / 21.0);
    p = fma_s(p, z, 2.0 / 19.0);
    p = fma_s(p, z, 2.0 / 17.0);
    p = fma_s(p, z, 2.0 / 15.0);
    p = fma_s(p, z, 2.0 / 13.0);
    p = fma_s(p, z, 2.0 / 11.0);
    p = fma_s(p, z, 2.0 / 9.0);
    p = fma_s(p, z, 2.0 / 7.0);
    p = fma_s(p, z, 2.0 / 5.0);
    p = fma_s(p, z, 2.0 / 3.0);
    const double lm = fma(-s, f - z * p, f);
    const double de = (double)e;
    const double y = fma(de, kLn2Hi, fma(de, kLn2Lo, lm));
    if (x > 0.0 && x < INFINITY) return y;
    return x == 0.0 ? -INFINITY : (x == INFINITY ? INFINITY : NAN);
}
// sin x for the clamp waveform: x = k pi/2 + r with k = rint(2x/pi) and r
// formed by three fused multiply-adds against pi/2 split into three doubles
// (accurate while |k| stays far below 2^50), |r| <= pi/4; sin r and cos r
// by their Taylor series to r^19/19! and r^18/18!, and the quadrant k mod 4
// picks +-sin r or +-cos r.  Written out for the same reason as exp_d (the
// library sine holds a large reduction table and its registers).
MECH_HD_INLINE double sin_d(double x) {
    const double k = rint(x * 0x1.45f306dc9c883p-1);   // 2/pi
    double r = fma(-k, 0x1.921fb54442d18p+0, x);
    r = fma(-k, 0x1.1a62633145c07p-54, r);
    r = fma(-k, -0x1.f1976b7ed8fbcp-110, r);
    const double z = r * r;
    double ps = -1.0 / 121645100408832000.0;   // -1/19!, then 1/17! ... 1/5!
    ps = fma_s(ps, z, 1.0 / 355687428096000.0);
    ps = fma_s(ps, z, -1.0 / 1307674368000.0);
    ps = fma_s(ps, z, 1.0 / 6227020800.0);
    ps = fma_s(ps, z, -1.0 / 39916800.0);
    ps = fma_s(ps, z, 1.0 / 362880.0);
    ps = fma_s(ps, z, -1.0 / 5040.0);
    ps = fma_s(ps, z, 1.0 / 120.0);
    ps = fma(ps, z, -1.0 / 6.0);
    const double sr = fma(r * z, ps, r);
    double pc = 1.0 / 6402373705728000.0;   // 1/18!, then -1/16! ... -1/4!
    pc = fma_s(pc, z, -1.0 / 20922789888000.0);
    pc = fma_s(pc, z, 1.0 / 87178291200.0);
    pc = fma_s(pc, z, -1.0 / 479001600.0);
    pc = fma_s(pc, z, 1.0 / 3628800.0);
    pc = fma_s(pc, z, -1.0 / 40320.0);
    pc = fma_s(pc, z, 1.0 / 720.0);
    pc = fma_s(pc, z, -1.0 / 24.0);
    pc = fma(pc, z, 0.5);   // now 1/2 - z/24 + ...
    const double cr = fma(-z, pc, 1.0);
    const double q = k - 4.0 * floor(k * 0.25);   // k mod 4, exact
    const double y = (q == 0.0 || q == 2.0) ? sr : cr;
    return (q >= 2.0) ? -y : y;
}

// The total (H 2^44 + L) 2^-67 of a fixed-point node sum's two signed words
// (mech_kernels.hip).  L's upper 20 bits are carried to H's place, so that every
// part is exact in FP64 while |total| < 2^30 and the last fused multiply-add
// rounds their sum once, whatever the number of contributions; beyond that H's
// part is rounded as well, and the result is within 1.5 ulp.  (Converted as one
// number L exceeds 2^53 from 2^10 contributions on, and where it cancels against
// H its rounding is what is left: over 1e-12 of some sums in tests/fixed_point.cpp.)
// L's low 44 bits convert by their place in the mantissa of 2^52.
MECH_HD_INLINE double fx_total(long long H, long long L) {
    const long long low = (L & 0xfffffffffffll) | 0x4330000000000000ll;
    const double h0 = (double)(unsigned)H + (double)((int)(L >> 32) >> 12);
    const double h = fma((double)(int)(H >> 32), 0x1p9, h0 * 0x1p-23);
    return fma(__builtin_bit_cast(double, low) - 0x1p52, 0x1p-67, h);
}

}  // namespace mech
