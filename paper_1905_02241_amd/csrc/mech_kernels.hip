// mech_kernels.hip -- CDNA4 (gfx950) kernels of the mechanism library.
//
// Current update (BREAKPOINT, paper section 3) and state update (DERIVATIVE +
// SOLVE cnexp, sparse and derivimplicit; sections 3 and 5.2) of eight
// mechanism types over SoA instance arrays, in three launch structures:
//
//   plain     one kernel per mechanism type and phase, a thread per
//             instance, node vectors reached through the node index,
//             many-to-one reductions by FP64 global atomics (the paper's
//             per-mechanism kernel structure; section 8 notes the cost of
//             its atomic reductions);
//   fused     one kernel per timestep over a table of node tiles: each block
//             stages its nodes' v in LDS, runs state(k-1), events(k) and
//             cur(k) of every instance in the tile (coalesced SoA streams, a
//             thread per instance), reduces into LDS accumulators, then
//             writes rhs/d and provides v_{k+1} for its own nodes.  No
//             global atomics;
//   resident  the fused kernel's tiles kept in LDS for many steps (clamp and
//             isolated modes), so STATEs cross HBM once per launch.
//
// Cable mode adds the tree solve (k_tree_*) between the current update and
// the voltage.
// The work is elementwise and exponential/division heavy (section 6 calls the
// state kernels compute bound and the current kernels bandwidth bound); there
// is no dense contraction, so no MFMA.  Precision: FP64 throughout, or FP32
// STATEs / rates / conductance products with the hardware exponential and
// FP64 v, driving force, Nernst, Mg block, finite difference and reduction.
#include "mech_internal.h"
#include "mech_math.h"
#include "mech.h"

#include <math.h>

#include <type_traits>

namespace mech {

// ------------------------------------------------------------ FP32 math --
// e^x = 2^(x log2 e) on the hardware exp2 unit (about 1 ulp).
__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }
__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }

// a*x/(1 - exp(-x/k)) with its removable singularity at x = 0.  Near the
// singular point the direct form cancels in FP32, so |u| < 0.5 (u = x/k) uses
// the Bernoulli-number series u/(1 - e^-u) = 1 + u/2 + u^2/12 - u^4/720 +
// u^6/30240 + O(u^8) (truncation < 4e-9 there).
__device__ __forceinline__ float linexp_f(float a, float k, float x) {
    const float u = x * (1.0f / k);
    const float u2 = u * u;
    const float ser = 1.0f + 0.5f * u + u2 * (1.0f / 12.0f + u2 * (-1.0f / 720.0f + u2 * (1.0f / 30240.0f)));
    const float dir = u * frcp(1.0f - fexp(-u));
    return a * k * (fabsf(u) < 0.5f ? ser : dir);
}

// 1 - e^-z for z >= 0.  The direct form loses accuracy for small z, where
// the exponential series z(1 - z/2(1 - z/3(1 - z/4(1 - z/5(1 - z/6))))) is
// used (truncation z^7/5040, relative < 5e-8 below 0.25).
__device__ __forceinline__ float one_minus_exp_f(float z) {
    const float ser = z * (1.0f - z * 0.5f * (1.0f - z * (1.0f / 3.0f) *
                      (1.0f - z * 0.25f * (1.0f - z * 0.2f * (1.0f - z * (1.0f / 6.0f))))));
    return z < 0.25f ? ser : 1.0f - fexp(-z);
}

// ------------------------------------------------------------ FP64 math --
// rcp_d, fdiv, exp_d, expm1_d, log_d and sin_d: mech_math.h.

// a x/(1 - exp(-x/k)), with the limit a k at x = 0; em1 = expm1(-x/k) is
// returned so that a caller can reuse exp(-x/k) = em1 + 1.
__device__ __forceinline__ double linexp_d(double a, double inv_k, double x, double lim, double &em1) {
    em1 = expm1_d(-x * inv_k);
    return x == 0.0 ? lim : fdiv(a * x, -em1);
}
__device__ __forceinline__ double linexp_d(double a, double inv_k, double x, double lim) {
    double em1;
    return linexp_d(a, inv_k, x, lim, em1);
}

// cnexp factor e^{-y} over one step (a rate that is not a number makes the
// gate's target one as well), or its (1,1) Pade approximant
// (1 - y/2)/(1 + y/2) (the optional replacement of the paper's section 5.2).
__device__ __forceinline__ double cnexp_factor(double y, int pade) {
    return pade ? fdiv(1.0 - 0.5 * y, 1.0 + 0.5 * y) : exp_decay_d(-y);
}
// 1 - factor in FP32 without cancellation: the series / exp form above, or
// y/(1 + y/2) for the Pade approximant.
__device__ __forceinline__ float one_minus_factor_f(float y, int pade) {
    return pade ? y * frcp(1.0f + 0.5f * y) : one_minus_exp_f(y);
}

// ----------------------------------------------------- rates and cnexp --
// Hodgkin-Huxley gates at v; x <- x_inf + (x - x_inf) exp(-dt q10 (a + b)).
// exp(-(v+35)/10) = e^{1/2} exp(-(v+40)/10) reuses alpha_m's expm1, and
// exp(-(v+65)/20) = exp(-(v+65)/80)^4 reuses beta_n's exponential.
__device__ __forceinline__ void hh_state(double v, const GlobDev &g, double &m, double &h, double &n) {
    const double e80 = exp_d((v + 65.0) * (-1.0 / 80.0));
    const double e80_2 = e80 * e80;
    double em1_m;
    const double am = linexp_d(0.1, 0.1, v + 40.0, 1.0, em1_m);
    const double bm = 4.0 * exp_d((v + 65.0) * (-1.0 / 18.0));
    const double ah = 0.07 * (e80_2 * e80_2);
    const double bh = fdiv(1.0, 1.0 + (em1_m + 1.0) * 1.6487212707001282);   // e^{1/2}
    const double an = linexp_d(0.01, 0.1, v + 55.0, 0.1);
    const double bn = 0.125 * e80;
    const double sm = am + bm, sh = ah + bh, sn = an + bn;
    const double mi = fdiv(am, sm), hi = fdiv(ah, sh), nI = fdiv(an, sn);
    const double c = g.dt * g.q10;
    m = mi + (m - mi) * cnexp_factor(c * sm, g.pade);
    h = hi + (h - hi) * cnexp_factor(c * sh, g.pade);
    n = nI + (n - nI) * cnexp_factor(c * sn, g.pade);
}

__device__ __forceinline__ void hh_state(double vd, const GlobDev &g, float &m, float &h, float &n) {
    const float v = (float)vd;
    const float e80 = fexp((v + 65.0f) * (-1.0f / 80.0f));
    const float e80_2 = e80 * e80;
    const float am = linexp_f(0.1f, 10.0f, v + 40.0f);
    const float bm = 4.0f * fexp((v + 65.0f) * (-1.0f / 18.0f));
    const float ah = 0.07f * (e80_2 * e80_2);
    const float bh = frcp(1.0f + fexp((v + 35.0f) * (-0.1f)));
    const float an = linexp_f(0.01f, 10.0f, v + 55.0f);
    const float bn = 0.125f * e80;
    const float sm = am + bm, sh = ah + bh, sn = an + bn;
    const float c = (float)(g.dt * g.q10);
    m += (am * frcp(sm) - m) * one_minus_factor_f(c * sm, g.pade);
    h += (ah * frcp(sh) - h) * one_minus_factor_f(c * sh, g.pade);
    n += (an * frcp(sn) - n) * one_minus_factor_f(c * sn, g.pade);
}

__device__ __forceinline__ void hh_inf(double v, double &m, double &h, double &n) {
    const double am = linexp_d(0.1, 0.1, v + 40.0, 1.0);
    const double bm = 4.0 * exp_d(-(v + 65.0) / 18.0);
    const double ah = 0.07 * exp_d(-(v + 65.0) / 20.0);
    const double bh = 1.0 / (1.0 + exp_d(-(v + 35.0) / 10.0));
    const double an = linexp_d(0.01, 0.1, v + 55.0, 0.1);
    const double bn = 0.125 * exp_d(-(v + 65.0) / 80.0);
    m = am / (am + bm);
    h = ah / (ah + bh);
    n = an / (an + bn);
}

// Ih: alpha = 0.005 exp(-(v+90)/20), beta = 0.005 exp((v+90)/20).
__device__ __forceinline__ void ih_state(double v, const GlobDev &g, double &m) {
    const double e = exp_d((v + 90.0) * 0.05);
    const double a = fdiv(0.005, e), b = 0.005 * e, s = a + b;
    const double mi = fdiv(a, s);
    m = mi + (m - mi) * cnexp_factor(g.dt * s, g.pade);
}
__device__ __forceinline__ void ih_state(double vd, const GlobDev &g, float &m) {
    const float e = fexp(((float)vd + 90.0f) * 0.05f);
    const float a = 0.005f * frcp(e), b = 0.005f * e, s = a + b;
    m += (a * frcp(s) - m) * one_minus_factor_f((float)g.dt * s, g.pade);
}
__device__ __forceinline__ double ih_inf(double v) {
    const double a = 0.005 * exp_d(-(v + 90.0) / 20.0), b = 0.005 * exp_d((v + 90.0) / 20.0);
    return a / (a + b);
}

// Ca-HVA gates: alpha_m = 0.1 (v+20)/(1 - exp(-(v+20)/5)), beta_m = 0.8
// exp(-(v+45)/15), alpha_h = 0.0005 exp(-(v+60)/25), beta_h = 0.006/(1 +
// exp(-(v+20)/10)).
__device__ __forceinline__ void ca_gates(double v, const GlobDev &g, double &m, double &h) {
    const double am = linexp_d(0.1, 0.2, v + 20.0, 0.5);
    const double bm = 0.8 * exp_d((v + 45.0) * (-1.0 / 15.0));
    const double ah = 0.0005 * exp_d((v + 60.0) * (-0.04));
    const double bh = fdiv(0.006, 1.0 + exp_d((v + 20.0) * (-0.1)));
    const double sm = am + bm, sh = ah + bh;
    const double mi = fdiv(am, sm), hi = fdiv(ah, sh);
    m = mi + (m - mi) * cnexp_factor(g.dt * sm, g.pade);
    h = hi + (h - hi) * cnexp_factor(g.dt * sh, g.pade);
}
__device__ __forceinline__ void ca_gates(double vd, const GlobDev &g, float &m, float &h) {
    const float v = (float)vd;
    const float am = linexp_f(0.1f, 5.0f, v + 20.0f);
    const float bm = 0.8f * fexp((v + 45.0f) * (-1.0f / 15.0f));
    const float ah = 0.0005f * fexp((v + 60.0f) * (-0.04f));
    const float bh = 0.006f * frcp(1.0f + fexp((v + 20.0f) * (-0.1f)));
    const float sm = am + bm, sh = ah + bh;
    const float dt = (float)g.dt;
    m += (am * frcp(sm) - m) * one_minus_factor_f(dt * sm, g.pade);
    h += (ah * frcp(sh) - h) * one_minus_factor_f(dt * sh, g.pade);
}
// Calcium pool: relaxes to cai_inf = cai0 - kappa tau_ca ica with time
// constant tau_ca, ica held at the value of the last current update.
__device__ __forceinline__ void ca_pool(const GlobDev &g, double ica, double &cai) {
    const double ci = g.cai0 - g.kt_ca * ica;
    cai = ci + (cai - ci) * g.ca_decay;
}
__device__ __forceinline__ void ca_pool(const GlobDev &g, float ica, float &cai) {
    const float ci = (float)g.cai0 - (float)g.kt_ca * ica;
    cai += (ci - cai) * (float)g.ca_omdecay;
}
__device__ __forceinline__ void ca_inf(double v, double &m, double &h) {
    const double am = linexp_d(0.1, 0.2, v + 20.0, 0.5);
    const double bm = 0.8 * exp_d(-(v + 45.0) / 15.0);
    const double ah = 0.0005 * exp_d(-(v + 60.0) / 25.0);
    const double bh = 0.006 / (1.0 + exp_d(-(v + 20.0) / 10.0));
    m = am / (am + bm);
    h = ah / (ah + bh);
}

// kmarkov: C1 <-(2a, b)-> C2 <-(a, 2b)-> O with a = q10 alpha_n, b = q10
// beta_n; implicit Euler (I - dt A) x_new = x_old is tridiagonal and
// diagonally dominant by columns, so the Thomas elimination needs no pivot.
template <class T>
__device__ __forceinline__ void kmarkov_solve(T a, T b, T dt, T &c1, T &c2, T &o) {
    const T d0 = T(1) + T(2) * a * dt, u0 = -b * dt;
    const T l1 = T(-2) * a * dt, d1 = T(1) + (a + b) * dt, u1 = T(-2) * b * dt;
    const T l2 = -a * dt, d2 = T(1) + T(2) * b * dt;
    const T r0 = T(1) / d0;
    const T c0p = u0 * r0, x0p = c1 * r0;
    const T d1p = d1 - l1 * c0p;
    const T r1 = T(1) / d1p;
    const T c1p = u1 * r1, x1p = (c2 - l1 * x0p) * r1;
    const T d2p = d2 - l2 * c1p;
    o = (o - l2 * x1p) / d2p;
    c2 = x1p - c1p * o;
    c1 = x0p - c0p * c2;
}
__device__ __forceinline__ void kmarkov_state(double v, const GlobDev &g, double &c1, double &c2, double &o) {
    const double an = linexp_d(0.01, 0.1, v + 55.0, 0.1);
    const double bn = 0.125 * exp_d((v + 65.0) * (-1.0 / 80.0));
    kmarkov_solve<double>(g.q10 * an, g.q10 * bn, g.dt, c1, c2, o);
}
__device__ __forceinline__ void kmarkov_state(double vd, const GlobDev &g, float &c1, float &c2, float &o) {
    const float v = (float)vd;
    const float an = linexp_f(0.01f, 10.0f, v + 55.0f);
    const float bn = 0.125f * fexp((v + 65.0f) * (-1.0f / 80.0f));
    const float q = (float)g.q10;
    kmarkov_solve<float>(q * an, q * bn, (float)g.dt, c1, c2, o);
}

// capump pool: implicit Euler c - c_old - dt F(c) = 0, F(c) = -kappa ica -
// vmax (c/(c+kp) - cai0/(cai0+kp)), by a fixed number of Newton steps on the
// analytic derivative F'(c) = -vmax kp/(c+kp)^2, starting from c_old.
__device__ __forceinline__ void capump_pool(const GlobDev &g, double ica, double &cai) {
    const double c0 = cai, infl = -g.kappa * ica;
    double c = c0;
    for (int it = 0; it < g.newton_iters; ++it) {
        const double r = fdiv(1.0, c + g.pump_kp);
        const double F = infl - (g.pump_vmax * (c * r) - g.pump_rest);
        const double dF = -g.pump_vmax * g.pump_kp * (r * r);
        c -= fdiv(c - c0 - g.dt * F, 1.0 - g.dt * dF);
    }
    cai = c;
}
__device__ __forceinline__ void capump_pool(const GlobDev &g, float ica, float &cai) {
    const float c0 = cai, infl = -(float)g.kappa * ica, vmax = (float)g.pump_vmax, kp = (float)g.pump_kp;
    const float rest = (float)g.pump_rest, dt = (float)g.dt;
    float c = c0;
    for (int it = 0; it < g.newton_iters; ++it) {
        const float r = 1.0f / (c + kp);
        const float F = infl - (vmax * (c * r) - rest);
        const float dF = -vmax * kp * (r * r);
        c -= (c - c0 - dt * F) / (1.0f - dt * dF);
    }
    cai = c;
}

// cabuf pool: free calcium c and buffer-bound calcium b, binding
// kon c (btot - b) - koff b, relaxation of c to cai0 with tau_ca.  Implicit
// Euler G(c, b) = (c - c_old - dt F_c, b - b_old - dt F_b) = 0 by a fixed
// number of Newton steps from the old state; each step applies the inverse
// of the 2x2 Jacobian I - dt dF/d(c, b) in closed form (adjugate over the
// determinant, which is 1 + dt (x + y + 1/tau_ca) + dt^2 y/tau_ca > 1 with
// x = kon (btot - b) >= 0 and y = kon c + koff > 0, so no pivot is needed).
__device__ __forceinline__ double recip(double x) { return rcp_d(x); }
__device__ __forceinline__ float recip(float x) { return 1.0f / x; }
template <class T>
__device__ __forceinline__ void cabuf_pool(const GlobDev &g, T ica, T &cai, T &cab) {
    const T c0 = cai, b0 = cab, infl = -(T)g.kappa * ica, dt = (T)g.dt;
    const T kon = (T)g.buf_kon, koff = (T)g.buf_koff, btot = (T)g.buf_total;
    const T cai_rest = (T)g.cai0, itau = (T)g.inv_tau_ca;
    T c = c0, b = b0;
    for (int it = 0; it < g.newton_iters; ++it) {
        const T x = kon * (btot - b), y = kon * c + koff;
        const T bind = c * x - koff * b;
        const T gc = c - c0 - dt * (infl - bind - (c - cai_rest) * itau);
        const T gb = b - b0 - dt * bind;
        // J = [[1 + dt (x + 1/tau), -dt y], [-dt x, 1 + dt y]]
        const T j00 = T(1) + dt * (x + itau), j01 = -dt * y, j10 = -dt * x, j11 = T(1) + dt * y;
        const T r = recip(j00 * j11 - j01 * j10);
        c -= (j11 * gc - j01 * gb) * r;
        b -= (j00 * gb - j10 * gc) * r;
    }
    cai = c;
    cab = b;
}

// Synapse decay: A <- A e^{-dt/tau}; in FP32 A <- A - A (1 - e^{-dt/tau}),
// which keeps the rounding of the factor from being amplified by tau/dt.
__device__ __forceinline__ void syn_decay(double *x, const GlobDev &g) {
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] *= g.decay[j];
}
__device__ __forceinline__ void syn_decay(float *x, const GlobDev &g) {
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] -= x[j] * (float)g.omdecay[j];
}

// ------------------------------------------------------------- events --
// SplitMix64 (Steele, Lea & Flood 2014): output n of the generator seeded
// with `seed` is mix(seed + n * golden_gamma); the draw of event stream gid
// at step k is output gid * 2^32 + k + 1.
__device__ __forceinline__ unsigned long long splitmix(unsigned long long seed, unsigned long long gid,
                                                       unsigned long long k) {
    unsigned long long z = seed + ((gid << 32) + k + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// ------------------------------------------------------------ currents --
// Each returns i(v) and the finite-difference conductance (i(v+dv) - i(v))/dv
// with STATEs frozen.  Conductance products are formed in the storage type;
// the driving force and everything after it in FP64.
template <class S>
__device__ __forceinline__ void hh_cur(double v, S m, S h, S n, S gnabar, S gkbar, S gl, double el,
                                       const GlobDev &g, double &i0, double &gg) {
    const double gna = (double)(gnabar * m * m * m * h);
    const double gk = (double)(gkbar * n * n * n * n);
    const double gll = (double)gl;
    i0 = gna * (v - g.ena) + gk * (v - g.ek) + gll * (v - el);
    if (g.analytic_g) {
        gg = gna + gk + gll;
        return;
    }
    const double vd = v + g.fd_dv;
    const double i1 = gna * (vd - g.ena) + gk * (vd - g.ek) + gll * (vd - el);
    gg = (i1 - i0) * g.inv_fd_dv;
}

template <class S>
__device__ __forceinline__ void lin_cur(double v, S gbar_x, double e, const GlobDev &g, double &i0,
                                        double &gg) {
    const double gc = (double)gbar_x;
    i0 = gc * (v - e);
    if (g.analytic_g) {
        gg = gc;
        return;
    }
    const double i1 = gc * (v + g.fd_dv - e);
    gg = (i1 - i0) * g.inv_fd_dv;
}

// Calcium current with the Nernst potential eca = RT/(2F) ln(cao/cai).
template <class S>
__device__ __forceinline__ double ca_cur(double v, S m, S h, S cai, S gbar, const GlobDev &g, double &i0,
                                         double &gg) {
    const double eca = g.nernst * log_d(g.cao / (double)cai);
    const double gc = (double)(gbar * m * m * h);
    i0 = gc * (v - eca);
    if (g.analytic_g) {
        gg = gc;
        return i0;
    }
    const double i1 = gc * (v + g.fd_dv - eca);
    gg = (i1 - i0) * g.inv_fd_dv;
    return i0;
}

// AMPA + NMDA with Mg block B(v) = 1/(1 + exp(-0.062 v) mg/3.57); nS*mV =
// pA, 1e-3 gives nA.  B(v+dv) reuses exp(-0.062 v) times exp(-0.062 dv).
template <class S>
__device__ __forceinline__ void syn_cur(double v, const S *x, const GlobDev &g, double &i0, double &gg) {
    const double ga = (double)(x[1] - x[0]);
    const double gn = (double)(x[3] - x[2]);
    const double ex = exp_d(-0.062 * v);
    const double b0 = fdiv(1.0, 1.0 + ex * g.mg_357);
    i0 = 1e-3 * (ga + gn * b0) * (v - g.e_syn);
    if (g.analytic_g) {
        // di/dv = 1e-3 (ga + gn (B + (v - e) B')), B' = 0.062 B (1 - B)
        gg = 1e-3 * (ga + gn * (b0 + (v - g.e_syn) * 0.062 * b0 * (1.0 - b0)));
        return;
    }
    const double b1 = fdiv(1.0, 1.0 + ex * g.mg_fd * g.mg_357);
    const double vd = v + g.fd_dv;
    const double i1 = 1e-3 * (ga + gn * b1) * (vd - g.e_syn);
    gg = (i1 - i0) * g.inv_fd_dv;
}

template <class S> __device__ __forceinline__ int bad(S x) { return isfinite(x) ? 0 : 1; }

// -------------------------------------------------- instance update ----
// Streamed SoA accesses, optionally with the non-temporal hint (the arrays
// are touched once per step, so they need not displace reusable lines).
template <bool NT, class T> __device__ __forceinline__ T ld(const T *p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT, class T> __device__ __forceinline__ void st(T *p, T v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// One instance of a slot: state update (if PH has kDoState) at v, events and
// current (if kDoCur) at the same v.  Returns the current and conductance
// contributions for the node and stores the new STATEs.
// FOLD (fused path): the calcium pool needs only cai and the ica of the
// current update, so it is advanced right after that update in the same pass
// rather than stored and re-read by the next pass's state update.
// The update is split into its loads (load_inst: every STATE and PARAMETER
// the pass reads, and the event stream id) and the rest (apply_inst), so
// that the fused tile loop can issue the loads of several instances before
// it computes any of them; instance() is the two in sequence.
template <class S> struct InstIn {
    S s[4];                 // STATEs
    S p[4];                 // PARAMETERs
    S ica;                  // the last ica (pool update in the state pass)
    unsigned long long id;  // event stream of a synapse
};

template <class S, int KIND, int PH, bool NT = false, bool FOLD = false>
__device__ __forceinline__ void load_inst(const SlotDev &sl, int i, InstIn<S> &q) {
    constexpr bool cur = (PH & kDoCur) != 0, state = (PH & kDoState) != 0;
    constexpr int n_st = KIND == MECH_PAS ? 0 : KIND == MECH_IH ? 1 : KIND == MECH_SYN ? 4 : 3;
    constexpr int n_par = KIND == MECH_PAS ? 2 : KIND == MECH_HH ? 4 : KIND == MECH_SYN ? 0 : 1;
#pragma unroll
    for (int j = 0; j < n_st; ++j) q.s[j] = ld<NT>((const S *)sl.st[j] + i);
    if constexpr (cur) {
#pragma unroll
        for (int j = 0; j < n_par; ++j) q.p[j] = ld<NT>((const S *)sl.par[j] + i);
    }
    if constexpr (KIND == MECH_CAHVA || KIND == MECH_CAPUMP || KIND == MECH_CABUF) {
        if (state && !FOLD) q.ica = ld<NT>((const S *)sl.ica + i);
    }
    if constexpr (KIND == MECH_CABUF) {
        if ((state && !FOLD) || (cur && FOLD)) q.s[3] = ld<NT>((const S *)sl.st[3] + i);
    }
    if constexpr (KIND == MECH_SYN && cur)
        q.id = sl.gid ? (unsigned long long)(long long)sl.gid[i] : (unsigned long long)i;
}

template <class S, int KIND, int PH, bool NT = false, bool FOLD = false>
__device__ __forceinline__ void apply_inst(const SlotDev &sl, int i, InstIn<S> &q, double v, const GlobDev &g,
                                           long long k, double &ci, double &cg, int &flag) {
    ci = 0.0;
    cg = 0.0;
    if constexpr (KIND == MECH_PAS) {
        if (PH & kDoCur) lin_cur<S>(v, q.p[0], (double)q.p[1], g, ci, cg);
    } else if constexpr (KIND == MECH_HH) {
        S &m = q.s[0], &h = q.s[1], &n = q.s[2];
        if (PH & kDoState) {
            hh_state(v, g, m, h, n);
            flag |= bad(m) | bad(h) | bad(n);
            st<NT>((S *)sl.st[0] + i, m); st<NT>((S *)sl.st[1] + i, h); st<NT>((S *)sl.st[2] + i, n);
        }
        if (PH & kDoCur) hh_cur<S>(v, m, h, n, q.p[0], q.p[1], q.p[2], (double)q.p[3], g, ci, cg);
    } else if constexpr (KIND == MECH_IH) {
        S &m = q.s[0];
        if (PH & kDoState) {
            ih_state(v, g, m);
            flag |= bad(m);
            st<NT>((S *)sl.st[0] + i, m);
        }
        if (PH & kDoCur) lin_cur<S>(v, (S)(q.p[0] * m), g.eh, g, ci, cg);
    } else if constexpr (KIND == MECH_CAHVA || KIND == MECH_CAPUMP) {
        S *M = (S *)sl.st[0], *H = (S *)sl.st[1], *CAI = (S *)sl.st[2], *ICA = (S *)sl.ica;
        S &m = q.s[0], &h = q.s[1], &cai = q.s[2];
        auto pool = [&g](S ica, S &c) {
            if constexpr (KIND == MECH_CAHVA) ca_pool(g, ica, c);
            else capump_pool(g, ica, c);
        };
        if (PH & kDoState) {
            ca_gates(v, g, m, h);
            if (!FOLD) pool(q.ica, cai);
            flag |= bad(m) | bad(h) | bad(cai);
            st<NT>(M + i, m); st<NT>(H + i, h);
            if (!FOLD) st<NT>(CAI + i, cai);
        }
        if (PH & kDoCur) {
            const S ica = (S)ca_cur<S>(v, m, h, cai, q.p[0], g, ci, cg);
            st<NT>(ICA + i, ica);
            if (FOLD) {
                pool(ica, cai);
                flag |= bad(cai);
                st<NT>(CAI + i, cai);
            }
        }
    } else if constexpr (KIND == MECH_KMARKOV) {
        S &c1 = q.s[0], &c2 = q.s[1], &o = q.s[2];
        if (PH & kDoState) {
            kmarkov_state(v, g, c1, c2, o);
            flag |= bad(c1) | bad(c2) | bad(o);
            st<NT>((S *)sl.st[0] + i, c1); st<NT>((S *)sl.st[1] + i, c2); st<NT>((S *)sl.st[2] + i, o);
        }
        if (PH & kDoCur) lin_cur<S>(v, (S)(q.p[0] * o), g.ek, g, ci, cg);
    } else if constexpr (KIND == MECH_CABUF) {
        S *M = (S *)sl.st[0], *H = (S *)sl.st[1], *CAI = (S *)sl.st[2], *CAB = (S *)sl.st[3];
        S *ICA = (S *)sl.ica;
        S &m = q.s[0], &h = q.s[1], &cai = q.s[2], &cab = q.s[3];
        if (PH & kDoState) {
            ca_gates(v, g, m, h);
            if (!FOLD) {
                cabuf_pool<S>(g, q.ica, cai, cab);
                flag |= bad(cab);
                st<NT>(CAI + i, cai); st<NT>(CAB + i, cab);
            }
            flag |= bad(m) | bad(h) | bad(cai);
            st<NT>(M + i, m); st<NT>(H + i, h);
        }
        if (PH & kDoCur) {
            const S ica = (S)ca_cur<S>(v, m, h, cai, q.p[0], g, ci, cg);
            st<NT>(ICA + i, ica);
            if (FOLD) {
                cabuf_pool<S>(g, ica, cai, cab);
                flag |= bad(cai) | bad(cab);
                st<NT>(CAI + i, cai); st<NT>(CAB + i, cab);
            }
        }
    } else if constexpr (KIND == MECH_SYN) {
        S *x = q.s;
        if (PH & kDoState) syn_decay(x, g);
        if (PH & kDoCur) {
            if (splitmix(g.seed, q.id, (unsigned long long)k) < g.threshold) {
                const double w = ((const double *)sl.par[0])[i];
                x[0] += (S)(w * g.fa);
                x[1] += (S)(w * g.fa);
                x[2] += (S)(w * g.fn);
                x[3] += (S)(w * g.fn);
                // a current update alone changes the STATEs only here (it
                // stored them for every synapse: one step of 2 M of them
                // 67 -> 55 us)
                if constexpr (!(PH & kDoState)) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) st<NT>((S *)sl.st[j] + i, x[j]);
                }
            }
            syn_cur<S>(v, x, g, ci, cg);
        }
        flag |= bad(x[0]) | bad(x[1]) | bad(x[2]) | bad(x[3]);
        if constexpr ((PH & kDoState) != 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) st<NT>((S *)sl.st[j] + i, x[j]);
        }
    }
}

template <class S, int KIND, int PH, bool NT = false, bool FOLD = false>
__device__ __forceinline__ void instance(const SlotDev &sl, int i, double v, const GlobDev &g, long long k,
                                         double &ci, double &cg, int &flag) {
    InstIn<S> q;
    load_inst<S, KIND, PH, NT, FOLD>(sl, i, q);
    apply_inst<S, KIND, PH, NT, FOLD>(sl, i, q, v, g, k, ci, cg, flag);
}

// A cahva, capump or cabuf instance under the shared calcium ion: its gates,
// and its current at the node's cai (ica returned for the node's total); the
// pool is the node's (ion_pool), not the instance's, and a cabuf instance's
// own free and bound calcium stay as they are.
template <class S, int PH, bool NT = false>
__device__ __forceinline__ void ca_shared(const SlotDev &sl, int i, double v, double cai, const GlobDev &g,
                                          double &ci, double &cg, double &ica, int &flag) {
    ci = 0.0;
    cg = 0.0;
    ica = 0.0;
    S *M = (S *)sl.st[0], *H = (S *)sl.st[1], *ICA = (S *)sl.ica;
    S m = ld<NT>(M + i), h = ld<NT>(H + i);
    if (PH & kDoState) {
        ca_gates(v, g, m, h);
        flag |= bad(m) | bad(h);
        st<NT>(M + i, m); st<NT>(H + i, h);
    }
    if (PH & kDoCur) {
        const S gbar = ld<NT>((const S *)sl.par[0] + i);
        const S ic = (S)ca_cur<S>(v, m, h, (S)cai, gbar, g, ci, cg);
        st<NT>(ICA + i, ic);
        ica = (double)ic;
    }
}

// The node's calcium pool: the linear pool law driven by the node's total
// calcium current, in FP64 for both storage types.
__device__ __forceinline__ void ion_pool(const GlobDev &g, double ica, double &cai) { ca_pool(g, ica, cai); }

// ---------------------------------------------------------- plain path --
// Segmented inclusive sum over a wave of instances sorted by node: after the
// log2(64) shuffle steps each lane holds the sum of its node's run up to
// itself, so the run's last lane carries the node's total.  Returns true on
// that lane.  Lanes with key < 0 (past the end) form no run.  Z: also sum z
// (the calcium current under the shared ion).
template <bool Z>
__device__ __forceinline__ bool segmented_sum(int key, double &x, double &y, double &z) {
    const int lane = (int)(threadIdx.x & 63);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double xo = __shfl_up(x, d, 64);
        const double yo = __shfl_up(y, d, 64);
        const double zo = Z ? __shfl_up(z, d, 64) : 0.0;
        const int ko = __shfl_up(key, d, 64);
        if (lane >= d && ko == key) {
            x += xo;
            y += yo;
            if (Z) z += zo;
        }
    }
    const int kn = __shfl_down(key, 1, 64);
    return key >= 0 && (lane == 63 || kn != key);
}

// The current update of one type, a thread per instance.  Identity types
// read-modify-write their node.  Node-sorted types sum each node's run within
// the wave (fixed shuffle order) and add it with one FP64 atomic, so a node
// receives one atomic per type; only a run that began in an earlier wave
// would add a second one in an order set by scheduling.  The part of such a
// run in this wave goes to the type's carry slot of this wave instead, and
// k_plain_carry adds those parts in wave order after the kernel.  rhs and d
// therefore do not change from run to run.  With atomic_scatter every
// instance adds its own atomic (the comparison point; order not fixed).
template <class S, int KIND>
__global__ __launch_bounds__(256) void k_plain_cur(PlainArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool shared = is_ca_kind(KIND) && a.g.shared_ca;
    int flag = 0;
    int ni = -1;
    double ci = 0.0, cg = 0.0, ica = 0.0;
    if (i < a.slot.n) {
        ni = a.slot.ni[i];
        const double v = a.nd.v[ni];
        if (shared) {
            ca_shared<S, kDoCur>(a.slot, i, v, a.nd.cai[ni], a.g, ci, cg, ica, flag);
        } else {
            instance<S, KIND, kDoCur>(a.slot, i, v, a.g, a.k, ci, cg, flag);
        }
        if (KIND == MECH_SYN) {
            const double sc = 1e2 / a.nd.area[ni];
            ci *= sc;
            cg *= sc;
        }
    }
    if (a.slot.identity) {
        // one instance per node: a plain read-modify-write, ordered after the
        // previous type's kernel on the stream (the first type: a write in
        // place of clearing the vectors beforehand)
        if (ni >= 0) {
            a.nd.rhs[ni] = (a.overwrite ? 0.0 : a.nd.rhs[ni]) - ci;
            a.nd.d[ni] = (a.overwrite ? 0.0 : a.nd.d[ni]) + cg;
            if (shared) a.nd.ica[ni] += ica;
        }
    } else if (a.atomic_scatter) {
        if (ni >= 0) {
            unsafeAtomicAdd(&a.nd.rhs[ni], -ci);
            unsafeAtomicAdd(&a.nd.d[ni], cg);
            if (shared) unsafeAtomicAdd(&a.nd.ica[ni], ica);
        }
    } else {
        const int lane = (int)(threadIdx.x & 63);
        const int i0 = i - lane;   // the wave's first instance
        if (i0 < a.slot.n) {
            const int c = i0 >> 6;
            // does the wave's first run continue a run of the previous wave?
            int prev = -1;
            if (lane == 0 && i0 > 0) prev = a.slot.ni[i0 - 1];
            prev = __shfl(prev, 0, 64);
            const int first = __shfl(ni, 0, 64);
            const bool cont = prev == first;
            double x = -ci, y = cg, z = ica;
            const bool last = shared ? segmented_sum<true>(ni, x, y, z) : segmented_sum<false>(ni, x, y, z);
            if (last) {
                if (cont && ni == first) {
                    a.carry_node[c] = ni;
                    a.carry_val[3 * (size_t)c] = x;
                    a.carry_val[3 * (size_t)c + 1] = y;
                    a.carry_val[3 * (size_t)c + 2] = z;
                } else {
                    unsafeAtomicAdd(&a.nd.rhs[ni], x);
                    unsafeAtomicAdd(&a.nd.d[ni], y);
                    if (shared) unsafeAtomicAdd(&a.nd.ica[ni], z);
                }
            }
            if (a.crossing && lane == 0 && !cont) a.carry_node[c] = -1;
        }
    }
    if (flag) atomicOr(a.err, 1);
}

// The parts of node runs that crossed into later waves (k_plain_cur's carry
// slots), added in wave order: the thread of the first slot of each chain
// (consecutive slots of one node) sums the chain and adds it to its node,
// which no other thread of this launch touches.
__global__ __launch_bounds__(256) void k_plain_carry(PlainArgs a, int n_chunks, int shared) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_chunks) return;
    const int n = a.carry_node[c];
    if (n < 0 || (c > 0 && a.carry_node[c - 1] == n)) return;
    double x = 0.0, y = 0.0, z = 0.0;
    for (int q = c; q < n_chunks && a.carry_node[q] == n; ++q) {
        x += a.carry_val[3 * (size_t)q];
        y += a.carry_val[3 * (size_t)q + 1];
        z += a.carry_val[3 * (size_t)q + 2];
    }
    a.nd.rhs[n] += x;
    a.nd.d[n] += y;
    if (shared) a.nd.ica[n] += z;
}

template <class S, int KIND>
__global__ __launch_bounds__(256) void k_plain_state(PlainArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    int flag = 0;
    if (i < a.slot.n) {
        const double v = a.nd.v[a.slot.ni[i]];
        double ci, cg;
        if (is_ca_kind(KIND) && a.g.shared_ca) {
            double ica;
            ca_shared<S, kDoState>(a.slot, i, v, 0.0, a.g, ci, cg, ica, flag);
        } else {
            instance<S, KIND, kDoState>(a.slot, i, v, a.g, a.k, ci, cg, flag);
        }
    }
    if (flag) atomicOr(a.err, 1);
}

// Per-node calcium ion: pools after the gates (plain path), and INITIAL.
__global__ void k_ion_pool(NodesDev nd, GlobDev g, int *err) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= nd.n_nodes) return;
    double c = nd.cai[n];
    ion_pool(g, nd.ica[n], c);
    nd.cai[n] = c;
    if (bad(c)) atomicOr(err, 1);
}
__global__ void k_ion_init(NodesDev nd, double cai0) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= nd.n_nodes) return;
    nd.cai[n] = cai0;
    nd.ica[n] = 0.0;
}

// INITIAL: gates at steady state at the bound v (computed in FP64 for both
// storage types), synapse states 0, cai = cai0, ica = 0.
template <class S, int KIND>
__global__ __launch_bounds__(256) void k_init(PlainArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.slot.n) return;
    const double v = a.nd.v[a.slot.ni[i]];
    S **st = (S **)a.slot.st;
    if constexpr (KIND == MECH_HH) {
        double m, h, n;
        hh_inf(v, m, h, n);
        st[0][i] = (S)m; st[1][i] = (S)h; st[2][i] = (S)n;
    } else if constexpr (KIND == MECH_IH) {
        st[0][i] = (S)ih_inf(v);
    } else if constexpr (is_ca_kind(KIND)) {
        double m, h;
        ca_inf(v, m, h);
        st[0][i] = (S)m; st[1][i] = (S)h; st[2][i] = (S)a.g.cai0;
        // cabuf: the bound calcium in equilibrium with cai0
        if (KIND == MECH_CABUF)
            st[3][i] = (S)(a.g.buf_total * a.g.buf_kon * a.g.cai0 / (a.g.buf_kon * a.g.cai0 + a.g.buf_koff));
        ((S *)a.slot.ica)[i] = (S)0;
    } else if constexpr (KIND == MECH_KMARKOV) {
        double m, h, n;
        hh_inf(v, m, h, n);
        st[0][i] = (S)((1.0 - n) * (1.0 - n));
        st[1][i] = (S)(2.0 * n * (1.0 - n));
        st[2][i] = (S)(n * n);
    } else if constexpr (KIND == MECH_SYN) {
        for (int j = 0; j < 4; ++j) st[j][i] = (S)0;
    }
}

__global__ void k_fill(double *a, double *b, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) { a[i] = 0.0; b[i] = 0.0; }
}
__global__ void k_fill_int(int *a, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = 0;
}
__global__ void k_set_k(long long *kdev, long long value) {
    if (threadIdx.x == 0) *kdev = value;
}
__global__ void k_bump_k(long long *kdev, long long by) {
    if (threadIdx.x == 0) *kdev += by;
}

__device__ __forceinline__ double clamp_v(const NodesDev &nd, int n, double t) {
    return nd.c_off[n] + nd.c_amp[n] * sin_d(2.0 * 3.14159265358979323846 * nd.c_freq[n] * t * 1e-3 + nd.c_phase[n]);
}

__global__ void k_vclamp(NodesDev nd, double t) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n < nd.n_nodes) nd.v[n] = clamp_v(nd, n, t);
}

// Backward Euler of an isolated compartment, 1e-3 cm (v1 - v0)/dt = rhs -
// d (v1 - v0), and an upward crossing of vthresh counts a spike.
__device__ __forceinline__ double isolated_v(const NodesDev &nd, const GlobDev &g, int n, double v0, double r,
                                             double dd) {
    const double v1 = v0 + r / (1e-3 * nd.cm[n] / g.dt + dd);
    if (v0 < g.vthresh && v1 >= g.vthresh) nd.spikes[n] += 1;
    return v1;
}

__global__ void k_visolated(NodesDev nd, GlobDev g) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n < nd.n_nodes) nd.v[n] = isolated_v(nd, g, n, nd.v[n], nd.rhs[n], nd.d[n]);
}

// ---------------------------------------------------------- cable solve --
// Backward Euler of the cable equation on each cell's tree, linearised with
// the mechanisms' rhs and d.  Row n, scaled by a_n = area_n/100 so that both
// ends of an edge see the same conductance g:
//   S_n dv_n - sum_j g_nj dv_j = T_n,
//   S_n = L_n + sum_j g_nj, L_n = a_n (1e-3 cm/dt + d_n),
//   T_n = a_n rhs_n + sum_j g_nj (v_j - v_n).
// A round (mech_tree.h) eliminates rows i that have a parent p (coupling U_i)
// and at most one child c (coupling N_i, until then U_c):
//   S_p -= U_i^2/S_i, L_p += L_i U_i/S_i, T_p += T_i U_i/S_i, and the same for c
//   with N_i; c then hangs off p with U_c = N_i U_i/S_i.
// After the last round dv = T/L at the roots, and the rounds are walked
// backwards with dv_i = (T_i + U_i dv_p + N_i dv_c)/(L_i + U_i + N_i), whose
// three quotients are formed for all rows at once beforehand.
// The differences S lose to cancellation what the couplings exceed L by; as
// factors they hardly pass it on.  rms error of dv over steps 0 to 200 of eight
// models against 128-bit arithmetic: 0.57 to 0.91 (once 1.2) of Hines
// elimination's in FP64; walking back with S too it was 0.62 to 1.54, above 1.4
// in every first step.
//
// A unit's rows and records sit in LDS.  What bounds the solve is the chain of
// dependent rounds and the memory latencies before and after them, not bytes.  A
// round is one LDS read, a reciprocal, an LDS write and a barrier: 600 to 850
// cycles (0.3 us), the way back a little less than the way up.  By the shader
// clock, cycles of a workgroup (medians):
//   whole cells of 200 to 2000     22.4 k: loads 3.7, tables and children 2.5, 11
//     rounds 7.9, quotients 0.9, 11 rounds back 7.0, voltage 0.7
//   pieces of 1024, first launch   29.5 k: loads 13.0 (two workgroups a CU and
//     all the memory traffic), tables and children 3.8, rounds 9.4, rows out 2.7
//   pieces, last launch            28.9 k: loads 10.7, the trunk's rounds 4.9 + 4.2,
//     hand-over 1.3, own rounds back 7.0, voltage 0.9
// Rounds with no more records than a wave has lanes are run by one wave without
// workgroup barriers.
//
// A cell larger than a unit takes two launches.  In the first, pieces
// eliminate up to their roots and the trunk's rows are assembled (the only
// reads of other units' v).  In the second, every piece solves its cell's
// trunk again for itself, with the piece roots' rows as ghost leaves (a
// trunk of a cell cut at 1024 nodes has at most a few hundred rows, and
// solving it in each piece takes a launch less than solving it once), then
// walks its own rounds backwards; the cell's first piece also writes the
// trunk's v.  Trunks that do not fit beside a piece take a launch of their
// own in between, in LDS or, if they are larger than that, with their rows
// in global memory.
//
// Solve of 64 cells of 200 to 20 000 compartments (369 k in all): 34.5 us a step,
// where elimination by heights in three launches took 88; of 6 cells of 200 to
// 2000 (3.4 k): 12.8 us, where it took 48.
// A row: L, T, U and S side by side, 32 bytes; of an eliminated row with a child
// left N in place of S.
typedef double f64x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f64x2 row_lt(const double *rows, int i) { return *(const f64x2 *)(rows + 4 * (size_t)i); }
__device__ __forceinline__ f64x2 row_us(const double *rows, int i) { return *(const f64x2 *)(rows + 4 * (size_t)i + 2); }
__device__ __forceinline__ void set_lt(double *rows, int i, double l, double t) {
    *(f64x2 *)(rows + 4 * (size_t)i) = f64x2{l, t};
}
__device__ __forceinline__ void set_us(double *rows, int i, double u, double s) {
    *(f64x2 *)(rows + 4 * (size_t)i + 2) = f64x2{u, s};
}
enum { kL = 0, kT = 1, kU = 2, kS = 3 };
__device__ __forceinline__ double &row_at(double *rows, int i, int k) { return rows[4 * (size_t)i + k]; }
struct TreeRecs {
    const char *children, *more, *kid, *fold, *elim;
    const int *rf, *re;
    int nr;
};
constexpr int kBatch = 2;   // loop iterations whose loads are issued together
constexpr int kRowsMax = 3; // rows of a unit in LDS for each thread (kCableLdsUnitMax of 1024)
// What the first kBatch rows of a thread keep from the assembly for the
// voltage update.
struct TreeKeep {
    int n[kBatch], src[kBatch];
    double v[kBatch];
};

// Workgroup barrier for phases that share data only through LDS: it waits
// for LDS traffic alone, so global loads issued before it stay in flight
// across it.  Rows in global memory need the full barrier, whose fence also
// orders global memory operations within the workgroup.
template <bool LDS> __device__ __forceinline__ void tree_barrier() {
    if constexpr (LDS) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    } else {
        __syncthreads();
    }
}
// Orders one wave's own LDS accesses (the hardware keeps their order; the
// compiler must not move them).
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Copies `bytes` (a multiple of 16, both ends aligned to 16) into LDS without
// passing through registers: nothing waits for the copy before tree_copied().
__device__ __forceinline__ void tree_copy(char *dst, const void *src, int bytes) {
    const int lane = (int)(threadIdx.x & 63), step = (int)(blockDim.x >> 6) * 1024;
    for (int o = uni((int)(threadIdx.x >> 6)) * 1024; o < bytes; o += step)
        if (o + 16 * lane < bytes)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)((const char *)src + o + 16 * lane),
                (__attribute__((address_space(3))) void *)(dst + o), 16, 0, 0);
}
// This wave's copies are in LDS (a barrier makes all waves' so).
__device__ __forceinline__ void tree_copied() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A unit's tables at `at`, which stands for the block's byte `from`.
__device__ __forceinline__ TreeRecs tree_recs(const TreeUnit &u, const char *at, int from) {
    const char *b = at - from;
    return TreeRecs{b, b + u.o_more, b + u.o_kid, b + u.o_fold, b + u.o_elim, (const int *)(b + u.o_rf), (const int *)(b + u.o_re), u.nr};
}
__device__ __forceinline__ double *tree_rows(char *lds, int np) {
    double *rows = (double *)lds;
    if (threadIdx.x == 0) {
        set_lt(rows, np, 0.0, 0.0);
        set_us(rows, np, 0.0, 1.0);
    }
    return rows;
}

// The rows of a list, of which the next entry is read ahead (an entry follows the
// last list).
template <bool LDS> struct TreeList {
    const char *more;
    int m;   // -1 at its end
    unsigned e;
    __device__ __forceinline__ TreeList(const TreeRecs &rc, int first) : more(rc.more), m(first), e(first >= 0 ? at(first) : 0u) {}
    __device__ __forceinline__ unsigned at(int i) const {
        return LDS ? ((const unsigned short *)more)[i] : ((const unsigned *)more)[i];
    }
    __device__ __forceinline__ int next() {
        const unsigned last = LDS ? 0x8000u : kMoreLast, x = e;
        e = at(m + 1);
        m = (x & last) ? -1 : m + 1;
        return (int)(LDS ? x & 0xfffu : x & ~kMoreLast);
    }
};
// First child of a row and the list of the others, -1 without.
template <bool LDS> __device__ __forceinline__ void children_of(const TreeRecs &rc, int i, int &ch, int &m) {
    if constexpr (LDS) {
        const unsigned x = ((const unsigned *)rc.children)[i];
        ch = (int)(x & 0xfff);
        if (ch == kNoRow) ch = -1;
        m = (x >> 12) == kChildNone ? -1 : (int)(x >> 12);
    } else {
        const int2 x = ((const int2 *)rc.children)[i];
        ch = x.x;
        m = x.y;
    }
}

// Folds the eliminated neighbours of one surviving row.  All neighbours are read
// before any is used, what the reciprocals need first: the chain through a round
// is one LDS read, one reciprocal and one LDS write.  N of its eliminated parent,
// the row's old coupling, has its place where the parent's S is until the round
// ends: it is returned and written in the next one (without a parent: S of the row
// that stands for it, as it is).
struct TreeNext {
    int p;
    double n;
};
__device__ __forceinline__ void put_next(double *r, const TreeNext &x) { row_at(r, x.p, kS) = x.n; }
__device__ __forceinline__ TreeNext fold_packed(double *r, const TreeRecs &rc, unsigned long long w, int np) {
    const int t = (int)(w & 0xfff), p = (int)((w >> 12) & 0xfff), c = (int)((w >> 24) & 0xfff);
    const int d = (int)((w >> 36) & 0xfff);
    int m = (int)(w >> 48) == (int)kMoreNone ? -1 : (int)(w >> 48);
    const f64x2 uc = row_us(r, c), ud = row_us(r, d), up = row_us(r, p), ut = row_us(r, t);
    const f64x2 lt = row_lt(r, t), lc = row_lt(r, c), ld = row_lt(r, d), lp = row_lt(r, p);
    const bool has = p != np;
    const double u = has ? ut.x : 0.0;
    const double fc = uc.x * rcp_d(uc.y), fd = ud.x * rcp_d(ud.y), fp = u * rcp_d(up.y);
    double S = fma(-u, fp, fma(-ud.x, fd, fma(-uc.x, fc, ut.y)));
    double L = fma(fp, lp.x, fma(fd, ld.x, fma(fc, lc.x, lt.x)));
    double T = fma(fp, lp.y, fma(fd, ld.y, fma(fc, lc.y, lt.y)));
    for (TreeList<true> more(rc, m); more.m >= 0;) {
        const int i = more.next();
        const f64x2 li = row_lt(r, i), ui = row_us(r, i);
        const double f = ui.x * rcp_d(ui.y);
        S = fma(-ui.x, f, S);
        L = fma(f, li.x, L);
        T = fma(f, li.y, T);
    }
    set_lt(r, t, L, T);
    set_us(r, t, has ? fp * up.x : ut.x, S);
    return TreeNext{p, has ? ut.x : 1.0};
}
// In global memory every N has a place of its own.  The reads of a record apart
// from the rest, so that a thread has two records' in flight.
struct TreeWide {
    int4 w;
    f64x2 lt, ut, lc, uc, lp, up;
};
__device__ __forceinline__ TreeWide read_wide(const double *r, const TreeRecs &rc, int q) {
    TreeWide x;
    x.w = ((const int4 *)rc.fold)[q];
    const int c = x.w.z >= 0 ? x.w.z : x.w.x, p = x.w.y >= 0 ? x.w.y : x.w.x;
    x.lt = row_lt(r, x.w.x);
    x.ut = row_us(r, x.w.x);
    x.lc = row_lt(r, c);
    x.uc = row_us(r, c);
    x.lp = row_lt(r, p);
    x.up = row_us(r, p);
    return x;
}
__device__ __forceinline__ void fold_wide(double *r, double *n, const TreeRecs &rc, const TreeWide &x) {
    const int t = x.w.x, p = x.w.y;
    double L = x.lt.x, T = x.lt.y, U = x.ut.x, S = x.ut.y;
    auto pass = [&](double u, double s, f64x2 l) {
        const double f = u * rcp_d(s);
        S = fma(-u, f, S);
        L = fma(f, l.x, L);
        T = fma(f, l.y, T);
        return f;
    };
    if (x.w.z >= 0) pass(x.uc.x, x.uc.y, x.lc);
    for (TreeList<false> more(rc, x.w.w); more.m >= 0;) {
        const int i = more.next();
        const f64x2 ui = row_us(r, i);
        pass(ui.x, ui.y, row_lt(r, i));
    }
    if (p >= 0) {
        n[p] = U;
        U = pass(U, x.up.y, x.lp) * x.up.x;
    }
    set_lt(r, t, L, T);
    set_us(r, t, U, S);
}

// The boundaries of a unit's rounds, one per lane of every wave (a unit in LDS
// has fewer than 64 rounds), so that a round reads them without a trip to LDS.
__device__ __forceinline__ int tree_bounds(const int *at, int nr) { return at[min((int)(threadIdx.x & 63), nr)]; }
__device__ __forceinline__ int bound_at(int b, int j) { return __builtin_amdgcn_readlane(b, j); }

// All rounds of a unit.  In LDS the next round's record is read before the
// barrier, so that it is there when the round starts.
template <bool LDS> __device__ __forceinline__ void tree_up(double *r, double *n, const TreeRecs &rc, int np) {
    const int tid = (int)threadIdx.x, B = (int)blockDim.x;
    if constexpr (LDS) {
        const unsigned long long *rec = (const unsigned long long *)rc.fold;
        const int bnd = tree_bounds(rc.rf, rc.nr), last = bound_at(bnd, rc.nr);
        const TreeNext none{np, 1.0};
        int j = 0;
        {
            // by all waves, up to two records a thread (kCableLdsUnitMax)
            auto few = [&](int i) { return i == rc.nr || bound_at(bnd, i + 1) - bound_at(bnd, i) <= kTreeWave; };
            TreeNext n1 = none, n2 = none;
            int q = tid;
            unsigned long long w = rec[min(q, max(last - 1, 0))];
            for (; !few(j); ++j) {
                const int hi = bound_at(bnd, j + 1);
                const unsigned long long next = rec[min(hi + tid, last - 1)];
                TreeNext m1 = none, m2 = none;
                if (q < hi) m1 = fold_packed(r, rc, w, np);
                if (q + B < hi) m2 = fold_packed(r, rc, rec[q + B], np);
                put_next(r, n1);
                put_next(r, n2);
                n1 = m1;
                n2 = m2;
                tree_barrier<true>();
                q = hi + tid;
                w = next;
            }
            put_next(r, n1);
            put_next(r, n2);
        }
        if (tid < 64 && j < rc.nr) {
            // by one wave; lanes past a round's records do its last one once more
            auto word = [&](int i) { return rec[min(bound_at(bnd, i) + tid, bound_at(bnd, min(i + 1, rc.nr)) - 1)]; };
            TreeNext n = none;
            unsigned long long w = word(j);
            for (; j < rc.nr; ++j) {
                const unsigned long long next = word(j + 1);
                const TreeNext m = fold_packed(r, rc, w, np);
                put_next(r, n);
                n = m;
                wave_order();
                w = next;
            }
            put_next(r, n);
        }
        tree_barrier<true>();
    } else {
        for (int j = 0; j < rc.nr; ++j) {
            const int hi = uni(rc.rf[j + 1]);
            for (int q = uni(rc.rf[j]) + tid; q < hi; q += 2 * B) {
                const TreeWide x = read_wide(r, rc, q), y = read_wide(r, rc, min(q + B, hi - 1));
                fold_wide(r, n, rc, x);
                if (q + B < hi) fold_wide(r, n, rc, y);
            }
            tree_barrier<false>();
        }
    }
}

// T, U and N become T/S, U/S and N/S, with S the sum of L and the couplings.
template <bool LDS>
__device__ __forceinline__ void tree_quotient(const double *from, double *to, const double *n, const TreeRecs &rc, int i) {
    const f64x2 lt = row_lt(from, i), us = row_us(from, i);
    double x;
    if constexpr (LDS) x = ((const unsigned *)rc.kid)[i >> 5] >> (i & 31) & 1 ? us.y : 0.0;
    else x = n[i];
    const double s = lt.x + (us.x + x), f = rcp_d(s);
    set_lt(to, i, lt.x, fdiv(lt.y, s));
    set_us(to, i, us.x * f, x * f);
}
template <bool LDS> __device__ __forceinline__ void tree_quotients(double *r, const double *n, const TreeRecs &rc, int np) {
    for (int i = (int)threadIdx.x; i < np; i += (int)blockDim.x) tree_quotient<LDS>(r, r, n, rc, i);
    tree_barrier<LDS>();
}

// The rounds backwards: dv of the eliminated rows, in T, from the rows that
// outlived them.  What a round reads of its own rows does not change any more
// and is read a round ahead, its record two rounds ahead: after a barrier only
// the neighbours' dv are read.
template <bool LDS> __device__ __forceinline__ void tree_down(double *r, const TreeRecs &rc) {
    const int tid = (int)threadIdx.x, B = (int)blockDim.x;
    if constexpr (LDS) {
        if (rc.nr == 0) return;
        const unsigned long long *rec = (const unsigned long long *)rc.elim;
        const int bnd = tree_bounds(rc.re, rc.nr), last = bound_at(bnd, rc.nr);
        struct Row {
            int i, p, c;
            double x, u, n;
        };
        auto load = [&](unsigned long long w) {
            Row s;
            s.i = (int)(w & 0xfff);
            s.p = (int)((w >> 12) & 0xfff);
            s.c = (int)((w >> 24) & 0xfff);
            const f64x2 un = row_us(r, s.i);
            s.x = row_at(r, s.i, kT);
            s.u = un.x;
            s.n = un.y;
            return s;
        };
        auto one = [&](const Row &s) {
            row_at(r, s.i, kT) = fma(s.n, row_at(r, s.c, kT), fma(s.u, row_at(r, s.p, kT), s.x));
        };
        auto small = [&](int i) { return bound_at(bnd, i + 1) - bound_at(bnd, i) <= kTreeWave; };
        int j = rc.nr - 1;
        if (tid < 64) {
            // by one wave; lanes past a round's records do its last one once more
            auto word = [&](int i) {
                const int k = max(i, 0);
                return rec[min(bound_at(bnd, k) + tid, bound_at(bnd, k + 1) - 1)];
            };
            int k = j;
            unsigned long long w1 = word(k - 1);
            Row row = load(word(k));
            for (; k >= 0 && small(k); --k) {
                const unsigned long long w2 = word(k - 2);
                const Row next = load(w1);
                one(row);
                wave_order();
                row = next;
                w1 = w2;
            }
        }
        while (j >= 0 && small(j)) --j;
        tree_barrier<true>();
        if (j < 0) return;
        auto word = [&](int i) { return rec[min(bound_at(bnd, max(i, 0)) + tid, last - 1)]; };
        unsigned long long w1 = word(j - 1);
        Row row = load(word(j));
        for (; j >= 0; --j) {
            const int lo = bound_at(bnd, j), hi = bound_at(bnd, j + 1);
            const unsigned long long w2 = word(j - 2);
            const Row next = load(w1);
            if (lo + tid < hi) one(row);
            for (int q = lo + tid + B; q < hi; q += B) one(load(rec[q]));
            tree_barrier<true>();
            row = next;
            w1 = w2;
        }
    } else {
        for (int j = rc.nr - 1; j >= 0; --j) {
            const int hi = uni(rc.re[j + 1]);
            for (int q = uni(rc.re[j]) + tid; q < hi; q += B) {
                const int4 w = ((const int4 *)rc.elim)[q];
                const f64x2 un = row_us(r, w.x);
                double x = fma(un.x, row_at(r, w.y, kT), row_at(r, w.x, kT));
                if (w.z != w.x) x = fma(un.y, row_at(r, w.z, kT), x);
                row_at(r, w.x, kT) = x;
            }
            tree_barrier<false>();
        }
    }
}

// The rows of a unit from this step's v, rhs, d and cm; ghosts (TAKE) bring
// the rows that their pieces handed over.  A row's currents to its children come
// from the children's rows, which leave them where S (in global memory N) will be.
template <bool LDS, bool TAKE>
__device__ __forceinline__ void tree_assemble(const CableDev &c, const NodesDev &nd, const GlobDev &g, double *r, double *N,
                                              const TreeRecs &rc, int p0, int np, TreeKeep &keep) {
    const int tid = (int)threadIdx.x, B = (int)blockDim.x;
    for (int i0 = tid; i0 < np; i0 += kBatch * B) {
        int4 w[kBatch];
        double a[kBatch], gu[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = i0 + k * B;
            if (i < np) {
                w[k] = c.pos[p0 + i];
                a[k] = c.pa[p0 + i];
                gu[k] = c.pu[p0 + i];
            }
        }
        double v[kBatch], vp[kBatch], x[kBatch], y[kBatch], cm[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
            if (i0 + k * B < np) {
                const int n = w[k].x;
                v[k] = nd.v[n];
                vp[k] = nd.v[w[k].y >= 0 ? w[k].y : n];
                if (TAKE && w[k].z >= 0) {
                    const f64x2 lt = row_lt(c.G, w[k].z);
                    y[k] = lt.x;
                    x[k] = lt.y;
                } else {
                    x[k] = nd.rhs[n];
                    y[k] = nd.d[n];
                }
                cm[k] = nd.cm[n];
            }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = i0 + k * B;
            if (i < np) {
                const double f = gu[k] * (vp[k] - v[k]);
                const bool ghost = TAKE && w[k].z >= 0;
                set_lt(r, i, ghost ? y[k] : a[k] * (1e-3 * cm[k] / g.dt + y[k]), ghost ? x[k] : fma(a[k], x[k], f));
                set_us(r, i, gu[k], f);
                if constexpr (!LDS) N[i] = w[k].w == -1 ? f : 0.0;
                if (i0 == tid) {
                    keep.n[k] = w[k].x;
                    keep.src[k] = w[k].z;
                    keep.v[k] = v[k];
                }
            }
        }
    }
    tree_copied();
    tree_barrier<LDS>();
    // T without the currents to the children, and S
    auto own = [&](int i) {
        int ch, m;
        children_of<LDS>(rc, i, ch, m);
        double T = row_at(r, i, kT), S = row_at(r, i, kL) + row_at(r, i, kU);
        TreeList<LDS> more(rc, m);
        while (ch >= 0) {
            S += row_at(r, ch, kU);
            if constexpr (LDS) {
                T -= row_at(r, ch, kS);
            } else {
                T -= N[ch];
                N[ch] = 0.0;
            }
            ch = more.m >= 0 ? more.next() : -1;
        }
        row_at(r, i, kT) = T;
        return S;
    };
    if constexpr (LDS) {
        // a row's S replaces what its parent's thread reads
        double S[kRowsMax];
#pragma unroll
        for (int k = 0; k < kRowsMax; ++k)
            if (tid + k * B < np) S[k] = own(tid + k * B);
        tree_barrier<true>();
#pragma unroll
        for (int k = 0; k < kRowsMax; ++k)
            if (tid + k * B < np) row_at(r, tid + k * B, kS) = S[k];
    } else {
        for (int i = tid; i < np; i += B) row_at(r, i, kS) = own(i);
    }
    tree_barrier<LDS>();
}

// v of the unit's own nodes from dv in T, and spikes; ghosts hand dv to the
// piece's root (HAND).  `r` are the unit's rows, `keep` holds the first rows' nodes and v, which are
// all rows unless the unit has more than kBatch per thread.
template <bool HAND>
__device__ __forceinline__ void tree_voltage(const CableDev &c, const NodesDev &nd, const GlobDev &g, double *r,
                                             int p0, int np, TreeKeep &keep) {
    const int tid = (int)threadIdx.x, B = (int)blockDim.x;
    for (int i0 = tid; i0 < np; i0 += kBatch * B) {
        if (i0 != tid) {
#pragma unroll
            for (int k = 0; k < kBatch; ++k)
                if (i0 + k * B < np) {
                    const int4 w = c.pos[p0 + i0 + k * B];
                    keep.n[k] = w.x;
                    keep.src[k] = w.z;
                    keep.v[k] = nd.v[w.x];
                }
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = i0 + k * B;
            if (i >= np) continue;
            const double dv = row_at(r, i, kT), v0 = keep.v[k];
            if (keep.src[k] >= 0) {
                if (HAND) row_at(c.G, keep.src[k], kT) = dv;
                continue;
            }
            const double v1 = v0 + dv;
            if (v0 < g.vthresh && v1 >= g.vthresh) nd.spikes[keep.n[k]] += 1;
            nd.v[keep.n[k]] = v1;
        }
    }
}

// First launch: whole cells to the end; pieces up to their roots; the rows of
// trunks that pieces solve.
__global__ __launch_bounds__(1024) void k_tree_a(CableDev c, NodesDev nd, GlobDev g) {
    extern __shared__ __align__(16) char tree_lds[];
    const TreeUnit u = c.units_a[blockIdx.x];
    const int tid = (int)threadIdx.x, B = (int)blockDim.x, p0 = u.p0, np = u.np;
    double *r = tree_rows(tree_lds, np);
    char *tab = tree_lds + tree_row_bytes(np);
    tree_copy(tab, c.block + 16 * (size_t)u.block, tree_up_bytes(u.mode, u.bytes, u.o_re, u.o_kid));
    const TreeRecs rc = tree_recs(u, tab, 0);
    TreeKeep keep;
    tree_assemble<true, false>(c, nd, g, r, nullptr, rc, p0, np, keep);
    double *out = c.G + 4 * (size_t)p0;
    if (u.mode == kUnitTop) {
        for (int i = tid; i < np; i += B) {
            const f64x2 lt = row_lt(r, i), us = row_us(r, i);
            set_lt(out, i, lt.x, lt.y);
            set_us(out, i, us.x, us.y);
        }
        return;
    }
    tree_up<true>(r, nullptr, rc, np);
    if (u.mode == kUnitPiece) {
        // a root's row stays as it is, for its trunk
        for (int i = tid; i < np; i += B) {
            tree_quotient<true>(r, out, nullptr, rc, i);
            if (c.pos[p0 + i].w != -1) row_at(out, i, kT) = row_at(r, i, kT);
        }
        return;
    }
    tree_quotients<true>(r, nullptr, rc, np);
    tree_down<true>(r, rc);
    tree_voltage<false>(c, nd, g, r, p0, np, keep);
}

// A trunk on its own.
template <bool LDS>
__global__ __launch_bounds__(1024) void k_tree_top(CableDev c, NodesDev nd, GlobDev g, const TreeUnit *units) {
    extern __shared__ __align__(16) char tree_lds[];
    const TreeUnit u = units[blockIdx.x];
    const char *block = c.block + 16 * (size_t)u.block;
    double *r, *n = nullptr;
    TreeRecs rc;
    if constexpr (LDS) {
        r = tree_rows(tree_lds, u.np);
        char *tab = tree_lds + tree_row_bytes(u.np);
        tree_copy(tab, block, u.bytes);
        rc = tree_recs(u, tab, 0);
    } else {
        r = c.G + 4 * (size_t)u.p0;
        n = c.N + u.p0;
        rc = tree_recs(u, block, 0);
    }
    TreeKeep keep;
    tree_assemble<LDS, true>(c, nd, g, r, n, rc, u.p0, u.np, keep);
    tree_up<LDS>(r, n, rc, u.np);
    tree_quotients<LDS>(r, n, rc, u.np);
    tree_down<LDS>(r, rc);
    tree_voltage<true>(c, nd, g, r, u.p0, u.np, keep);
}

// Last launch: a piece's rows from its roots' dv, which come from the trunk
// solved here or in its own launch; and v of the trunks solved here.
__global__ __launch_bounds__(1024) void k_tree_b(CableDev c, NodesDev nd, GlobDev g) {
    extern __shared__ __align__(16) char tree_lds[];
    const TreeUnit u = c.units_b[2 * blockIdx.x], t = c.units_b[2 * blockIdx.x + 1];
    const int tid = (int)threadIdx.x, B = (int)blockDim.x, p0 = u.p0, np = u.np;
    const bool piece = u.mode == kUnitPiece, trunk = !piece || u.solves_trunk;
    // first rows' nodes, v and (a root's) ghost row
    TreeKeep keep;
    int ghost[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
        const int i = tid + k * B;
        if (i < np) {
            const int4 w = c.pos[p0 + i];
            keep.n[k] = w.x;
            keep.src[k] = w.z;
            ghost[k] = w.w;
        }
    }
    char *at = tree_lds;
    double *x = (double *)at;   // the piece's rows
    TreeRecs rp{};
    if (piece) {
        tree_copy(at, c.G + 4 * (size_t)p0, 32 * np);
        at += tree_row_bytes(np);
        tree_copy(at, c.block + 16 * (size_t)u.block + u.o_re, u.bytes - u.o_re);
        rp = tree_recs(u, at, u.o_re);
        at += u.bytes - u.o_re;
    }
    double *r = nullptr;   // the trunk's
    if (trunk) {
        const int nt = t.np;
        r = tree_rows(at, nt);
        char *tab = at + tree_row_bytes(nt);
        tree_copy(tab, c.block + 16 * (size_t)t.block, t.bytes);
        const TreeRecs rc = tree_recs(t, tab, 0);
        for (int i = tid; i < nt; i += B) {
            const int src = c.pos[t.p0 + i].z;
            const f64x2 lt = row_lt(c.G, src >= 0 ? src : t.p0 + i);
            const f64x2 us = row_us(c.G, t.p0 + i);
            set_lt(r, i, lt.x, lt.y);
            set_us(r, i, us.x, src >= 0 ? lt.x + us.x : us.y);
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
            if (tid + k * B < np) keep.v[k] = nd.v[keep.n[k]];
        tree_copied();
        tree_barrier<true>();
        tree_up<true>(r, nullptr, rc, nt);
        tree_quotients<true>(r, nullptr, rc, nt);
        tree_down<true>(r, rc);
        if (!piece) {
            tree_voltage<false>(c, nd, g, r, p0, nt, keep);
            return;
        }
        for (int i0 = tid; i0 < np; i0 += kBatch * B) {
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int i = i0 + k * B;
                if (i >= np) continue;
                const int gr = i0 == tid ? ghost[k] : c.pos[p0 + i].w;
                if (gr >= 0) row_at(x, i, kT) = row_at(r, gr, kT);
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
            if (tid + k * B < np) keep.v[k] = nd.v[keep.n[k]];
        tree_copied();
    }
    if (tid == 0) row_at(x, np, kT) = 0.0;   // the missing child of a leaf
    tree_barrier<true>();
    tree_down<true>(x, rp);
    tree_voltage<false>(c, nd, g, x, p0, np, keep);
}

hipError_t launch_cable(const CableDev &c, const NodesDev &nd, const GlobDev &g, hipStream_t s) {
    if (c.n_a > 0) k_tree_a<<<c.n_a, c.block_a, c.lds_a, s>>>(c, nd, g);
    if (c.n_top > 0) k_tree_top<true><<<c.n_top, c.block_a, c.lds_top, s>>>(c, nd, g, c.units_top);
    if (c.n_top_g > 0) k_tree_top<false><<<c.n_top_g, 1024, 0, s>>>(c, nd, g, c.units_top_g);
    if (c.n_b > 0) k_tree_b<<<c.n_b, c.block_b, c.lds_b, s>>>(c, nd, g);
    return hipGetLastError();
}

// Per position, from the bound area and g_axial: the conductance to the parent
// and area/100 (1 at a node without edges, whose row needs no scaling: its step
// is then the isolated update's to the last rounding).
__global__ __launch_bounds__(256) void k_cable_coeffs(CableDev c, const double *area) {
    const TreeUnit u = c.units[blockIdx.x];
    const TreeRecs rc = tree_recs(u, c.block + 16 * (size_t)u.block, 0);
    for (int i = (int)threadIdx.x; i < u.np; i += (int)blockDim.x) {
        const int p = u.p0 + i, n = c.pos[p].x;
        const double gu = c.parent[n] >= 0 ? c.g_axial[n] : 0.0;
        int ch, m;
        if (u.wide) children_of<false>(rc, i, ch, m);
        else children_of<true>(rc, i, ch, m);
        c.pu[p] = gu;
        c.pa[p] = ch < 0 && c.parent[n] < 0 ? 1.0 : area[n] * 1e-2;
    }
}

hipError_t launch_cable_coeffs(const CableDev &c, const double *area, hipStream_t s) {
    if (c.n_units > 0) k_cable_coeffs<<<c.n_units, 256, 0, s>>>(c, area);
    return hipGetLastError();
}

hipError_t cable_allow_lds(size_t bytes) {
    const void *fns[] = {(const void *)k_tree_a, (const void *)k_tree_top<true>, (const void *)k_tree_b};
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------- fused path --
// Order-independent node sums.  The waves of a tile add their instances'
// contributions to a node in whatever order they run, and FP64 addition is
// not associative, so floating-point accumulators would make rhs, d and
// every later v, STATE and spike count depend on scheduling and on the
// launch shape.  Each node sum is therefore kept in fixed point, as two
// 64-bit integer words added with integer LDS atomics, which are
// associative.  A contribution x (|x| < 2^20) is split into
// h = round(x 2^23) and l = round((x 2^23 - h) 2^44), |l| <= 2^43, so that
// x = (h 2^44 + l) 2^-67 within half a unit 2^-67 (exactly when
// |x| >= 2^-15, whose last mantissa bit is then at or above 2^-67).  Both roundings use the FP64 adder: adding
// M = 1.5 * 2^52 to y (|y| < 2^51) leaves round(y) in the low bits of the
// sum, and y - ((y + M) - M) is the exact remainder.  With at most 2^19
// contributions per node neither word's sum can overflow, so no carry is
// needed while adding; the flush combines the words and rounds to FP64 once.
// A larger or non-finite contribution raises the kernel's error flag (its
// words are then meaningless, and the step is reported as failed at the next
// mech_sync).  The host rejects workloads with more instances on one node
// (kMaxPerNode).
struct Acc {
    unsigned long long *lo, *hi;
};
__device__ __forceinline__ void fx_zero(Acc a, int j) {
    a.lo[j] = 0ull;
    a.hi[j] = 0ull;
}
__device__ __forceinline__ long long fx_round(double y, double &rem) {
    constexpr double M = 0x1.8p52;
    const double t = y + M;
    rem = y - (t - M);
    return (long long)(__double_as_longlong(t) - __double_as_longlong(M));
}
__device__ __forceinline__ void fx_add(Acc a, int j, double x, int &flag) {
    flag |= fabs(x) < 0x1p20 ? 0 : 1;
    double r;
    const long long h = fx_round(x * 0x1p23, r);
    double r2;
    const long long l = fx_round(r * 0x1p44, r2);
    atomicAdd(a.hi + j, (unsigned long long)h);
    atomicAdd(a.lo + j, (unsigned long long)l);
}
// The total of the two words, rounded once.
__device__ __forceinline__ double fx_get(Acc a, int j) { return fx_total((long long)a.hi[j], (long long)a.lo[j]); }

// LDS per tile node: v and 100/area (two doubles), the rhs and d
// accumulators (four 64-bit words); under the shared calcium ion also the
// node's cai and its calcium current accumulator (three more words).
// One instance's contributions into its node's sums (the synapse's in
// nA and uS, scaled by 100/area into mA/cm2 and S/cm2).
template <int KIND, int PH>
__device__ __forceinline__ void tile_add(int j, double ci, double cg, const double *sc, Acc ar, Acc ad,
                                         int &flag) {
    if (PH & kDoCur) {
        if (KIND == MECH_SYN) {
            ci *= sc[j];
            cg *= sc[j];
        }
        fx_add(ar, j, -ci, flag);
        fx_add(ad, j, cg, flag);
    }
}

// The globals of a kernel whose first argument is FusedArgs, read from the
// argument segment where they are used.  The compiler otherwise loads all of
// them once, runs out of scalar registers over the eight types' code and keeps
// the rest in lanes of vector registers, from where every use is a vector
// instruction.
__device__ __forceinline__ const GlobDev &arg_globals() {
    auto p = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(FusedArgs, g);
    asm volatile("" : "+s"(p));
    return *(const GlobDev *)p;
}

// Instance i of a slot within a tile whose nodes start at nlo.
template <class S, int KIND, int PH, bool NT, bool EXT>
__device__ __forceinline__ void tile_one(const SlotDev &sl, int i, int nlo, const double *vl, const double *sc,
                                         Acc ar, Acc ad, const double *cl, Acc ai, const GlobDev &g,
                                         long long k, bool ion, int &flag) {
    // an identity slot (instance i on node i) needs no index load
    const int j = (sl.identity ? i : ld<NT>(sl.ni + i)) - nlo;
    double ci, cg;
    if (EXT && is_ca_kind(KIND) && ion) {
        double ica;
        ca_shared<S, PH, NT>(sl, i, vl[j], cl[j], g, ci, cg, ica, flag);
        if (PH & kDoCur) fx_add(ai, j, ica, flag);
    } else {
        instance<S, KIND, PH, NT, true>(sl, i, vl[j], g, k, ci, cg, flag);
    }
    tile_add<KIND, PH>(j, ci, cg, sc, ar, ad, flag);
}

// A slot's run of a tile.  `first` is the thread that takes the run's first
// instance: the runs of a tile are dealt to the block's waves one after the
// other, so that no wave is left without work while others have several types
// to do (every run used to start at the first wave).  us per step, before and
// after: 15 k instances of eight types 16.4 -> 11.5, 330 k of five 13.4 -> 12.2,
// 8.3 M of four 141.4 -> 139.7.
template <class S, int KIND, int PH, bool NT, bool EXT>
__device__ __forceinline__ void tile_slot(const SlotDev &sl, int lo, int hi, int first, int nlo, const double *vl,
                                          const double *sc, Acc ar, Acc ad, const double *cl, Acc ai,
                                          const GlobDev &g, long long k, bool ion, int &flag) {
    int t = (int)threadIdx.x - first;
    if (t < 0) t += (int)blockDim.x;
    for (int i = lo + t; i < hi; i += (int)blockDim.x)
        tile_one<S, KIND, PH, NT, EXT>(sl, i, nlo, vl, sc, ar, ad, cl, ai, g, k, ion, flag);
}

// Workgroups are dispatched round-robin over the 8 XCDs (workgroup b runs on
// XCD b mod 8), each with its own L2.  With XCD-contiguous ordering the
// virtual workgroup b processes tile start(x) + b/8 of XCD x = b mod 8, so
// neighbouring tiles, which share the cache lines at their boundaries, sit
// in the same L2.  A bijection of [0, T) for any T.
__device__ __forceinline__ int tile_of(int b, int T, int xcd_order) {
    if (!xcd_order) return b;
    const int x = b & 7, j = b >> 3, q = T >> 3, r = T & 7;
    return x * q + min(x, r) + j;
}

// Every instance of a tile in the phases PH, dealt to the waves as in a pass of
// the phases DEAL (one without a current update leaves pas out).  A macro: as a
// function taking the arguments by reference it cost the FP32 kernel 3 VGPRs
// and the FP64 one 8 % of its speed.
#define MECH_TILE_PASS(PH, DEAL) \
    do { \
        int first = 0; \
        for (int s = 0; s < a.n_slots; ++s) { \
            const SlotDev &sl = a.slot[s]; \
            const int lo = r0[1 + s], hi = r1[1 + s]; \
            switch (sl.kind) { \
            case MECH_PAS: \
                if ((PH) & kDoCur) tile_slot<S, MECH_PAS, (PH), NT, EXT>(sl, lo, hi, first, nlo, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); \
                break; \
            case MECH_HH: tile_slot<S, MECH_HH, (PH), NT, EXT>(sl, lo, hi, first, nlo, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); break; \
            case MECH_IH: tile_slot<S, MECH_IH, (PH), NT, EXT>(sl, lo, hi, first, nlo, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); break; \
            case MECH_CAHVA: tile_slot<S, MECH_CAHVA, (PH), NT, EXT>(sl, lo, hi, first, nlo, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); break; \
            case MECH_SYN: tile_slot<S, MECH_SYN, (PH), NT, EXT>(sl, lo, hi, first, nlo, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); break; \
            case MECH_KMARKOV: tile_slot<S, MECH_KMARKOV, (PH), NT, EXT>(sl, lo, hi, first, nlo, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); break; \
            case MECH_CAPUMP: tile_slot<S, MECH_CAPUMP, (PH), NT, EXT>(sl, lo, hi, first, nlo, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); break; \
            case MECH_CABUF: \
                if constexpr (EXT) tile_slot<S, MECH_CABUF, (PH), NT, EXT>(sl, lo, hi, first, nlo, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); \
                break; \
            default: break; \
            } \
            if (!(sl.kind == MECH_PAS && !((DEAL) & kDoCur))) first += (hi - lo + 63) & ~63; \
            while (first >= (int)blockDim.x) first -= (int)blockDim.x; \
        } \
    } while (0)

// EXT: the extended instantiations, which add the buffered-calcium type and
// the shared calcium ion (a run-time switch there).  They are kept apart so
// that the default instantiations keep their register budget.
template <class S, int PH, int VM, bool NT, bool EXT = false>
__global__ __launch_bounds__(1024) void k_fused(FusedArgs a, int tn) {
    extern __shared__ double lds[];
    unsigned long long *w = (unsigned long long *)lds;
    double *vl = lds, *sc = lds + tn;
    const Acc ar{w + 2 * tn, w + 3 * tn}, ad{w + 4 * tn, w + 5 * tn};
    double *cl = lds + 6 * tn;
    const Acc ai{w + 7 * tn, w + 8 * tn};
    const bool ion = EXT && a.g.shared_ca;
    // middle passes (graphs) count from the device's step counter
    const long long k = PH == (kDoCur | kDoState) ? *a.kdev + a.kofs : a.kbase;
    int flag = 0;
    for (int b = blockIdx.x; b < a.n_tiles; b += gridDim.x) {
        const int t = tile_of(b, a.n_tiles, a.xcd_order);
        const int *r0 = a.tiles + (size_t)t * a.row;
        const int *r1 = r0 + a.row;
        const int nlo = r0[0], nn = r1[0] - nlo;
        for (int j = threadIdx.x; j < nn; j += blockDim.x) {
            vl[j] = a.nd.v[nlo + j];
            if (PH & kDoCur) {
                fx_zero(ar, j);
                fx_zero(ad, j);
                if (a.has_syn) sc[j] = 1e2 / a.nd.area[nlo + j];
                if (ion) {
                    cl[j] = a.nd.cai[nlo + j];
                    fx_zero(ai, j);
                }
            }
        }
        __syncthreads();
        MECH_TILE_PASS(PH, PH);
        if (PH & kDoCur) {
            __syncthreads();
            for (int j = threadIdx.x; j < nn; j += blockDim.x) {
                const int n = nlo + j;
                const double r = fx_get(ar, j), dd = fx_get(ad, j);
                a.nd.rhs[n] = r;
                a.nd.d[n] = dd;
                if (VM == MECH_V_ISOLATED) a.nd.v[n] = isolated_v(a.nd, a.g, n, vl[j], r, dd);
                if (VM == MECH_V_CLAMP) a.nd.v[n] = clamp_v(a.nd, n, (double)(k + 1) * a.g.dt);
                if (ion) {
                    // the node's pool advances with this step's calcium current,
                    // as a cahva instance's own pool does in this pass
                    double c = cl[j];
                    const double ica = fx_get(ai, j);
                    ion_pool(a.g, ica, c);
                    flag |= bad(c);
                    a.nd.cai[n] = c;
                    a.nd.ica[n] = ica;
                }
            }
        }
        __syncthreads();
    }
    if (flag) atomicOr(a.err, 1);
}

// ------------------------------------------- single phases in one launch --
// mech_cur and mech_state for callers that solve for v themselves: every type
// in one launch, where the per-type launches (two for a type with several
// instances on a node, and a fill) cost a small context far more than their
// work.  A step of cur, the caller's solve in two torch calls and state, with
// launches per type / with one each: 15 k instances of eight types 94 / 21 us,
// 100 k of C5's mix 46 / 17, 1 M 62 / 33, 8.3 M 267 / 245.
//
// The current update works on the fused path's node tiles and keeps FP64 sums
// in a fixed order without atomics: instances leave their contributions in
// LDS, then a thread per node adds its node's, type by type in instance order.
// A node with kLongRun or more instances of a type (`crowded` contexts) has that
// run summed beforehand by a wave, every 64th by a lane and the lanes' sums in
// a fixed order: one thread takes 0.1 us for each.  us of a current update with a
// launch per type / a thread a run / this: 2000 synapses on one node 17.5 / 209
// / 16.2, 500 on each of 4000 nodes 39 / 83 / 24.  The line: 64 on each of 20 k
// nodes 28.4 / 24.3 / 25.9, 64 on one node 14.8 / 12.3 / 7.8.
// LDS: per node v and 100/area, then the first contribution of each type
// (kNoFirst: none), per instance the contributions and the tile-local node,
// and a list of the long runs.
constexpr unsigned short kNoFirst = 0xffff;

template <class S, int KIND>
__device__ __forceinline__ void phase_cur_slot(const FusedArgs &a, const SlotDev &sl, int lo, int hi, int first, int at, int nlo,
                                               const double *vl, const double *sc, double *cx, double *cy, double *cz,
                                               unsigned short *nj, unsigned short *start, bool ion, int &flag) {
    int t = (int)threadIdx.x - first;
    if (t < 0) t += (int)blockDim.x;
    for (int i = lo + t; i < hi; i += (int)blockDim.x) {
        const int n = sl.ni[i], j = n - nlo, q = at + i - lo;
        const bool head = i == lo || sl.ni[i - 1] != n;
        double ci, cg, ica = 0.0;
        if (is_ca_kind(KIND) && ion) ca_shared<S, kDoCur>(sl, i, vl[j], a.nd.cai[n], a.g, ci, cg, ica, flag);
        else instance<S, KIND, kDoCur>(sl, i, vl[j], a.g, a.kbase, ci, cg, flag);
        if (KIND == MECH_SYN) {
            ci *= sc[j];
            cg *= sc[j];
        }
        cx[q] = ci;
        cy[q] = cg;
        if (ion) cz[q] = ica;
        nj[q] = (unsigned short)j;
        if (head) start[j] = (unsigned short)q;
    }
}

template <class S, bool CROWDED>
__global__ __launch_bounds__(256) void k_phase_cur(FusedArgs a, int accumulate, int tn, int ti) {
    extern __shared__ double lds[];
    const bool ion = a.g.shared_ca != 0;
    double *vl = lds, *sc = vl + tn, *cx = sc + tn, *cy = cx + ti, *cz = cy + ti;
    unsigned short *nj = (unsigned short *)(ion ? cz + ti : cz), *start = nj + ti;
    const int t = tile_of((int)blockIdx.x, a.n_tiles, a.xcd_order);
    const int *r0 = a.tiles + (size_t)t * a.row;
    const int *r1 = r0 + a.row;
    const int nlo = r0[0], nn = r1[0] - nlo;
    int flag = 0;
    for (int j = threadIdx.x; j < nn; j += blockDim.x) {
        vl[j] = a.nd.v[nlo + j];
        if (a.has_syn) sc[j] = 1e2 / a.nd.area[nlo + j];
        for (int s = 0; s < a.n_slots; ++s) start[s * tn + j] = kNoFirst;
    }
    __syncthreads();
    int first = 0, at = 0;
    for (int s = 0; s < a.n_slots; ++s) {
        const SlotDev &sl = a.slot[s];
        const int lo = r0[1 + s], hi = r1[1 + s];
        unsigned short *st = start + s * tn;
        switch (sl.kind) {
#define MECH_PHASE_CASE(K)                                                                                          \
    case K: phase_cur_slot<S, K>(a, sl, lo, hi, first, at, nlo, vl, sc, cx, cy, cz, nj, st, ion, flag); break;
        MECH_PHASE_CASE(MECH_PAS)
        MECH_PHASE_CASE(MECH_HH)
        MECH_PHASE_CASE(MECH_IH)
        MECH_PHASE_CASE(MECH_CAHVA)
        MECH_PHASE_CASE(MECH_SYN)
        MECH_PHASE_CASE(MECH_KMARKOV)
        MECH_PHASE_CASE(MECH_CAPUMP)
        MECH_PHASE_CASE(MECH_CABUF)
#undef MECH_PHASE_CASE
        default: break;
        }
        at += hi - lo;
        first += (hi - lo + 63) & ~63;
        while (first >= (int)blockDim.x) first -= (int)blockDim.x;
    }
    if constexpr (CROWDED) {
        // each long run's total in its first entry; the second no longer names
        // the node, which ends the run
        int &n_long = *(int *)(start + ((a.n_slots * tn + 1) & ~1));   // ti is a multiple of 4
        unsigned short *list = (unsigned short *)(&n_long + 1);
        if (threadIdx.x == 0) n_long = 0;
        __syncthreads();
        int end = 0;
        for (int s = 0; s < a.n_slots; ++s) {
            end += r1[1 + s] - r0[1 + s];
            for (int j = threadIdx.x; j < nn; j += blockDim.x) {
                const int q = start[s * tn + j] + kLongRun - 1;   // kNoFirst is past every end
                if (q < end && nj[q] == j) list[atomicAdd(&n_long, 1)] = (unsigned short)(s * tn + j);
            }
        }
        __syncthreads();
        const int lane = (int)(threadIdx.x & 63);
        for (int w = (int)(threadIdx.x >> 6); w < n_long; w += (int)(blockDim.x >> 6)) {
            const int s = list[w] / tn, j = list[w] - s * tn, q0 = start[list[w]];
            int stop = 0;
            for (int u = 0; u <= s; ++u) stop += r1[1 + u] - r0[1 + u];
            double x = 0.0, y = 0.0, z = 0.0;
            for (int q = q0 + lane; q < stop && nj[q] == j; q += 64) {
                x += cx[q];
                y += cy[q];
                if (ion) z += cz[q];
            }
            for (int m = 32; m > 0; m >>= 1) {
                x += __shfl_xor(x, m, 64);
                y += __shfl_xor(y, m, 64);
                z += __shfl_xor(z, m, 64);
            }
            if (lane == 0) {
                cx[q0] = x;
                cy[q0] = y;
                if (ion) cz[q0] = z;
                nj[q0 + 1] = kNoFirst;
            }
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < nn; j += blockDim.x) {
        double r = 0.0, d = 0.0, z = 0.0;
        int end = 0;
        for (int s = 0; s < a.n_slots; ++s) {
            end += r1[1 + s] - r0[1 + s];
            const int q0 = start[s * tn + j];
            if (q0 == kNoFirst) continue;
            for (int q = q0; q < end && nj[q] == j; ++q) {
                r -= cx[q];
                d += cy[q];
                if (ion) z += cz[q];
            }
        }
        const int n = nlo + j;
        a.nd.rhs[n] = accumulate ? a.nd.rhs[n] + r : r;
        a.nd.d[n] = accumulate ? a.nd.d[n] + d : d;
        if (ion) a.nd.ica[n] = accumulate ? a.nd.ica[n] + z : z;
    }
    if (flag) atomicOr(a.err, 1);
}

// The state update of every type: blocks of 256 instances, a type's blocks one
// after the other.
template <class S>
__global__ __launch_bounds__(256) void k_phase_state(FusedArgs a) {
    int b = (int)blockIdx.x, s = 0;
    for (; s < a.n_slots; ++s) {
        const int nb = a.slot[s].kind == MECH_PAS ? 0 : (a.slot[s].n + 255) >> 8;
        if (b < nb) break;
        b -= nb;
    }
    if (s == a.n_slots) return;
    const SlotDev &sl = a.slot[s];
    const int i = b * 256 + (int)threadIdx.x;
    if (i >= sl.n) return;
    const double v = a.nd.v[sl.ni[i]];
    double ci, cg, ica;
    int flag = 0;
    if (is_ca_kind(sl.kind) && a.g.shared_ca) {
        ca_shared<S, kDoState>(sl, i, v, 0.0, a.g, ci, cg, ica, flag);
    } else {
        switch (sl.kind) {
#define MECH_PHASE_CASE(K)                                              \
    case K: instance<S, K, kDoState>(sl, i, v, a.g, 0, ci, cg, flag); break;
        MECH_PHASE_CASE(MECH_HH)
        MECH_PHASE_CASE(MECH_IH)
        MECH_PHASE_CASE(MECH_CAHVA)
        MECH_PHASE_CASE(MECH_SYN)
        MECH_PHASE_CASE(MECH_KMARKOV)
        MECH_PHASE_CASE(MECH_CAPUMP)
        MECH_PHASE_CASE(MECH_CABUF)
#undef MECH_PHASE_CASE
        default: break;
        }
    }
    if (flag) atomicOr(a.err, 1);
}

// -------------------------------------------------- several steps a launch --
// A tile's steps in one launch, for contexts whose instance arrays stay in the
// L2s from one step to the next: launches and the reading of the tile's nodes,
// not the arrays, are then most of a step.  Each step is k_fused's, STATEs are
// loaded and stored in every one of them (always by the same thread, so that
// no step waits for another's stores to be visible), the tile's node data
// stays in LDS, and rhs, d, v, spikes and the node ion are written after the
// last step.  A call's first pass (current update alone, from the clamp's
// value in clamp mode) and its last (state update alone) are in the launch too,
// as code of their own: as conditions inside the pass they cost every step 4 %.
// Clamp and isolated modes, whose tiles do not depend on each other.
// us of a 32-step call, a launch a step (replayed from graphs) / the middle
// steps in one launch / all in one: 10 k hh 173 / 98 / 91, 67 k hh+pas in FP32
// 201 / 90 / 84, 67 k of C5's mix in FP32 227 / 126 / 126, 15 k of eight types
// 374 / 268 / 250, 266 k synapses 275 / 159 / 155; of a ten-step call on 1 k
// instances of the mix 165 / 46 / 38.
template <class S, int VM, bool EXT>
__global__ __launch_bounds__(1024) void k_steps(FusedArgs a, int nsteps, int first_pass, int last_pass) {
    extern __shared__ double lds[];
    constexpr int PH = kDoCur | kDoState;
    constexpr bool NT = false;
    const bool ion = EXT && a.g.shared_ca;
    const bool syn = a.has_syn != 0;
    int flag = 0;
    const int t = tile_of((int)blockIdx.x, a.n_tiles, a.xcd_order);
    const int *r0 = a.tiles + (size_t)t * a.row;
    const int *r1 = r0 + a.row;
    const int nlo = r0[0], nn = r1[0] - nlo;
    unsigned long long *w = (unsigned long long *)lds;
    double *vl = lds, *q = lds + 5 * nn;
    const Acc ar{w + nn, w + 2 * nn}, ad{w + 3 * nn, w + 4 * nn};
    double *sc = q;
    if (syn) q += nn;
    double *md = q;   // 1e-3 cm/dt (isolated) or the clamp waveform, 4 per node
    q += (VM == MECH_V_CLAMP ? 4 : 1) * nn;
    double *cl = q;
    const Acc ai{(unsigned long long *)q + nn, (unsigned long long *)q + 2 * nn};
    if (ion) q += 3 * nn;
    int *spk = (int *)q;
    for (int j = threadIdx.x; j < nn; j += blockDim.x) {
        const int n = nlo + j;
        vl[j] = VM == MECH_V_CLAMP && first_pass ? clamp_v(a.nd, n, (double)a.kbase * a.g.dt) : a.nd.v[n];
        fx_zero(ar, j);
        fx_zero(ad, j);
        if (syn) sc[j] = 1e2 / a.nd.area[n];
        if (VM == MECH_V_CLAMP) {
            md[4 * j] = a.nd.c_off[n];
            md[4 * j + 1] = a.nd.c_amp[n];
            md[4 * j + 2] = a.nd.c_freq[n];
            md[4 * j + 3] = a.nd.c_phase[n];
        } else {
            md[j] = 1e-3 * a.nd.cm[n] / a.g.dt;
            spk[j] = 0;
        }
        if (ion) {
            cl[j] = a.nd.cai[n];
            fx_zero(ai, j);
        }
    }
    __syncthreads();
    for (int sub = 0; sub < nsteps; ++sub) {
        const long long k = a.kbase + sub;
        if (first_pass && sub == 0) MECH_TILE_PASS(kDoCur, PH);
        else MECH_TILE_PASS(PH, PH);
        __syncthreads();
        const bool last = sub + 1 == nsteps;
        for (int j = threadIdx.x; j < nn; j += blockDim.x) {
            const int n = nlo + j;
            const double rr = fx_get(ar, j), dd = fx_get(ad, j), v0 = vl[j];
            double v1;
            if (VM == MECH_V_ISOLATED) {
                v1 = v0 + rr / (md[j] + dd);
                if (v0 < a.g.vthresh && v1 >= a.g.vthresh) spk[j] += 1;
            } else {
                const double t1 = (double)(k + 1) * a.g.dt;
                v1 = md[4 * j] + md[4 * j + 1] * sin_d(2.0 * 3.14159265358979323846 * md[4 * j + 2] * t1 * 1e-3 +
                                                     md[4 * j + 3]);
            }
            vl[j] = v1;
            fx_zero(ar, j);
            fx_zero(ad, j);
            if (ion) {
                double c = cl[j];
                const double ica = fx_get(ai, j);
                ion_pool(a.g, ica, c);
                flag |= bad(c);
                cl[j] = c;
                fx_zero(ai, j);
                if (last) {
                    a.nd.cai[n] = c;
                    a.nd.ica[n] = ica;
                }
            }
            if (last) {
                a.nd.rhs[n] = rr;
                a.nd.d[n] = dd;
                a.nd.v[n] = v1;
                if (VM == MECH_V_ISOLATED && spk[j]) a.nd.spikes[n] += spk[j];
            }
        }
        __syncthreads();
    }
    if (last_pass) {
        const long long k = 0;
        MECH_TILE_PASS(kDoState, PH);
    }
    if (flag) atomicOr(a.err, 1);
}

// ---------------------------------------------------- time-fused path --
// One workgroup per tile, as in k_fused, but the tile stays in LDS for
// `nsub` steps: its nodes' v, accumulators and voltage-mode data, and every
// instance array of its instances.  Each step runs the same per-instance
// code (tile_slot and instance, on a slot descriptor that points into LDS),
// then a flush provides v_{k+1}; STATEs go back to memory once, at the end.
// Only modes in which the kernel provides v itself (clamp, isolated) can
// run this way.  The arithmetic of each step is that of k_fused.

// A slot's arrays for n instances of `kind` at p, in the order of
// res_slot_bytes: STATEs, PARAMETERs, ica, the tile-local node index, the
// event stream id.  With a compile-time kind the layout folds to constants.
template <class S>
__device__ __forceinline__ SlotDev res_carve(int kind, int n, char *p) {
    const KindShape ks = kind_shape(kind);
    SlotDev l{};
    l.kind = kind;
    l.n = n;
    l.identity = 0;
#pragma unroll
    for (int j = 0; j < kMaxStates; ++j)
        if (j < ks.n_state) {
            l.st[j] = p;
            p += res_round8((size_t)n * sizeof(S));
        }
#pragma unroll
    for (int j = 0; j < kMaxParams; ++j)
        if (j < ks.n_param) {
            l.par[j] = p;
            p += res_round8((size_t)n * (((ks.param_double >> j) & 1) ? 8 : sizeof(S)));
        }
    if (ks.has_ica) {
        l.ica = p;
        p += res_round8((size_t)n * sizeof(S));
    }
    l.ni = (const int *)p;
    p += res_round8((size_t)n * 4);
    l.gid = ks.has_gid ? (const int *)p : nullptr;
    return l;
}

// Stage a slot's run [lo, lo + n) of the tile into LDS (IN) or write its
// STATEs and ica back (!IN).
template <class S, bool IN>
__device__ __forceinline__ void res_copy(const SlotDev &g, const SlotDev &l, int lo, int n, int nlo) {
    const KindShape ks = kind_shape(g.kind);
    for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) {
        const int gi = lo + i;
#pragma unroll
        for (int j = 0; j < kMaxStates; ++j)
            if (j < ks.n_state) {
                S *a = (S *)g.st[j] + gi, *b = (S *)l.st[j] + i;
                if (IN) *b = *a;
                else *a = *b;
            }
        if (ks.has_ica) {
            S *a = (S *)g.ica + gi, *b = (S *)l.ica + i;
            if (IN) *b = *a;
            else *a = *b;
        }
        if (IN) {
#pragma unroll
            for (int j = 0; j < kMaxParams; ++j)
                if (j < ks.n_param) {
                    if ((ks.param_double >> j) & 1) ((double *)l.par[j])[i] = ((const double *)g.par[j])[gi];
                    else ((S *)l.par[j])[i] = ((const S *)g.par[j])[gi];
                }
            ((int *)l.ni)[i] = (g.identity ? gi : g.ni[gi]) - nlo;
            if (l.gid) ((int *)l.gid)[i] = g.gid ? g.gid[gi] : gi;
        }
    }
}

// One pass over every instance of the staged tile (phases PH at step k).
// The slots' runs are laid end to end, each padded to a whole wave, and the
// block's threads stride over that sequence: every thread gets an equal
// share whatever the mix of types, and every wave works on one type.  A wave
// reads its run's start, LDS offset, count and kind from a table in LDS with
// an entry for every 64 positions (`blk`), or, where a tile leaves no room
// for that, finds its run by comparing its position with the runs' ends and
// takes the run's entry (`tab`; the ends as well from LDS: scalar registers
// are the scarce resource here, and every value kept in them across the loop
// is spilled and reloaded with VALU instructions).
// us per 64 steps, by the runs' ends and by the table: 1 M nodes hh+pas FP32
// 711 and 658, FP64 1041 and 989; 1 M of C5's mix FP32 478 and 436, FP64 726
// and 690 (the ends in scalar registers, or the tile table in memory, were
// slower still).
__device__ __forceinline__ int4 res_run(const int4 *tab, int g) {
    const int4 e0 = tab[kMaxSlots], e1 = tab[kMaxSlots + 1];
    return tab[(g >= e0.x) + (g >= e0.y) + (g >= e0.z) + (g >= e0.w) + (g >= e1.x) + (g >= e1.y) + (g >= e1.z)];
}
template <class S, int PH, bool EXT>
__device__ __forceinline__ void res_pass(const int4 *tab, const int4 *blk, char *inst,
                                         const double *vl, const double *sc, Acc ar, Acc ad, const double *cl,
                                         Acc ai, long long k, bool ion, int &flag) {
    const int total = __builtin_amdgcn_readfirstlane(tab[kMaxSlots + 1].w);
    const int lane = (int)(threadIdx.x & 63);
    for (int g0 = (int)threadIdx.x - lane; g0 < total; g0 += (int)blockDim.x) {
        const int gw = __builtin_amdgcn_readfirstlane(g0);
        const int4 t = blk ? blk[gw >> 6] : res_run(tab, gw);
        const int base = __builtin_amdgcn_readfirstlane(t.x), o = __builtin_amdgcn_readfirstlane(t.y);
        const int n = __builtin_amdgcn_readfirstlane(t.z), kind = __builtin_amdgcn_readfirstlane(t.w);
        const int i = gw - base + lane;
        if (i >= n) continue;
        char *p = inst + o;
        switch (kind) {
#define MECH_RES_CASE(K)                                                                                   \
    case K: tile_one<S, K, PH, false, EXT>(res_carve<S>(K, n, p), i, 0, vl, sc, ar, ad, cl, ai, arg_globals(), k, ion, flag); break;
        case MECH_PAS:
            if (PH & kDoCur)
                tile_one<S, MECH_PAS, PH, false, EXT>(res_carve<S>(MECH_PAS, n, p), i, 0, vl, sc, ar, ad, cl, ai, arg_globals(), k,
                                                      ion, flag);
            break;
        MECH_RES_CASE(MECH_HH)
        MECH_RES_CASE(MECH_IH)
        MECH_RES_CASE(MECH_CAHVA)
        MECH_RES_CASE(MECH_SYN)
        MECH_RES_CASE(MECH_KMARKOV)
        MECH_RES_CASE(MECH_CAPUMP)
#undef MECH_RES_CASE
        case MECH_CABUF:
            if constexpr (EXT)
                tile_one<S, MECH_CABUF, PH, false, EXT>(res_carve<S>(MECH_CABUF, n, p), i, 0, vl, sc, ar, ad, cl, ai,
                                                        arg_globals(), k, ion, flag);
            break;
        default: break;
        }
    }
}

template <class S, int VM, bool EXT>
__global__ __launch_bounds__(1024) void k_resident(FusedArgs a, ResArgs r) {
    extern __shared__ double lds[];
    const bool ion = EXT && a.g.shared_ca;
    const bool syn = a.has_syn != 0;
    int flag = 0;
    for (int b = blockIdx.x; b < a.n_tiles; b += gridDim.x) {
        const int t = tile_of(b, a.n_tiles, a.xcd_order);
        const int *r0 = a.tiles + (size_t)t * a.row;
        const int *r1 = r0 + a.row;
        const int nlo = r0[0], nn = r1[0] - nlo;
        // node region and slot table (res_node_bytes), then the slots' instance arrays
        unsigned long long *w = (unsigned long long *)lds;
        double *vl = lds, *q = lds + 5 * nn;
        const Acc ar{w + nn, w + 2 * nn}, ad{w + 3 * nn, w + 4 * nn};
        double *sc = q;
        if (syn) q += nn;
        double *md = q;   // 1e-3 cm/dt (isolated) or the clamp waveform, 4 per node
        q += (VM == MECH_V_CLAMP ? 4 : 1) * nn;
        double *cl = q;
        const Acc ai{(unsigned long long *)q + nn, (unsigned long long *)q + 2 * nn};
        if (ion) q += 3 * nn;
        int *spk = (int *)q;
        const size_t toff = (((char *)q - (char *)lds) + res_round8(4 * (size_t)nn) + 15) & ~(size_t)15;
        int4 *tab = (int4 *)((char *)lds + toff);
        char *inst = (char *)(tab + kMaxSlots + 2);
        // per slot: start of its run, LDS offset of its arrays, count, kind
        if (threadIdx.x == 0) {
            int pos = 0, bytes = 0;
            int e[2 * 4];
            for (int s = 0; s < kMaxSlots; ++s) {
                const bool on = s < a.n_slots;
                const int n = on ? r1[1 + s] - r0[1 + s] : 0, kind = on ? a.slot[s].kind : -1;
                tab[s] = make_int4(pos, bytes, n, kind);
                pos += (n + 63) & ~63;
                bytes += on ? (int)res_slot_bytes(kind, n, sizeof(S)) : 0;
                e[s] = on ? pos : 0x7fffffff;
            }
            // run ends of slots 0..6, then the total (the last run's end)
            tab[kMaxSlots] = make_int4(e[0], e[1], e[2], e[3]);
            tab[kMaxSlots + 1] = make_int4(e[4], e[5], e[6], pos);
        }
        for (int j = threadIdx.x; j < nn; j += blockDim.x) {
            const int n = nlo + j;
            vl[j] = a.nd.v[n];
            fx_zero(ar, j);
            fx_zero(ad, j);
            if (syn) sc[j] = 1e2 / a.nd.area[n];
            if (VM == MECH_V_CLAMP) {
                md[4 * j] = a.nd.c_off[n];
                md[4 * j + 1] = a.nd.c_amp[n];
                md[4 * j + 2] = a.nd.c_freq[n];
                md[4 * j + 3] = a.nd.c_phase[n];
            } else {
                md[j] = 1e-3 * a.nd.cm[n] / a.g.dt;
            }
            if (ion) {
                cl[j] = a.nd.cai[n];
                fx_zero(ai, j);
            }
            spk[j] = 0;
        }
        {
            char *p = inst;
            for (int s = 0; s < a.n_slots; ++s) {
                const int n = r1[1 + s] - r0[1 + s];
                const SlotDev l = res_carve<S>(a.slot[s].kind, n, p);
                res_copy<S, true>(a.slot[s], l, r0[1 + s], n, nlo);
                p += res_slot_bytes(a.slot[s].kind, n, sizeof(S));
            }
        }
        __syncthreads();
        int4 *blk = r.table ? (int4 *)((char *)lds + r.table) : nullptr;
        if (blk) {
            const int total = tab[kMaxSlots + 1].w;
            for (int q = threadIdx.x; q < total >> 6; q += blockDim.x) blk[q] = res_run(tab, q << 6);
            __syncthreads();
        }
        for (int sub = 0; sub < r.nsub; ++sub) {
            const long long k = r.k0 + sub;
            if (sub == 0 && !r.first_state)
                res_pass<S, kDoCur, EXT>(tab, blk, inst, vl, sc, ar, ad, cl, ai, k, ion, flag);
            else
                res_pass<S, kDoCur | kDoState, EXT>(tab, blk, inst, vl, sc, ar, ad, cl, ai, k, ion, flag);
            __syncthreads();
            // flush: the same voltage provision as k_fused's, from LDS
            const bool last = sub + 1 == r.nsub;
            for (int j = threadIdx.x; j < nn; j += blockDim.x) {
                const int n = nlo + j;
                const double rr = fx_get(ar, j), dd = fx_get(ad, j), v0 = vl[j];
                double v1;
                if (VM == MECH_V_ISOLATED) {
                    v1 = v0 + rr / (md[j] + dd);
                    if (v0 < a.g.vthresh && v1 >= a.g.vthresh) spk[j] += 1;
                } else {
                    const double t1 = (double)(k + 1) * a.g.dt;
                    v1 = md[4 * j] + md[4 * j + 1] * sin_d(2.0 * 3.14159265358979323846 * md[4 * j + 2] * t1 * 1e-3 +
                                                         md[4 * j + 3]);
                }
                vl[j] = v1;
                fx_zero(ar, j);
                fx_zero(ad, j);
                const double ica = ion ? fx_get(ai, j) : 0.0;
                if (ion) {
                    double c = cl[j];
                    ion_pool(a.g, ica, c);
                    flag |= bad(c);
                    cl[j] = c;
                }
                if (last) {
                    a.nd.rhs[n] = rr;
                    a.nd.d[n] = dd;
                    a.nd.v[n] = v1;
                    if (ion) {
                        a.nd.cai[n] = cl[j];
                        a.nd.ica[n] = ica;
                    }
                }
                if (ion) fx_zero(ai, j);
            }
            __syncthreads();
        }
        if (r.last_state) {
            res_pass<S, kDoState, EXT>(tab, blk, inst, vl, sc, ar, ad, cl, ai, r.k0 + r.nsub, ion, flag);
            __syncthreads();
        }
        {
            char *p = inst;
            for (int s = 0; s < a.n_slots; ++s) {
                const int n = r1[1 + s] - r0[1 + s];
                const SlotDev l = res_carve<S>(a.slot[s].kind, n, p);
                res_copy<S, false>(a.slot[s], l, r0[1 + s], n, nlo);
                p += res_slot_bytes(a.slot[s].kind, n, sizeof(S));
            }
        }
        if (VM == MECH_V_ISOLATED)
            for (int j = threadIdx.x; j < nn; j += blockDim.x)
                if (spk[j]) a.nd.spikes[nlo + j] += spk[j];
        __syncthreads();
    }
    if (flag) atomicOr(a.err, 1);
}

// --------------------------------------------------------- HBM probe --
// Streaming probes that set the achievable ceiling the kernels are held to:
// op 0 copy, op 1 read (xor-reduced so the loads stay live), op 2 write,
// op 3 two reads and one write (dst = src_a ^ src_b, the STREAM-triad mix),
// op 4 reads in the even workgroups and writes in the odd ones (the read and
// write streams come from different waves).  Each thread keeps U independent
// accesses of T (16 or 8 bytes) in flight per round; NTL / NTS put the
// non-temporal hint on the loads / stores.  The grid-stride mapping
// interleaves all workgroups over the whole range; `chunked` gives each
// workgroup one contiguous range instead (threads still stride by the
// workgroup, so every wave access stays contiguous).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <class T> __device__ __forceinline__ unsigned fold(T x) {
    unsigned r = 0;
#pragma unroll
    for (int c = 0; c < (int)(sizeof(T) / 4); ++c) r |= x[c];
    return r;
}

template <int OP, int U, bool NTL, bool NTS, class T>
__global__ __launch_bounds__(256) void k_stream(T *__restrict__ dst, const T *__restrict__ src, size_t n,
                                                 int chunked, T *__restrict__ sink) {
    int nb = (int)gridDim.x, b = (int)blockIdx.x;
    bool reads = OP != 2, writes = OP != 1;
    if (OP == 4) {
        reads = (b & 1) == 0;
        writes = !reads;
        nb >>= 1;
        b >>= 1;
    }
    size_t i, stride, end = n;
    if (chunked) {
        const size_t per = (n + (size_t)nb - 1) / (size_t)nb;
        const size_t lo = min(n, per * (size_t)b);
        end = min(n, lo + per);
        i = lo + threadIdx.x;
        stride = blockDim.x;
    } else {
        i = (size_t)b * blockDim.x + threadIdx.x;
        stride = (size_t)nb * blockDim.x;
    }
    T acc = (T)0u;
    if (reads && !writes) {
        for (; i + (U - 1) * stride < end; i += U * stride) {
            T x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = ld<NTL>(src + i + u * stride);
#pragma unroll
            for (int u = 0; u < U; ++u) acc ^= x[u];
        }
        for (; i < end; i += stride) acc ^= ld<NTL>(src + i);
        if (fold(acc) == 0x9E3779B9u) sink[0] = acc;   // practically never; keeps the loads live
    } else if (writes && !reads) {
        for (; i + (U - 1) * stride < end; i += U * stride) {
#pragma unroll
            for (int u = 0; u < U; ++u) st<NTS>(dst + i + u * stride, (T)(unsigned)(i + u));
        }
        for (; i < end; i += stride) st<NTS>(dst + i, (T)(unsigned)i);
    } else {
        for (; i + (U - 1) * stride < end; i += U * stride) {
            T x[U], y[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = ld<NTL>(src + i + u * stride);
            if (OP == 3) {
#pragma unroll
                for (int u = 0; u < U; ++u) y[u] = ld<NTL>(src + n + i + u * stride);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) st<NTS>(dst + i + u * stride, OP == 3 ? (T)(x[u] ^ y[u]) : x[u]);
        }
        for (; i < end; i += stride) {
            const T x = ld<NTL>(src + i);
            st<NTS>(dst + i, OP == 3 ? (T)(x ^ ld<NTL>(src + n + i)) : x);
        }
    }
}

// op 5: seven FP64 arrays of n elements, the shape of one Hodgkin-Huxley
// slot of the fused step: three read and rewritten (the STATEs), four read
// only (the PARAMETERs).  AOS interleaves the arrays in blocks of 256
// elements (element i of array a at ((i / 256) 7 + a) 256 + i % 256), so a
// wave's seven accesses fall in one 14 KiB region instead of seven pages
// n elements apart; n is a multiple of 256 then.
// `mapping`: 0 grid-stride, 1 one contiguous range per workgroup, 2 tiles of
// 2048 elements dealt round-robin to the workgroups (the fused kernel's
// pattern: each workgroup streams its own range, and the ranges in flight at
// one time are neighbours).
template <int U, bool NTL, bool NTS, bool AOS>
__global__ __launch_bounds__(256) void k_rmw7(double *__restrict__ base, size_t n, int mapping) {
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    auto at = [n](int a, size_t j) -> size_t {
        return AOS ? ((j >> 8) * 7 + (size_t)a) * 256 + (j & 255) : (size_t)a * n + j;
    };
    auto one = [&](size_t j) {
        double x[7];
#pragma unroll
        for (int a = 0; a < 7; ++a) x[a] = ld<NTL>(base + at(a, j));
        st<NTS>(base + at(0, j), x[0] * x[3] + x[4]);
        st<NTS>(base + at(1, j), x[1] * x[5] + x[6]);
        st<NTS>(base + at(2, j), x[2] * x[3] + x[6]);
    };
    auto range = [&](size_t i, size_t stride, size_t end) {
        for (; i + (U - 1) * stride < end; i += U * stride) {
            double x[U][7];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int a = 0; a < 7; ++a) x[u][a] = ld<NTL>(base + at(a, i + u * stride));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t j = i + u * stride;
                st<NTS>(base + at(0, j), x[u][0] * x[u][3] + x[u][4]);
                st<NTS>(base + at(1, j), x[u][1] * x[u][5] + x[u][6]);
                st<NTS>(base + at(2, j), x[u][2] * x[u][3] + x[u][6]);
            }
        }
        for (; i < end; i += stride) one(i);
    };
    if (mapping == 2) {
        constexpr size_t T = 2048;
        for (size_t lo = (size_t)b * T; lo < n; lo += (size_t)nb * T) range(lo + threadIdx.x, blockDim.x, min(n, lo + T));
    } else if (mapping == 1) {
        const size_t per = (n + (size_t)nb - 1) / (size_t)nb;
        const size_t lo = min(n, per * (size_t)b);
        range(lo + threadIdx.x, blockDim.x, min(n, lo + per));
    } else {
        range((size_t)b * blockDim.x + threadIdx.x, (size_t)nb * blockDim.x, n);
    }
}

// op 6: twenty FP64 arrays of n elements in four groups of five (two read
// and rewritten, three read only), streamed in tiles of 2048 elements dealt
// round-robin to the workgroups, one group after another within a tile: the
// fused kernel's pattern of several mechanism types per node tile.  TM
// (tile-major) stores each tile's twenty arrays contiguously
// (element j of array a at ((j / 2048) 20 + a) 2048 + j % 2048), so a tile
// is one contiguous range; n is a multiple of 2048.
template <int U, bool NTL, bool NTS, bool TM>
__global__ __launch_bounds__(256) void k_rmw20(double *__restrict__ base, size_t n) {
    constexpr size_t T = 2048;
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    auto at = [n](int a, size_t j) -> size_t {
        return TM ? ((j / T) * 20 + (size_t)a) * T + (j % T) : (size_t)a * n + j;
    };
    for (size_t lo = (size_t)b * T; lo < n; lo += (size_t)nb * T) {
        const size_t end = min(n, lo + T);
#pragma unroll 1
        for (int g = 0; g < 4; ++g) {
            const int a0 = 5 * g;
            size_t i = lo + threadIdx.x;
            for (; i + (U - 1) * blockDim.x < end; i += U * blockDim.x) {
                double x[U][5];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int a = 0; a < 5; ++a) x[u][a] = ld<NTL>(base + at(a0 + a, i + u * blockDim.x));
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const size_t j = i + u * blockDim.x;
                    st<NTS>(base + at(a0, j), x[u][0] * x[u][2] + x[u][3]);
                    st<NTS>(base + at(a0 + 1, j), x[u][1] * x[u][4] + x[u][3]);
                }
            }
            for (; i < end; i += blockDim.x) {
                double x[5];
#pragma unroll
                for (int a = 0; a < 5; ++a) x[a] = ld<NTL>(base + at(a0 + a, i));
                st<NTS>(base + at(a0, i), x[0] * x[2] + x[3]);
                st<NTS>(base + at(a0 + 1, i), x[1] * x[4] + x[3]);
            }
        }
    }
}
template <int U, bool NTL, bool NTS>
static hipError_t rmw20_go(int tm, void *d, size_t bytes, int grid, hipStream_t s) {
    const size_t n = bytes / 160;
    if (tm) k_rmw20<U, NTL, NTS, true><<<grid, 256, 0, s>>>((double *)d, n);
    else k_rmw20<U, NTL, NTS, false><<<grid, 256, 0, s>>>((double *)d, n);
    return hipGetLastError();
}

template <int OP, int U, bool NTL, bool NTS>
static hipError_t stream_go(int wide, void *d, const void *r, size_t bytes, int grid, int chunked, hipStream_t s) {
    if (wide) {
        k_stream<OP, U, NTL, NTS, u32x4><<<grid, 256, 0, s>>>((u32x4 *)d, (const u32x4 *)r, bytes / 16, chunked,
                                                               (u32x4 *)d);
    } else {
        k_stream<OP, U, NTL, NTS, u32x2><<<grid, 256, 0, s>>>((u32x2 *)d, (const u32x2 *)r, bytes / 8, chunked,
                                                               (u32x2 *)d);
    }
    return hipGetLastError();
}
template <int U, bool NTL, bool NTS>
static hipError_t rmw7_go(int aos, void *d, size_t bytes, int grid, int chunked, hipStream_t s) {
    const size_t n = bytes / 56;
    if (aos) k_rmw7<U, NTL, NTS, true><<<grid, 256, 0, s>>>((double *)d, n, chunked);
    else k_rmw7<U, NTL, NTS, false><<<grid, 256, 0, s>>>((double *)d, n, chunked);
    return hipGetLastError();
}
template <int OP, int U>
static hipError_t stream_nt(int flags, void *d, const void *r, size_t bytes, int grid, hipStream_t s) {
    const int wide = !(flags & MECH_PROBE_8B);
    int ch = (flags & MECH_PROBE_CHUNKED) ? 1 : 0;
    if constexpr (OP == 6) {
        const int tm = (flags & MECH_PROBE_AOSOA) ? 1 : 0;
        switch (flags & (MECH_PROBE_NT_LOAD | MECH_PROBE_NT_STORE)) {
        case 0: return rmw20_go<U, false, false>(tm, d, bytes, grid, s);
        case MECH_PROBE_NT_LOAD: return rmw20_go<U, true, false>(tm, d, bytes, grid, s);
        case MECH_PROBE_NT_STORE: return rmw20_go<U, false, true>(tm, d, bytes, grid, s);
        default: return rmw20_go<U, true, true>(tm, d, bytes, grid, s);
        }
    } else if constexpr (OP == 5) {
        const int aos = (flags & MECH_PROBE_AOSOA) ? 1 : 0;
        if (flags & MECH_PROBE_TILED) ch = 2;
        switch (flags & (MECH_PROBE_NT_LOAD | MECH_PROBE_NT_STORE)) {
        case 0: return rmw7_go<U, false, false>(aos, d, bytes, grid, ch, s);
        case MECH_PROBE_NT_LOAD: return rmw7_go<U, true, false>(aos, d, bytes, grid, ch, s);
        case MECH_PROBE_NT_STORE: return rmw7_go<U, false, true>(aos, d, bytes, grid, ch, s);
        default: return rmw7_go<U, true, true>(aos, d, bytes, grid, ch, s);
        }
    } else {
        switch (flags & (MECH_PROBE_NT_LOAD | MECH_PROBE_NT_STORE)) {
        case 0: return stream_go<OP, U, false, false>(wide, d, r, bytes, grid, ch, s);
        case MECH_PROBE_NT_LOAD: return stream_go<OP, U, true, false>(wide, d, r, bytes, grid, ch, s);
        case MECH_PROBE_NT_STORE: return stream_go<OP, U, false, true>(wide, d, r, bytes, grid, ch, s);
        default: return stream_go<OP, U, true, true>(wide, d, r, bytes, grid, ch, s);
        }
    }
}
template <int OP>
static hipError_t stream_u(int unroll, int flags, void *d, const void *r, size_t bytes, int grid, hipStream_t s) {
    switch (unroll) {
    case 1: return stream_nt<OP, 1>(flags, d, r, bytes, grid, s);
    case 2: return stream_nt<OP, 2>(flags, d, r, bytes, grid, s);
    case 4: return stream_nt<OP, 4>(flags, d, r, bytes, grid, s);
    case 8: return stream_nt<OP, 8>(flags, d, r, bytes, grid, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_stream(int op, int unroll, int flags, void *dst, const void *src, size_t bytes, int grid,
                         hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    switch (op) {
    case 0: return stream_u<0>(unroll, flags, dst, src, bytes, grid, s);
    case 1: return stream_u<1>(unroll, flags, dst, src, bytes, grid, s);
    case 2: return stream_u<2>(unroll, flags, dst, src, bytes, grid, s);
    case 3: return stream_u<3>(unroll, flags, dst, src, bytes, grid, s);
    case 4: return stream_u<4>(unroll, flags, dst, src, bytes, grid, s);
    case 5: return stream_u<5>(unroll, flags, dst, src, bytes, grid, s);
    case 6: return stream_u<6>(unroll, flags, dst, src, bytes, grid, s);
    default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------ launchers --
static inline int blocks(int n, int b) { return (n + b - 1) / b; }

hipError_t launch_fill(double *a, double *b, int n, hipStream_t s) {
    if (n > 0) k_fill<<<blocks(n, 256), 256, 0, s>>>(a, b, n);
    return hipGetLastError();
}
hipError_t launch_fill_int(int *a, int n, hipStream_t s) {
    if (n > 0) k_fill_int<<<blocks(n, 256), 256, 0, s>>>(a, n);
    return hipGetLastError();
}
hipError_t launch_set_k(long long *kdev, long long value, hipStream_t s) {
    k_set_k<<<1, 64, 0, s>>>(kdev, value);
    return hipGetLastError();
}
hipError_t launch_bump_k(long long *kdev, long long by, hipStream_t s) {
    k_bump_k<<<1, 64, 0, s>>>(kdev, by);
    return hipGetLastError();
}
hipError_t launch_vclamp(const NodesDev &nd, double t, hipStream_t s) {
    if (nd.n_nodes > 0) k_vclamp<<<blocks(nd.n_nodes, 256), 256, 0, s>>>(nd, t);
    return hipGetLastError();
}
hipError_t launch_visolated(const NodesDev &nd, const GlobDev &g, hipStream_t s) {
    if (nd.n_nodes > 0) k_visolated<<<blocks(nd.n_nodes, 256), 256, 0, s>>>(nd, g);
    return hipGetLastError();
}

template <class S>
static hipError_t init_t(const PlainArgs &a, hipStream_t s) {
    const int gr = blocks(a.slot.n, 256);
    switch (a.slot.kind) {
    case MECH_HH: k_init<S, MECH_HH><<<gr, 256, 0, s>>>(a); break;
    case MECH_IH: k_init<S, MECH_IH><<<gr, 256, 0, s>>>(a); break;
    case MECH_CAHVA: k_init<S, MECH_CAHVA><<<gr, 256, 0, s>>>(a); break;
    case MECH_SYN: k_init<S, MECH_SYN><<<gr, 256, 0, s>>>(a); break;
    case MECH_KMARKOV: k_init<S, MECH_KMARKOV><<<gr, 256, 0, s>>>(a); break;
    case MECH_CAPUMP: k_init<S, MECH_CAPUMP><<<gr, 256, 0, s>>>(a); break;
    case MECH_CABUF: k_init<S, MECH_CABUF><<<gr, 256, 0, s>>>(a); break;
    default: break;
    }
    return hipGetLastError();
}
hipError_t launch_init(bool fp32, const PlainArgs &a, hipStream_t s) {
    if (a.slot.n == 0) return hipSuccess;
    return fp32 ? init_t<float>(a, s) : init_t<double>(a, s);
}

template <class S>
static hipError_t cur_t(const PlainArgs &a, hipStream_t s) {
    const int gr = blocks(a.slot.n, 256);
    switch (a.slot.kind) {
    case MECH_PAS: k_plain_cur<S, MECH_PAS><<<gr, 256, 0, s>>>(a); break;
    case MECH_HH: k_plain_cur<S, MECH_HH><<<gr, 256, 0, s>>>(a); break;
    case MECH_IH: k_plain_cur<S, MECH_IH><<<gr, 256, 0, s>>>(a); break;
    case MECH_CAHVA: k_plain_cur<S, MECH_CAHVA><<<gr, 256, 0, s>>>(a); break;
    case MECH_SYN: k_plain_cur<S, MECH_SYN><<<gr, 256, 0, s>>>(a); break;
    case MECH_KMARKOV: k_plain_cur<S, MECH_KMARKOV><<<gr, 256, 0, s>>>(a); break;
    case MECH_CAPUMP: k_plain_cur<S, MECH_CAPUMP><<<gr, 256, 0, s>>>(a); break;
    case MECH_CABUF: k_plain_cur<S, MECH_CABUF><<<gr, 256, 0, s>>>(a); break;
    default: break;
    }
    return hipGetLastError();
}
hipError_t launch_plain_cur(bool fp32, const PlainArgs &a, hipStream_t s) {
    if (a.slot.n == 0) return hipSuccess;
    const hipError_t e = fp32 ? cur_t<float>(a, s) : cur_t<double>(a, s);
    if (e != hipSuccess || a.slot.identity || a.atomic_scatter || !a.crossing) return e;
    const int n_chunks = (a.slot.n + 63) / 64;
    k_plain_carry<<<blocks(n_chunks, 256), 256, 0, s>>>(a, n_chunks, a.g.shared_ca ? 1 : 0);
    return hipGetLastError();
}

template <class S>
static hipError_t state_t(const PlainArgs &a, hipStream_t s) {
    const int gr = blocks(a.slot.n, 256);
    switch (a.slot.kind) {
    case MECH_HH: k_plain_state<S, MECH_HH><<<gr, 256, 0, s>>>(a); break;
    case MECH_IH: k_plain_state<S, MECH_IH><<<gr, 256, 0, s>>>(a); break;
    case MECH_CAHVA: k_plain_state<S, MECH_CAHVA><<<gr, 256, 0, s>>>(a); break;
    case MECH_SYN: k_plain_state<S, MECH_SYN><<<gr, 256, 0, s>>>(a); break;
    case MECH_KMARKOV: k_plain_state<S, MECH_KMARKOV><<<gr, 256, 0, s>>>(a); break;
    case MECH_CAPUMP: k_plain_state<S, MECH_CAPUMP><<<gr, 256, 0, s>>>(a); break;
    case MECH_CABUF: k_plain_state<S, MECH_CABUF><<<gr, 256, 0, s>>>(a); break;
    default: break;  // pas has no STATE
    }
    return hipGetLastError();
}
hipError_t launch_plain_state(bool fp32, const PlainArgs &a, hipStream_t s) {
    if (a.slot.n == 0) return hipSuccess;
    return fp32 ? state_t<float>(a, s) : state_t<double>(a, s);
}

template <class S, int PH, bool NT, bool EXT>
static hipError_t fused_vm(int vmode, const FusedArgs &a, int grid, int block, size_t lds, int tn,
                           hipStream_t s) {
    switch (vmode) {
    case MECH_V_CLAMP: k_fused<S, PH, MECH_V_CLAMP, NT, EXT><<<grid, block, lds, s>>>(a, tn); break;
    case MECH_V_ISOLATED: k_fused<S, PH, MECH_V_ISOLATED, NT, EXT><<<grid, block, lds, s>>>(a, tn); break;
    default: k_fused<S, PH, MECH_V_EXTERNAL, NT, EXT><<<grid, block, lds, s>>>(a, tn); break;
    }
    return hipGetLastError();
}
template <class S, bool NT, bool EXT = false>
static hipError_t fused_t(int phases, int vmode, const FusedArgs &a, int grid, int block, size_t lds, int tn,
                          hipStream_t s) {
    switch (phases) {
    case kDoCur: return fused_vm<S, kDoCur, NT, EXT>(vmode, a, grid, block, lds, tn, s);
    case kDoState:
        k_fused<S, kDoState, MECH_V_EXTERNAL, NT, EXT><<<grid, block, lds, s>>>(a, tn);
        return hipGetLastError();
    default: return fused_vm<S, kDoCur | kDoState, NT, EXT>(vmode, a, grid, block, lds, tn, s);
    }
}
size_t phase_lds_bytes(int tile_nodes, int tile_instances, int n_slots, bool ion, bool crowded) {
    return 16 * (size_t)tile_nodes + (ion ? 26 : 18) * (size_t)tile_instances + 2 * (size_t)n_slots * tile_nodes +
           (crowded ? 6 + 2 * ((size_t)tile_instances / kLongRun) : 0);
}
hipError_t launch_phase_cur(bool fp32, const FusedArgs &a, int accumulate, bool crowded, int tn, int ti,
                            hipStream_t s) {
    if (a.n_tiles == 0) return hipSuccess;
    const size_t lds = phase_lds_bytes(tn, ti, a.n_slots, a.g.shared_ca != 0, crowded);
    auto go = [&](auto kernel) {
        kernel<<<a.n_tiles, 256, lds, s>>>(a, accumulate, tn, ti);
        return hipGetLastError();
    };
    if (crowded) return go(fp32 ? k_phase_cur<float, true> : k_phase_cur<double, true>);
    return go(fp32 ? k_phase_cur<float, false> : k_phase_cur<double, false>);
}
hipError_t launch_phase_state(bool fp32, const FusedArgs &a, hipStream_t s) {
    long long nb = 0;
    for (int i = 0; i < a.n_slots; ++i)
        if (a.slot[i].kind != MECH_PAS) nb += (a.slot[i].n + 255) / 256;
    if (nb == 0) return hipSuccess;
    if (fp32) k_phase_state<float><<<(unsigned)nb, 256, 0, s>>>(a);
    else k_phase_state<double><<<(unsigned)nb, 256, 0, s>>>(a);
    return hipGetLastError();
}

size_t steps_lds_bytes(int tile_nodes, int vmode, bool syn, bool ion) {
    return (size_t)tile_nodes * (8 * res_node_doubles(vmode, syn, ion) + 4);
}
template <class S, bool EXT>
static hipError_t steps_t(int vmode, const FusedArgs &a, int n, int first, int last, int block, size_t lds,
                          hipStream_t s) {
    if (vmode == MECH_V_CLAMP) k_steps<S, MECH_V_CLAMP, EXT><<<a.n_tiles, block, lds, s>>>(a, n, first, last);
    else k_steps<S, MECH_V_ISOLATED, EXT><<<a.n_tiles, block, lds, s>>>(a, n, first, last);
    return hipGetLastError();
}
hipError_t launch_steps(bool fp32, int vmode, const FusedArgs &a, int nsteps, int first, int last, int block, int tn,
                        hipStream_t s) {
    if (a.n_tiles == 0) return hipSuccess;
    const bool ext = a.g.shared_ca || a.has_ext;
    const size_t lds = steps_lds_bytes(tn, vmode, a.has_syn != 0, a.g.shared_ca != 0);
    if (ext)
        return fp32 ? steps_t<float, true>(vmode, a, nsteps, first, last, block, lds, s)
                    : steps_t<double, true>(vmode, a, nsteps, first, last, block, lds, s);
    return fp32 ? steps_t<float, false>(vmode, a, nsteps, first, last, block, lds, s)
                : steps_t<double, false>(vmode, a, nsteps, first, last, block, lds, s);
}

size_t fused_lds_bytes(int tile_nodes, bool ion) { return (ion ? 9 : 6) * 8 * (size_t)tile_nodes; }

// Lets every fused instantiation take up to `bytes` of dynamic LDS.
hipError_t fused_allow_lds(size_t bytes) {
    const int b = (int)bytes;
    const void *fns[] = {
#define MECH_FUSED_FNS(S, NT, EXT)                                                                              \
    (const void *)k_fused<S, kDoState, MECH_V_EXTERNAL, NT, EXT>,                                                 \
        (const void *)k_fused<S, kDoCur, MECH_V_EXTERNAL, NT, EXT>,                                               \
        (const void *)k_fused<S, kDoCur, MECH_V_CLAMP, NT, EXT>,                                                  \
        (const void *)k_fused<S, kDoCur, MECH_V_ISOLATED, NT, EXT>,                                               \
        (const void *)k_fused<S, kDoCur | kDoState, MECH_V_EXTERNAL, NT, EXT>,                                    \
        (const void *)k_fused<S, kDoCur | kDoState, MECH_V_CLAMP, NT, EXT>,                                       \
        (const void *)k_fused<S, kDoCur | kDoState, MECH_V_ISOLATED, NT, EXT>
        MECH_FUSED_FNS(double, false, false), MECH_FUSED_FNS(float, false, false),
        MECH_FUSED_FNS(double, true, false), MECH_FUSED_FNS(float, true, false),
        MECH_FUSED_FNS(double, false, true), MECH_FUSED_FNS(float, false, true),
#undef MECH_FUSED_FNS
        (const void *)k_steps<double, MECH_V_CLAMP, false>, (const void *)k_steps<double, MECH_V_CLAMP, true>,
        (const void *)k_steps<double, MECH_V_ISOLATED, false>, (const void *)k_steps<double, MECH_V_ISOLATED, true>,
        (const void *)k_steps<float, MECH_V_CLAMP, false>, (const void *)k_steps<float, MECH_V_CLAMP, true>,
        (const void *)k_steps<float, MECH_V_ISOLATED, false>, (const void *)k_steps<float, MECH_V_ISOLATED, true>
    };
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, b);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <class S, bool EXT>
static hipError_t resident_t(int vmode, const FusedArgs &a, const ResArgs &r, int grid, int block, size_t lds,
                             hipStream_t s) {
    if (vmode == MECH_V_CLAMP) k_resident<S, MECH_V_CLAMP, EXT><<<grid, block, lds, s>>>(a, r);
    else k_resident<S, MECH_V_ISOLATED, EXT><<<grid, block, lds, s>>>(a, r);
    return hipGetLastError();
}
hipError_t launch_resident(bool fp32, int vmode, const FusedArgs &a, const ResArgs &r, int grid, int block,
                           size_t lds_bytes, hipStream_t s) {
    if (a.n_tiles == 0 || grid == 0 || r.nsub <= 0) return hipSuccess;
    if (vmode != MECH_V_CLAMP && vmode != MECH_V_ISOLATED) return hipErrorInvalidValue;
    if (a.g.shared_ca || a.has_ext)
        return fp32 ? resident_t<float, true>(vmode, a, r, grid, block, lds_bytes, s)
                    : resident_t<double, true>(vmode, a, r, grid, block, lds_bytes, s);
    return fp32 ? resident_t<float, false>(vmode, a, r, grid, block, lds_bytes, s)
                : resident_t<double, false>(vmode, a, r, grid, block, lds_bytes, s);
}
hipError_t resident_allow_lds(size_t bytes) {
    const int b = (int)bytes;
    const void *fns[] = {
#define MECH_RES_FNS(S)                                                                                            \
    (const void *)k_resident<S, MECH_V_CLAMP, false>, (const void *)k_resident<S, MECH_V_ISOLATED, false>,        \
        (const void *)k_resident<S, MECH_V_CLAMP, true>, (const void *)k_resident<S, MECH_V_ISOLATED, true>
        MECH_RES_FNS(double), MECH_RES_FNS(float)
#undef MECH_RES_FNS
    };
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, b);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_ion_pool(const NodesDev &nd, const GlobDev &g, int *err, hipStream_t s) {
    if (nd.n_nodes > 0) k_ion_pool<<<blocks(nd.n_nodes, 256), 256, 0, s>>>(nd, g, err);
    return hipGetLastError();
}
hipError_t launch_ion_init(const NodesDev &nd, const GlobDev &g, hipStream_t s) {
    if (nd.n_nodes > 0) k_ion_init<<<blocks(nd.n_nodes, 256), 256, 0, s>>>(nd, g.cai0);
    return hipGetLastError();
}

hipError_t launch_fused(bool fp32, int phases, int vmode, const FusedArgs &a, int grid, int block, int tn,
                        hipStream_t s) {
    if (a.n_tiles == 0 || grid == 0) return hipSuccess;
    const size_t lds_bytes = fused_lds_bytes(tn, a.g.shared_ca != 0);
    // the extended set (shared calcium ion, cabuf) has temporal-hint
    // instantiations only
    if (a.g.shared_ca || a.has_ext)
        return fp32 ? fused_t<float, false, true>(phases, vmode, a, grid, block, lds_bytes, tn, s)
                    : fused_t<double, false, true>(phases, vmode, a, grid, block, lds_bytes, tn, s);
    if (a.nontemporal)
        return fp32 ? fused_t<float, true>(phases, vmode, a, grid, block, lds_bytes, tn, s)
                    : fused_t<double, true>(phases, vmode, a, grid, block, lds_bytes, tn, s);
    return fp32 ? fused_t<float, false>(phases, vmode, a, grid, block, lds_bytes, tn, s)
                : fused_t<double, false>(phases, vmode, a, grid, block, lds_bytes, tn, s);
}

}  // namespace mech
