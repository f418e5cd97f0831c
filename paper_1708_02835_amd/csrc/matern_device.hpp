// Device evaluation of the Matérn covariance, Sec. 2.2 Eq. (2):
//   C(r; θ) = θ1 / (2^(θ3-1) Γ(θ3)) · (r/θ2)^θ3 · K_θ3(r/θ2),  C(0) = θ1.
//
// K_ν for arbitrary real ν > 0 follows Temme's method (N. M. Temme, J. Comput.
// Phys. 19 (1975) 324-337): write ν = μ + nl with |μ| <= 1/2, obtain K_μ and
// K_μ+1, then recur upward in order with K_a+1 = K_a-1 + (2a/x) K_a, which is
// stable for K.
//   * x <= 2: Temme's power series in (x/2)^2, whose leading coefficient uses
//     Γ1(μ) = (1/Γ(1-μ) - 1/Γ(1+μ)) / (2μ) and Γ2(μ) = (1/Γ(1-μ) + 1/Γ(1+μ)) / 2,
//     both taken from the Taylor series of 1/Γ(1+z) so that μ -> 0 has no
//     cancellation.
//   * x > 2: the representation K_μ(x) = sqrt(π) (2x)^μ e^-x U(μ+1/2, 2μ+1, 2x)
//     with the confluent hypergeometric function U.  The values z_k =
//     U(μ+1/2+k, 2μ+1, 2x) obey z_k-1 = 2(k+x) z_k - ((k+1/2)^2 - μ^2) z_k+1,
//     are the minimal solution of that recurrence (so Miller's backward
//     recurrence finds their ratios), and satisfy the normalisation
//     Σ_k [(μ+1/2)_k (1/2-μ)_k / k!] z_k = (2x)^-(μ+1/2), which follows from the
//     Laplace integral of U and the binomial series.  Hence
//     K_μ = sqrt(π/(2x)) e^-x / S with S = Σ_k c_k z_k / z_0, and
//     K_μ+1 = K_μ (μ + 1/2 + x - (1/4 - μ^2) z_1/z_0) / x.
//     The recurrence depth needed for binary64 accuracy falls like 1/x.
// Half-integer smoothness 1/2, 3/2, 5/2 uses the elementary closed forms
// (Sec. 2.2 names the exponential model for θ3 = 1/2).
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"
#include "rgamma_table.hpp"

namespace gl {

struct MaternSetup {
    double theta1, theta2, nu;
    double mu;     // ν - nl, |μ| <= 1/2
    double pref;   // θ1 · 2^(1-ν) / Γ(ν)
    double g1, g2; // Temme Γ1(μ), Γ2(μ)
    double hgp;    // ½ Γ(1+μ)
    double hgm;    // ½ Γ(1-μ)
    double fact;   // μπ / sin(μπ)
    int nl;        // number of upward recurrence steps
    int kind;      // 0: general ν, 1: ν = 1/2, 2: ν = 3/2, 3: ν = 5/2
};

// 1/x for normal x well inside the exponent range: the hardware reciprocal
// (about 2^-23) with one third-order correction, four instructions where the
// division with its scaling takes ten.
__host__ __device__ inline double plain_rcp(double x)
{
#ifdef __HIP_DEVICE_COMPILE__
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
#else
    return 1.0 / x;
#endif
}

// The functions below write their fused operations out and allow no others:
// left to the compiler, either product of a sum of two may be the one that is
// not rounded, and kernels that should agree bit for bit would not.

// Zero, as a value the compiler knows nothing about: an index with it keeps
// the constants of the loops below in LDS.  They do not change from element
// to element, and hoisted out of a caller's loop they would take hundreds of
// registers.
__host__ __device__ inline int opaque_zero()
{
    int z = 0;
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+v"(z));
#endif
    return z;
}

__host__ __device__ inline MaternSetup matern_setup(double t1, double t2, double t3)
{
    MaternSetup s;
    s.theta1 = t1;
    s.theta2 = t2;
    s.nu = t3;
    s.kind = (t3 == 0.5) ? 1 : (t3 == 1.5) ? 2 : (t3 == 2.5) ? 3 : 0;
    int nl = (int)floor(t3 + 0.5);
    double mu = t3 - nl;
    s.nl = nl;
    s.mu = mu;
    // even and odd parts of 1/Γ(1+z) at z = μ
    double m2 = mu * mu, ev = 0.0, od = 0.0;
    for (int k = GL_RGAMMA_TERMS - 2; k >= 0; k -= 2) ev = ev * m2 + gl_rgamma_coef[k];
    for (int k = GL_RGAMMA_TERMS - 1; k >= 1; k -= 2) od = od * m2 + gl_rgamma_coef[k];
    s.g2 = ev;
    s.g1 = -od;
    const double rgp = ev + mu * od;  // 1/Γ(1+μ) = Σ c_k μ^k
    const double rgm = ev - mu * od;  // 1/Γ(1-μ) = Σ c_k (-μ)^k
    s.hgp = 0.5 / rgp;
    s.hgm = 0.5 / rgm;
    double pm = M_PI * mu;
    if (fabs(pm) < 1e-4) {
        double p2 = pm * pm;
        s.fact = 1.0 + p2 / 6.0 + 7.0 * p2 * p2 / 360.0;
    } else {
        s.fact = pm / sin(pm);
    }
    // Γ(ν) from Γ(1+μ) = 1/rgp: Γ(μ+nl) = Γ(1+μ) Π_{j=1}^{nl-1} (μ+j); nl = 0 → Γ(μ) = Γ(1+μ)/μ
    double gnu;
    if (nl == 0) {
        gnu = 1.0 / (rgp * mu);
    } else {
        gnu = 1.0 / rgp;
        for (int j = 1; j < nl; ++j) gnu *= (mu + j);
    }
    s.pref = t1 * exp2(1.0 - t3) / gnu;
    return s;
}

// Per-k constants of the series and the recurrence below, for one μ: filled
// once per workgroup in LDS so the per-element loops only multiply and add.
// Both loops take four terms at a time, so the constants of a group are read
// together and their LDS latency is paid once per group.  (Σ12 of 40,000 ×
// 1,000 points at ν = 1: 1,256 µs with a table lookup and a test in every step,
// a division instead wherever the compiler could not rule the table out and
// six more per element, 645 µs now; bound by the binary64 instructions, about
// 1,200 cycles per 64 elements before the loops and 28 per step.)
constexpr int GL_TEMME_TERMS = 40;
constexpr int GL_MILLER_MAX = 80;
struct alignas(16) BesselTab {
    double te[4 * (GL_TEMME_TERMS + 1)];  // 1/(k - μ), 1/(k + μ), their product, 1/k
    double mi[2 * (GL_MILLER_MAX + 1)];   // (k + 1/2)² - μ², ((k - 1/2)² - μ²)/k
};

// Every thread of the workgroup calls this before the first matern_eval with
// the table; it ends with a barrier.
__device__ inline void bessel_tab_init(const MaternSetup &s, BesselTab &t)
{
    for (int k = threadIdx.x; k <= GL_MILLER_MAX; k += blockDim.x) {
        const double dk = (double)k;
        if (k >= 1 && k <= GL_TEMME_TERMS) {
            const double rm = 1.0 / (dk - s.mu), rp = 1.0 / (dk + s.mu);
            t.te[4 * k] = rm;
            t.te[4 * k + 1] = rp;
            t.te[4 * k + 2] = rm * rp;
            t.te[4 * k + 3] = 1.0 / dk;
        }
        t.mi[2 * k] = (dk + 0.5) * (dk + 0.5) - s.mu * s.mu;
        t.mi[2 * k + 1] = k ? ((dk - 0.5) * (dk - 0.5) - s.mu * s.mu) / dk : 0.0;
    }
    __syncthreads();
}

// K_μ(x) and K_μ+1(x) for x <= 2 (Temme's series), unscaled; lx = log(2/x),
// xi = 1/x.  One exponential e^σ, σ = μ lx, gives sinh σ, cosh σ and (x/2)^∓μ.
// TAB: the constants come from the table.
template <bool TAB>
__host__ __device__ inline void bessel_k_temme(const MaternSetup &s, double x, double xi, double lx, double &k0,
                                               double &k1, const BesselTab *tab)
{
#pragma clang fp contract(off)
    const double mu = s.mu;
    const double sig = mu * lx;
    const double e = exp(sig), ei = plain_rcp(e);
    double shs;  // sinh(σ)/σ
    if (fabs(sig) < 0.1) {
        const double q = sig * sig;  // Taylor series to σ⁸, remainder below 3e-18
        shs = fma(q, 1.0 / 72.0, 1.0);
        shs = fma(q * (1.0 / 42.0), shs, 1.0);
        shs = fma(q * (1.0 / 20.0), shs, 1.0);
        shs = fma(q * (1.0 / 6.0), shs, 1.0);
    } else {
        shs = 0.5 * (e - ei) * plain_rcp(sig);
    }
    double f = s.fact * fma(0.5 * (e + ei), s.g1, shs * lx * s.g2);
    double p = e * s.hgp;   // ½ (x/2)^-μ Γ(1+μ)
    double q = ei * s.hgm;  // ½ (x/2)^μ Γ(1-μ)
    double c = 1.0;
    const double d = 0.25 * x * x;
    double sum0 = f, sum1 = p;
    const double *te = TAB ? tab->te + 4 * opaque_zero() : nullptr;
    // terms in groups of four; the test on the last of a group
    for (int g = 1; g <= GL_TEMME_TERMS; g += 4) {
        double t0 = 0.0, t1 = 0.0;
#pragma unroll
        for (int k = g; k < g + 4; ++k) {
            const double dk = (double)k;
            double rm, rp, rr, rk;
            if constexpr (TAB) {
                rm = te[4 * k];
                rp = te[4 * k + 1];
                rr = te[4 * k + 2];
                rk = te[4 * k + 3];
            } else {
                rm = 1.0 / (dk - mu);
                rp = 1.0 / (dk + mu);
                rr = rm * rp;
                rk = 1.0 / dk;
            }
            f = fma(dk, f, p + q) * rr;
            c *= d * rk;
            p *= rm;
            q *= rp;
            t0 = f;
            t1 = fma(-dk, f, p);
            sum0 = fma(c, t0, sum0);
            sum1 = fma(c, t1, sum1);
        }
        if (fabs(c * t0) < 1e-17 * fabs(sum0) && fabs(c * t1) < 1e-17 * fabs(sum1)) break;
    }
    k0 = sum0;
    k1 = 2.0 * sum1 * xi;
}

// e^x K_μ(x) and e^x K_μ+1(x) for x > 2 (backward recurrence for U ratios); xi = 1/x.
template <bool TAB>
__host__ __device__ inline void bessel_k_miller_scaled(const MaternSetup &s, double x, double xi, double &k0, double &k1,
                                                       const BesselTab *tab)
{
#pragma clang fp contract(off)
    const double mu2 = s.mu * s.mu;
    int kmax = (int)(8.0 + 140.0 * xi) + 3;
    kmax = (kmax < GL_MILLER_MAX ? kmax : GL_MILLER_MAX) & ~3;  // whole groups of four
    const double x2 = 2.0 * x;
    double z1 = 0.0, z0 = 1.0;  // z_{K+1}, z_K
    double t = 1.0;             // Horner accumulation of Σ c_k z_k from the top
    const double *mi = TAB ? tab->mi + 2 * opaque_zero() : nullptr;
    // The group counter does not depend on the lane (a lane joins at its own
    // depth), so the constants' addresses are the wave's.
    for (int g = GL_MILLER_MAX; g >= 4; g -= 4) {
        if (g > kmax) continue;
#pragma unroll
        for (int k = g; k > g - 4; --k) {
            const double dk = (double)k;
            double ma, mb;
            if constexpr (TAB) {
                ma = mi[2 * k];
                mb = mi[2 * k + 1];
            } else {
                ma = (dk + 0.5) * (dk + 0.5) - mu2;
                mb = ((dk - 0.5) * (dk - 0.5) - mu2) / dk;
            }
            const double zm = fma(x2 + 2.0 * dk, z0, -(ma * z1));
            z1 = z0;
            z0 = zm;
            t = fma(mb, t, zm);
        }
    }
    const double r0 = z1 * plain_rcp(z0);
    k0 = sqrt(0.5 * M_PI * xi) * z0 * plain_rcp(t);  // over S = t / z0
    k1 = k0 * fma(mu2 - 0.25, r0, s.mu + 0.5 + x) * xi;
}

// The half-integer closed forms at x = r/θ2 (s.kind 1, 2, 3).
__host__ __device__ inline double matern_closed(const MaternSetup &s, double x)
{
#pragma clang fp contract(off)
    switch (s.kind) {
    case 1: return s.theta1 * exp(-x);
    case 2: return s.theta1 * (1.0 + x) * exp(-x);
    default: return s.theta1 * (1.0 + x + x * x / 3.0) * exp(-x);
    }
}

// Matérn covariance at distance r for a half-integer setup (s.kind != 0):
// the same values as matern_eval, without the Bessel evaluator (so kernels
// that only take this path keep few registers).
__host__ __device__ inline double matern_eval_closed(const MaternSetup &s, double r)
{
    if (r == 0.0) return s.theta1;
    const double x = r / s.theta2;
    if (x > 2000.0) return 0.0;
    return matern_closed(s, x);
}

// Matérn covariance at distance r (r >= 0); with TAB, tab is from
// bessel_tab_init for the same setup.
template <bool TAB>
__host__ __device__ inline double matern_eval_t(const MaternSetup &s, double r, const BesselTab *tab)
{
#pragma clang fp contract(off)
    if (r == 0.0) return s.theta1;
    const double x = r / s.theta2;
    // Past x = 2000 the correlation C/θ1 is below e^-1600 for every ν <= 50,
    // so C underflows to 0 for any finite θ1; returning early also keeps
    // the closed forms' polynomials and the recurrences below finite.
    if (x > 2000.0) return 0.0;
    if (s.kind != 0) return matern_closed(s, x);
    // Below 1e-150 the distance is far inside rounding of a repeated location;
    // the clamp keeps K_μ+1 (about x^-3/2 at most) and the scaled recurrence
    // below finite.
    const double xc = fmax(x, 1e-150);
    double ka, kb;
    const bool small = (xc <= 2.0);
    const double lgx = log(xc);  // serves the series' log(2/x) and x^ν or x^ν e^-x
    const double xi = plain_rcp(xc);
    if (small) bessel_k_temme<TAB>(s, xc, xi, M_LN2 - lgx, ka, kb, tab);
    else bessel_k_miller_scaled<TAB>(s, xc, xi, ka, kb, tab);
    double knu;
    double lsc = 0.0;  // natural log of the power of two divided out of (ka, kb)
    if (s.nl == 0) {
        knu = ka;
    } else {
        // (ka, kb) = (K_μ+i-1, K_μ+i) → K_μ+nl.  K grows with the order, like
        // (2/x)^ν Γ(ν)/2 for small x, and overflows binary64 at large ν while
        // x^ν underflows; the pair is rescaled by 2^-900 whenever it passes
        // 2^500, so it stays below 2^124 after a rescale, one step multiplies
        // it by at most 1 + 2ν/x < 2^505 (ν <= 50, x >= 1e-150), and the
        // scale joins the exponent of x^ν at the end.
        if (kb > 0x1p500) {
            ka *= 0x1p-900;
            kb *= 0x1p-900;
            lsc += 900.0 * M_LN2;
        }
        for (int i = 1; i < s.nl; ++i) {
            double kc = fma(2.0 * (s.mu + i) * xi, kb, ka);
            ka = kb;
            kb = kc;
            if (kb > 0x1p500) {
                ka *= 0x1p-900;
                kb *= 0x1p-900;
                lsc += 900.0 * M_LN2;
            }
        }
        knu = kb;
    }
    return s.pref * exp(fma(s.nu, lgx, small ? lsc : lsc - xc)) * knu;
}

__host__ __device__ inline double matern_eval(const MaternSetup &s, double r) { return matern_eval_t<false>(s, r, nullptr); }
__device__ inline double matern_eval(const MaternSetup &s, double r, const BesselTab *tab)
{
    return matern_eval_t<true>(s, r, tab);
}

__host__ __device__ inline double dist2d(double x1, double y1, double x2, double y2)
{
#pragma clang fp contract(off)
    double dx = x1 - x2, dy = y1 - y2;
    return sqrt(fma(dx, dx, dy * dy));
}

// Great-circle distance on a sphere of radius rho (Sec. 7.4): x = longitude,
// y = latitude in degrees; the haversine h = sin²(Δφ/2) + cos φ1 cos φ2
// sin²(Δλ/2) gives d = 2 rho asin(√h), h clamped to [0, 1].
__host__ __device__ inline double gcd_dist_cos(double x1, double y1, double c1, double x2, double y2, double c2,
                                               double rho)  // c: cos of the latitude
{
#pragma clang fp contract(off)
    const double deg = M_PI / 180.0;
    const double sp = sin(0.5 * ((y2 - y1) * deg));
    const double sl = sin(0.5 * ((x2 - x1) * deg));
    double h = fma(c1 * c2 * sl, sl, sp * sp);
    h = fmin(fmax(h, 0.0), 1.0);
    return 2.0 * rho * asin(sqrt(h));
}

__host__ __device__ inline double gcd_dist(double x1, double y1, double x2, double y2, double rho)
{
    const double deg = M_PI / 180.0;
    return gcd_dist_cos(x1, y1, cos(y1 * deg), x2, y2, cos(y2 * deg), rho);
}

__host__ __device__ inline double geo_dist(const Geom &g, double x1, double y1, double x2, double y2)
{
    return g.metric ? gcd_dist(x1, y1, x2, y2, g.radius) : dist2d(x1, y1, x2, y2);
}

}  // namespace gl
