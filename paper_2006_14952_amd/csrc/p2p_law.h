// FP64 force law of P2P: its constants, computed on the host.  Plain C++, so that a host
// program can measure it.
#pragma once
#include <math.h>

#include <mutex>

namespace hfmm {

// f_(1) = -1/r^3 + S(t)/(8 r_s^3) as in the FP32 form, S fitted to FP64 rounding.  S's terms
// are summed from the smallest, so the sum is good to a few units of 1e-16 of 1/r^3, which is
// what the particles' forces are rounded to by their nearest pairs anyway.  Accelerations of
// 4096 particles against extended precision (median, 99th percentile of the relative error,
// means of four boxes): uniform 2.3e-16 and 1.1e-15, clustered 2.0e-16 and 1.5e-15; the erfc/exp
// form on unshifted coordinates 2.8e-16 and 3.8e-15, 2.1e-16 and 2.4e-15.
constexpr int kP2PPoly64Max = 23;
struct P2PConst64 {
    double c[kP2PPoly64Max];  // S(t) / (8 r_s^3), coefficients of t^0 .. t^(ncoef-1)
    double two_over_rc2, rc2, rs, irc2, irc3;
    // The form works in lengths times `scale`, the power of two that brings r_cut into
    // [1/2, 1): exact, and no power of a length leaves the range of the type, however small
    // or large the box (the gaps squared in FP32 by the box tests least of all).
    double scale;
    float scale32;  // the same for the FP32 boxes
    float cut;      // r_cut and a margin for the box tests; infinite: no tests
    int ncoef;      // coefficients of the fit; 0: no fit (erfc and exp)
};

// S(v) in extended precision: sum (-1)^k v^k / (k! (2k+3)), whose terms stay below e^v.
inline long double S_of_v_ext(long double v)
{
    long double s = 0, term = 1;
    for (int k = 0; k < 80; ++k) {
        s += term / (2 * k + 3);
        term *= -v / (k + 1);
    }
    return 4.0L / sqrtl(3.14159265358979323846264338327950288L) * s;
}

// Interpolation of S at the m Chebyshev points through its Chebyshev series, rewritten in
// powers of t, in extended precision.
inline void fit_S64(double vcut, int m, double *coef)
{
    const long double pi = 3.14159265358979323846264338327950288L;
    long double f[kP2PPoly64Max], mono[kP2PPoly64Max] = {0};
    for (int k = 0; k < m; ++k) f[k] = S_of_v_ext((cosl(pi * (k + 0.5L) / m) + 1.0L) * 0.5L * vcut);
    long double t0[kP2PPoly64Max] = {1}, t1[kP2PPoly64Max] = {0, 1}, t2[kP2PPoly64Max];
    for (int j = 0; j < m; ++j) {
        long double cj = 0;
        for (int k = 0; k < m; ++k) cj += f[k] * cosl(pi * j * (k + 0.5L) / m);
        cj *= (j ? 2.0L : 1.0L) / m;
        for (int q = 0; q < m; ++q) mono[q] += cj * t0[q];
        for (int q = 0; q < m; ++q) t2[q] = (q ? 2.0L * t1[q - 1] : 0.0L) - t0[q];  // T_(j+2)
        for (int q = 0; q < m; ++q) {
            t0[q] = t1[q];
            t1[q] = t2[q];
        }
    }
    for (int j = 0; j < m; ++j) coef[j] = (double)mono[j];
}

// Coefficients by r_cut / r_s alone, from the fit's error before its coefficients are rounded
// (in r^3 f_(1); 20 of them reach 2e-16 at 4.96, 23 past 5.5).  The lines lie between the
// ratios in use, whose last bits vary with r_s.  No fit beyond the second: there r^3 f_(1) has
// fallen to 1/170 at the cutoff, and the cancellation would show in the forces of isolated
// particles.
inline int law64_ncoef(double ratio) { return ratio <= 4.85 ? 20 : ratio <= 5.05 ? 23 : 0; }

inline void law64_setup(double r_s, double r_cut, int split, P2PConst64 &k)
{
    k = P2PConst64{};
    int e;
    const double rc = frexp(r_cut, &e);
    k.scale = ldexp(1.0, -e);
    k.rs = r_s * k.scale;
    k.rc2 = rc * rc;
    k.two_over_rc2 = 2.0 / k.rc2;
    k.irc2 = 1.0 / k.rc2;
    k.irc3 = k.irc2 / rc;
    if (split == 1) return;
    k.ncoef = law64_ncoef(r_cut / r_s);
    if (k.ncoef == 0) return;
    static std::mutex mu;  // the last fit is kept
    static double cached_vcut = -1.0, cached[kP2PPoly64Max];
    static int cached_m = 0;
    const double vcut = k.rc2 / (4.0 * k.rs * k.rs);
    std::lock_guard<std::mutex> lk(mu);
    if (vcut != cached_vcut || k.ncoef != cached_m) {
        fit_S64(vcut, k.ncoef, cached);
        cached_vcut = vcut;
        cached_m = k.ncoef;
    }
    const double inv8rs3 = 1.0 / (8.0 * k.rs * k.rs * k.rs);
    for (int j = 0; j < k.ncoef; ++j) k.c[j] = cached[j] * inv8rs3;
}

}  // namespace hfmm
