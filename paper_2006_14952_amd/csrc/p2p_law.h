// FP64 force law of P2P: its constants, computed on the host, and the weight of one pair.
// Also compiles as plain C++, so that a host program can measure both.
#pragma once
#include <math.h>
#include <string.h>

#ifdef __HIPCC__
#define HFMM_HD __host__ __device__ __forceinline__
#else
#define HFMM_HD inline
#endif

namespace hfmm {

// f_(1) = S(r^2) - 1/r^3 up to r_cut.  S, a smooth function of r^2, is written about the
// cutoff, with d = r_cut^2 - r^2 >= 0:
//   S = S_0 + d T(d),  T = sum c_k d^k, k < ncoef (19 or 22; the polynomial split: 1)
// Near the cutoff S and 1/r^3 agree to one part in 1/h, h = r^3 |f_(1)| (57 at 4.5 r_s, 170 at
// 5 r_s).  So S_0 is held to twice the precision, S_0 - 1/r^3 is formed from the exact cube of an
// estimate and its correction (law64_weight), good to a few roundings of f_(1), and the rest,
// d T, vanishes with d.  The terms that matter in T are positive, as all of S's Taylor series is.
// Largest relative error of a pair's weight, any separation, against 80-bit arithmetic: 1.4e-15
// at r_cut = 4.5 r_s, 2.3e-15 at 5 r_s; by erfc and exp 2.0e-15 and 2.4e-15 (the means by tenths of
// r_cut: up to 1.33 times theirs between 0.6 and 0.9, at 5 r_s 2.0 times between 0.5 and 0.8, and
// below them elsewhere); with S - 1/r^3
// formed from a polynomial over the whole range, an operation a pair less, 2.3e-14 and 1.9e-13.
// Accelerations of 4096 particles against extended precision at 4.5 r_s (median, 99th percentile
// of the relative error): uniform 1.9e-16 and 8.0e-16, clustered 1.6e-16 and 7.4e-16; by erfc and
// exp on unshifted coordinates 2.4e-16 and 3.9e-15, 1.9e-16 and 3.0e-15.
constexpr int kLawShort = 19, kP2PPoly64Max = 22;
struct P2PConst64 {
    double c[kP2PPoly64Max];
    double s0, s0_lo;  // S_0 and what FP64 leaves of it
    double rc2, rs;
    // The form works in lengths times `scale`, the power of two that brings r_cut into
    // [1/2, 1): exact, and no power of a length leaves the range of the type, however small
    // or large the box (the gaps squared in FP32 by the box tests least of all).
    double scale;
    float scale32;  // the same for the FP32 boxes
    float cut;      // r_cut and a margin for the box tests; infinite: no tests
    int ncoef;      // coefficients of T; 0: erfc and exp
};

// One pair of the FP64 form: the weight m f_(1)(r), zero outside 0 < r^2 < r_cut^2.  y: an
// estimate of 1/r to about 23 bits.  It is cut to 26 bits, so that y^2 and the residual
// e = 1 - r^2 y^2 are exact to far below FP64's last place, and 1/r^3 = y^3 (1 - e)^(-3/2).
// S_0 - y^3 is rounded once with 19 coefficients, two operations a pair less than the exact form
// that 22 need (3.5e-15 otherwise at 5 r_s) and the polynomial split, whose force vanishes with
// d^2.  The self pair's NaN is dropped by the select.
template <int NPC> HFMM_HD double law64_weight(const P2PConst64 &k, double r2, double m, double y)
{
    const bool in = r2 > 0.0 && r2 < k.rc2;
    if constexpr (NPC == 0) {
        const double rr2 = in ? r2 : 1.0, r = sqrt(rr2), u = r * (0.5 / k.rs);
        const double h = erfc(u) + r * (1.0 / (k.rs * 1.7724538509055160273)) * exp(-u * u);
        return in ? -m * h / (rr2 * r) : 0.0;
    } else {
        long long b;
        memcpy(&b, &y, 8);
        b &= ~0x7ffffffll;
        memcpy(&y, &b, 8);
        const double y2 = y * y, e = fma(-r2, y2, 1.0), q = fma(1.875, e, 1.5) * e;
        const double d = k.rc2 - r2;
        double T = k.c[NPC - 1];
#pragma unroll
        for (int c = NPC - 2; c >= 0; --c) T = fma(T, d, k.c[c]);
        double f1;
        if constexpr (NPC == kLawShort) {
            f1 = fma(d, T, fma(-y2, y, k.s0)) + fma(-(y2 * y), q, k.s0_lo);
        } else {
            // the rounded y^3 (an fma: a product would be contracted into the difference, which is
            // then exact near the cutoff) and what the rounding left
            const double y3 = fma(y2, y, 0.0), lo = fma(y2, y, -y3);
            f1 = fma(d, T, k.s0 - y3) + (fma(-y3, q, k.s0_lo) - lo);
        }
        return in ? m * f1 : 0.0;
    }
}

// Coefficients by r_cut / r_s alone: the error left by the shortening of T, before its
// coefficients are rounded, stays below one rounding of f_(1) itself up to 4.558 (19) and
// 5.366 (22).  The lines lie between the ratios in use, whose last bits vary with r_s.  No fit
// beyond the second: S - S_0 then outweighs f_(1) so far that its roundings pass those of
// erfc and exp.
inline int law64_ncoef(double ratio) { return ratio <= 4.55 ? kLawShort : ratio <= 5.05 ? kP2PPoly64Max : 0; }

// S = 4/sqrt(pi) int_0^1 y^2 exp(-v y^2) dy, v = r^2 / (4 r_s^2), about v0 in extended
// precision: S = s0 + x sum T[k] x^k, x = 1 - v / v0 in [0, 1].  The Taylor coefficients
// v0^k / k! 4/sqrt(pi) I_k, I_k = int_0^1 y^(2k+2) exp(-v0 y^2) dy, follow by downward
// recurrence (all terms positive); their series is then shortened to m terms by taking off
// multiples of the shifted Chebyshev polynomials, highest first.
inline void law64_series(long double v0, int m, long double &s0, long double *T)
{
    constexpr int N = 48;  // v0 <= 6.4: the first term left out is below 1e-22
    struct Cheb {
        long double e[N][N];
        Cheb() : e{}
        {
            e[0][0] = 1;
            e[1][0] = -1;
            e[1][1] = 2;
            for (int j = 2; j < N; ++j)
                for (int q = 0; q <= j; ++q) e[j][q] = 2 * ((q ? 2 * e[j - 1][q - 1] : 0) - e[j - 1][q]) - e[j - 2][q];
        }
    };
    static const Cheb cheb;
    long double I[N + 2], t[N];
    const long double ev = expl(-v0);
    I[N + 1] = ev / (2 * N + 5);
    for (int k = N; k >= 0; --k) I[k] = (ev + 2 * v0 * I[k + 1]) / (2 * k + 3);
    long double p = 2.25675833419102514779231781243L;  // 4 / sqrt(pi)
    s0 = p * I[0];
    for (int k = 0; k < N; ++k) {
        p *= v0 / (k + 1);
        t[k] = p * I[k + 1];
    }
    for (int j = N - 1; j >= m; --j) {
        const long double a = t[j] / cheb.e[j][j];
        for (int q = 0; q <= j; ++q) t[q] -= a * cheb.e[j][q];
    }
    for (int k = 0; k < m; ++k) T[k] = t[k];
}

// A few microseconds; a tree keeps the result (P2PLaw64).
inline void law64_setup(double r_s, double r_cut, int split, P2PConst64 &k)
{
    k = P2PConst64{};
    int e;
    const double rc = frexp(r_cut, &e);
    k.scale = ldexp(1.0, -e);
    k.rs = r_s * k.scale;
    k.rc2 = rc * rc;
    const long double rc2 = k.rc2;
    if (split == 1) {  // S = 5/(2 r_c^3) - 3 r^2/(2 r_c^5); f_(1) vanishes with d^2, so S_0 is formed exactly:
        // 1/r_c^3 = s0 (1 + (1 - s0 r_c^3)), and r_c^2 = rc2 + low moves S_0 off it
        const double low = fma(rc, rc, -k.rc2), cube = k.rc2 * rc, cube_lo = fma(k.rc2, rc, -cube) + low * rc;
        k.s0 = 1.0 / cube;
        k.s0_lo = k.s0 * (fma(-k.s0, cube, 1.0) - k.s0 * cube_lo + 1.5 * low / k.rc2);
        k.c[0] = (double)(1.5L / (rc2 * rc2 * rc));
        k.ncoef = 1;
        return;
    }
    k.ncoef = law64_ncoef(r_cut / r_s);
    if (k.ncoef == 0) return;
    long double s0, T[kP2PPoly64Max];
    law64_series(rc2 / (4 * (long double)k.rs * k.rs), k.ncoef, s0, T);
    long double p = 1 / (8 * (long double)k.rs * k.rs * k.rs);
    k.s0 = (double)(s0 * p);
    k.s0_lo = (double)(s0 * p - k.s0);
    for (int j = 0; j < k.ncoef; ++j) {
        p /= rc2;
        k.c[j] = (double)(T[j] * p);
    }
}

// The constants of the last evaluation and what they were computed for.
struct P2PLaw64 {
    P2PConst64 k{};
    double box = 0, r_s = 0, r_cut = 0;
    int split = -1;
};

}  // namespace hfmm
