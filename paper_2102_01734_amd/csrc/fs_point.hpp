// fs_point.hpp -- per-point arithmetic of the long-characteristics formal
// solution, shared by the box and the spherical sweep kernels (gfx950).
//
// Per point (Listing 1 of the paper): optical steps from the voxel opacities
// and path lengths (step 3), interpolation weights with the linear fallback
// (step 4) and the vacuum fix-up (4a), the Lambda* data (4b) and exp(-dtau)
// for the intensity update (5).  Everything here is evaluated in double; the
// results are rounded to the recurrence type T at the end.
#pragma once

#include <hip/hip_runtime.h>

namespace rt3d {

// c - a b with a constant c (a polynomial coefficient).  The negated factor
// keeps the compiler on the three-address v_fma_f64, which reads c from a
// scalar register pair: the two-address v_fmac form it prefers for a plain
// a b + c would copy c into the destination at every use, and take 14 vector
// registers for the coefficients.  The polynomials below are therefore written
// in the negated argument.
__device__ __forceinline__ double fma3(const double &a, double b, double c) { return __builtin_fma(a, -b, c); }

// The same for a literal a: two constants, so an FMA by name (the compiler
// would fold the negation into a and fall back to v_fmac).
__device__ __forceinline__ double fma3(double &&a, double b, double c)
{
    double d;
    asm("v_fma_f64 %0, %1, -%2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

__device__ __forceinline__ double seg_depth(double chi, double s)
{
#pragma clang fp contract(off)
    return chi * s;
}

// 1/x from the hardware reciprocal estimate refined by Newton steps
// r <- r + r (1 - x r), each of which doubles the correct bits: two steps for
// double results, one when the weights are rounded to single precision.
template <bool FULL = true>
__device__ __forceinline__ double rcp_f64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    r = __builtin_fma(r, e, r);
    if (!FULL) return r;
    e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}

// exp(-D) for 1/4 <= D, double results: the Cody-Waite argument reduction
// x = -D = n ln2 + r, |r| <= ln2/2, where n ln2 is subtracted in two parts
// (ln2 split into a high part with trailing zero bits, so that n times it is
// exact, and the low remainder; the split of the fdlibm exponential), exp(r)
// by its degree-12 Taylor polynomial, scaled by 2^n.  D is clamped at 745,
// where the result is already below the smallest subnormal.
__device__ __forceinline__ double exp_neg(double D)
{
    const double x = -(D < 745.0 ? D : 745.0);
    const double n = __builtin_rint(x * 1.4426950408889634);
    double r = __builtin_fma(-n, 6.93147180369123816490e-01, x);
    r = __builtin_fma(-n, 1.90821492927058770002e-10, r);
    double p = 1.0 / 479001600.0;
    p = __builtin_fma(p, r, 1.0 / 39916800.0);
    p = __builtin_fma(p, r, 1.0 / 3628800.0);
    p = __builtin_fma(p, r, 1.0 / 362880.0);
    p = __builtin_fma(p, r, 1.0 / 40320.0);
    p = __builtin_fma(p, r, 1.0 / 5040.0);
    p = __builtin_fma(p, r, 1.0 / 720.0);
    p = __builtin_fma(p, r, 1.0 / 120.0);
    p = __builtin_fma(p, r, 1.0 / 24.0);
    p = __builtin_fma(p, r, 1.0 / 6.0);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    return __builtin_ldexp(p, (int)n);
}

// Attenuation moments for single-precision results, one polynomial for every
// step D > 0 (see kernel_moments for the definitions).  x = -min(D, 745) =
// n ln2 + r with n = rint(x / ln2) and |r| <= ln2/2; the reduction takes one
// FMA with ln2 rounded to double, whose error (|n| <= 1075 times 2.3e-17)
// stays below 3e-14.  The tail u = e^r - 1 - r = r^2 (1/2 + r P(r)), with
// P(r) = sum_{j>=0} r^j/(j+3)! from its degree-6 interpolant at the Chebyshev
// nodes of |r| <= ln2/2 (relative error 1.6e-11 there).  Where n = 0 (D below ln2/2) r is -D
// exactly and the moments follow from u with no cancellation: e1 = u,
// e0 = D - u, ex = 1 - e0, e2 = D^2 - 2 e1 = -2 r^3 P.  Elsewhere
// ex = 2^n (1 + r + u) and the closed forms below, which lose at most about
// five bits to cancellation from D = ln2/2 up.  (The code holds -n and -r.)
//
// WANT_H (the box sweep): the last output is h = D e1 - e2 instead of e2, the
// only combination its weights need besides e1: D^3 (1/2 + r P - 2 P) where
// n = 0 (no cancellation beyond a factor of three), 2 e1 - D e0 elsewhere, one
// instruction fewer on either side than e2 and then h.  Both sides run under a
// lane mask, 14 instructions; measured against it on 129^3 x 2048 (63.5 ms a
// launch): jumps for wavefronts that are thin, thick or mixed as a whole, 64.5
// ms with fewer instructions, and one formula for both sides without a mask,
// 67.3 ms with three more.
template <bool WANT_H = false>
__device__ __forceinline__ void moments_single(double D, double &ex, double &e0, double &e1, double &e2)
{
    // z = min(D, 745) by one instruction (the library minimum would first
    // quiet signalling NaNs, which arithmetic never produces); a NaN step
    // gives a finite z, and e1, e2 keep the NaN.  r here is the negated
    // reduced argument
    double z;
    asm("v_min_f64 %0, %1, %2" : "=v"(z) : "v"(D), "s"(745.0));
    const double n = __builtin_rint(z * 1.4426950408889634);
    const double r = __builtin_fma(n, -0.6931471805599453, z);
    // degree-6 Chebyshev interpolant of P on |r| <= ln2/2 (gen_moment_poly.py)
    double P = fma3(2.761004197490652e-06, r, 2.485957814859904e-05);
    P = fma3(P, r, 0.00019841238150245533);
    P = fma3(P, r, 0.0013888854049701165);
    P = fma3(P, r, 0.008333333338101687);
    P = fma3(P, r, 0.0416666667189806);
    P = fma3(P, r, 0.16666666666666652);
    const double r2 = r * r;
    const double h = __builtin_fma(-r, P, 0.5);  // u = r^2 h
    if (n == 0.0) {
        e1 = r2 * h;
        e0 = __builtin_fma(-r2, h, D);  // spelled out, as below: kernels that share the moments agree to the bit
        ex = 1.0 - e0;
        e2 = WANT_H ? (D * r2) * __builtin_fma(-2.0, P, h) : (2.0 * r2) * (r * P);
    } else {
        ex = __builtin_ldexp(__builtin_fma(r2, h, 1.0 - r), -(int)n);
        e0 = 1.0 - ex;
        e1 = D - e0;
        e2 = WANT_H ? __builtin_fma(2.0, e1, -(D * e0)) : __builtin_fma(D, D, -2.0 * e1);
    }
}

// Attenuation moments over an optical step D > 0:
//   ex = exp(-D), e0 = 1 - ex, e1 = D - e0, e2 = D^2 - 2 e1.
// Double results (FULL): below D = 1/4, e2 comes from its 12-term Taylor
// series 2 D^3 sum_j (-D)^j/(j+3)! and e1, e0, ex follow from it without
// cancellation; from 1/4 up the closed forms are used (separate branches: a
// wave whose steps straddle 1/4 runs both).  Single-precision results take
// moments_single, one path for all D.
template <bool FULL>
__device__ __forceinline__ void kernel_moments(double D, double &ex, double &e0, double &e1, double &e2)
{
    if constexpr (!FULL) {
        moments_single(D, ex, e0, e1, e2);
        return;
    }
    double p = 1.0 / 87178291200.0;                // 1/14!
    p = __builtin_fma(-D, p, 1.0 / 6227020800.0);  // 1/13!
    p = __builtin_fma(-D, p, 1.0 / 479001600.0);   // 1/12!
    p = __builtin_fma(-D, p, 1.0 / 39916800.0);    // 1/11!
    p = __builtin_fma(-D, p, 1.0 / 3628800.0);     // 1/10!
    p = __builtin_fma(-D, p, 1.0 / 362880.0);      // 1/9!
    p = __builtin_fma(-D, p, 1.0 / 40320.0);       // 1/8!
    p = __builtin_fma(-D, p, 1.0 / 5040.0);        // 1/7!
    p = __builtin_fma(-D, p, 1.0 / 720.0);         // 1/6!
    p = __builtin_fma(-D, p, 1.0 / 120.0);         // 1/5!
    p = __builtin_fma(-D, p, 1.0 / 24.0);          // 1/4!
    p = __builtin_fma(-D, p, 1.0 / 6.0);           // 1/3!
    const double D2 = D * D;
    if (D < 0.25) {
        const double c = (D2 + D2) * D, u = __builtin_fma(-c, p, D2);
        e2 = c * p;
        e1 = 0.5 * u;
        e0 = __builtin_fma(-0.5, u, D);
        ex = 1.0 - e0;
        return;
    }
    ex = exp_neg(D);
    e0 = 1.0 - ex;
    e1 = D - e0;
    e2 = __builtin_fma(D, D, -2.0 * e1);
}

// Smallest optical step used in the arithmetic: a vacuum segment (D = 0,
// Listing 1 step 4a) is evaluated at this step, which leaves the intensity
// unchanged to within 1e-100 of S and keeps the shared reciprocal finite.
constexpr double kMinStep = 1e-100;

// Weights of the segment from the previous point (upwind optical step D) to
// the current one, the downwind step being Dp (ignored when last), in the
// type T of the recurrence:
//   I_m = I_{m-1} ex + a S_{m-1} + b S_m + g S_{m+1}.
// Parabolic: the Lagrange quadratic through the three points integrated
// against exp(-(D-t)); with r = 1/(D Dp (D+Dp)),
//   b = ((D+Dp) e1 - e2) (D+Dp) r,  g = (e2 - D e1) D r,  a = e0 - b - g.
// Linear (the last point of a ray, Dp < D/2, or where the parabolic b would
// reach 1, i.e. Dp e0 <= D e1 - e2):  b = e1/D, a = e0 - b, g = 0.
// dlin = e1/D is the diagonal of the linear-interpolation operator.
template <typename T>
struct PointW {
    T a, b, g, ex, dlin;
};

// FULL: double-accurate moments (the default for double results); false: the
// shorter forms that suffice where the results are rounded to single precision.
template <typename T, bool FULL = sizeof(T) == 8>
__device__ __forceinline__ PointW<T> point_weights(double D, double Dp, bool last)
{
    const double Dv = D < kMinStep ? kMinStep : D;  // NaN propagates
    double ex, e0, e1, e2;
    kernel_moments<FULL>(Dv, ex, e0, e1, e2);
    const double Dq = Dp < kMinStep ? Dv : Dp;   // keeps r finite on last/vacuum points; NaN propagates
    const double Ds = Dv + Dq;
    const double r = rcp_f64<FULL>(Dv * Dq * Ds);
    const double bl = e1 * ((Dq * Ds) * r);      // e1 / D
    const bool lin = last || (Dp < 0.5 * D) || (Dp * e0 <= __builtin_fma(Dv, e1, -e2));
    const double bp = __builtin_fma(Ds, e1, -e2) * (Ds * r);
    const double gp = (e2 - Dv * e1) * (Dv * r);
    PointW<T> w;
    w.ex = T(ex);
    w.dlin = T(bl);
    if (sizeof(T) == 8) {
        w.b = lin ? T(bl) : T(bp);
        w.g = lin ? T(0) : T(gp);
        w.a = lin ? T(e0 - bl) : T(e0 - bp - gp);
    } else {
        const T bl_t = T(bl), al_t = T(e0 - bl), bp_t = T(bp), gp_t = T(gp), ap_t = T(e0 - bp - gp);
        w.b = lin ? bl_t : bp_t;
        w.g = lin ? T(0) : gp_t;
        w.a = lin ? al_t : ap_t;
    }
    return w;
}

// point_weights for optical steps that are already at least kMinStep (sums of
// half_depth): no clamping here.  LAST: the final point of a ray (linear
// weights; Dp is not read); `last` says the same per lane (Dp any step).  DLIN: also the linear operator's diagonal e1/D.
// The linear weights are the parabolic ones in the limit of an infinite
// downwind step.  Double results: a point that takes them is evaluated with Dp
// replaced by 2^300 (beta = e1/D (1 + O(D/2^300)), gamma far below the rounding
// for any physical step; D D'(D + D') stays finite for every D below 2^360).
// Single results: with h = 0, which is the same limit at any D', by one select
// of one word; D D'(D + D') stays finite for every D below 2^340, and float
// opacities give steps below 2^140.
//
// Reciprocals of single results: REFINE takes one Newton step after the hardware
// estimate (about 2^-48), which the shell's sweep needs: its opacities reach optical
// steps of 1e6 and more, where alpha is about 1/D and is left of e0 - beta - gamma, so
// that an error d of the reciprocal is one of d D in alpha.  Without, d is at most
// 4.6e-8 (2^-24.4) over a million random arguments: below the rounding of beta and
// gamma to single precision, and the three weights still sum to e0 whatever it is, but
// alpha is good to its own rounding only for steps of order one; at D = 1e6 it is a
// few per cent off, and from about 2e7 up it may be negative.  The box sweep does
// without (two of its 71 vector instructions a point): what alpha then misses is at
// most 4.6e-8 of the upwind source, which is that source's own rounding, and shows
// only where the sources downwind of a thick step are that much weaker.
template <typename T, bool LAST, bool DLIN = true, bool REFINE = false>
__device__ __forceinline__ PointW<T> point_weights_pos(double D, double Dp, bool last = false)
{
    constexpr bool FULL = sizeof(T) == 8;
    PointW<T> w;
    w.dlin = T(0);
    double ex, e0, e1;
    if constexpr (FULL) {
        double e2;
        kernel_moments<true>(D, ex, e0, e1, e2);
        const double h = __builtin_fma(D, e1, -e2);  // D e1 - e2
        const bool lin = LAST || last || (Dp < 0.5 * D) || (Dp * e0 <= h);
        const double Dq = lin ? 0x1p300 : Dp;
        const double Ds = D + Dq;
        const double r = rcp_f64<true>(D * Dq * Ds);
        const double b = __builtin_fma(Ds, e1, -e2) * (Ds * r);
        const double g = h * (-D * r);
        w.ex = T(ex);
        w.b = T(b);
        w.g = T(g);
        w.a = T(e0 - b - g);
        if constexpr (DLIN) w.dlin = T(e1 * rcp_f64<true>(D));
        return w;
    } else {
        double h;  // D e1 - e2
        moments_single<true>(D, ex, e0, e1, h);
        w.ex = T(ex);
        if constexpr (LAST) {
            const double b = e1 * (REFINE ? rcp_f64<false>(D) : __builtin_amdgcn_rcp(D));
            w.b = w.dlin = T(b);
            w.g = T(0);
            w.a = T(e0 - b);
            return w;
        }
        const bool lin = last || (Dp < 0.5 * D) || (Dp * e0 <= h);
        const double Ds = D + Dp;
        const double r = REFINE ? rcp_f64<false>(D * Dp * Ds) : __builtin_amdgcn_rcp(D * Dp * Ds);
        // linear points: h = 0 in b = (h + D' e1) / (D D'), g = -h / (D' (D + D'))
        // leaves b = e1/D and g = 0.  Clearing the high word is enough: what is
        // left, below 1e-313, is nothing beside D' e1 > 1e-301.
        h = __hiloint2double(lin ? 0 : __double2hiint(h), __double2loint(h));
        const double b = __builtin_fma(Dp, e1, h) * (Ds * r);
        const double g = h * (-D * r);
        w.b = T(b);
        w.g = T(g);
        w.a = T(e0 - b - g);
        if constexpr (DLIN) w.dlin = T(e1 * (REFINE ? rcp_f64<false>(D) : __builtin_amdgcn_rcp(D)));
        return w;
    }
}

// Half the optical depth of a segment, chi s / 2 + kMinStep / 2, from half its
// path length (halving is exact): the optical step between two points is then
// the plain sum of their half depths, and equals (ta + tb)/2 of the full depths
// ta, tb >= 0 bit for bit for every depth above 2^-270.  A vacuum step,
// ta = tb = 0, becomes kMinStep, and so the shared reciprocal of the weights
// stays finite.  NaN and Inf propagate.
__device__ __forceinline__ double half_depth(double chi, double s_half)
{
    double d;
    // three addresses: the two-address form would copy the constant addend first
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(chi), "s"(s_half), "v"(0.5 * kMinStep));
    return d;
}

// The step between two half depths, without contraction.
__device__ __forceinline__ double step_of(double ha, double hb)
{
#pragma clang fp contract(off)
    return ha + hb;
}

// Entry half-segment: constant S from the entry point to the first point.
template <typename T>
__device__ __forceinline__ void entry_weights(double D0, T &ex_t, T &e0_t)
{
    constexpr bool FULL = sizeof(T) == 8;
    double ex, e0, e1, e2;
    kernel_moments<FULL>(D0 < kMinStep ? kMinStep : D0, ex, e0, e1, e2);
    ex_t = T(ex);
    e0_t = T(e0);
}

}  // namespace rt3d
