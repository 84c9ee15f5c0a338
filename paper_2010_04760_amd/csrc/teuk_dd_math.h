// Double-double arithmetic and the WENO5 flux of the double-double state, apart from
// the kernel so that the arithmetic can be compiled for the host as well (a test
// compares its rounding error with binary128).
//
// All of it is rounded exactly as written: multiply-add contraction is off, fused
// operations are spelled out as fma.
//   - error-free transformations: TwoSum (Knuth), FastTwoSum (Dekker), TwoProd
//     by one FMA;
//   - double-word sum, products and reciprocal after Joldes, Muller and
//     Popescu, "Tight and rigorous error bounds for basic building blocks of
//     double-word arithmetic" (ACM TOMS 2017): AccurateDWPlusDW (relative error
//     <= 3u^2), DWPlusFP (2u^2), DWTimesFP3 (2u^2), DWTimesDW3 (4u^2), u = 2^-53;
//     the reciprocal is the double reciprocal corrected by one Newton step
//     carried to second order in the residual.
// Sums and products of the flux are all normalised: products with unnormalised low
// words in the weights and in their sum, and short sums of differences, take a quarter of
// the kernel's instructions away (2048 x 64 60.9 -> 48.9 us a step), but raise the rms
// error of a flux by 7 % on rough data and 14 % on data of 1e-6, that of a packet of 2.5
// points a width by 7 %.
#pragma once

#include "teuk_dd_tables.h"

#ifdef __clang__
#pragma clang fp contract(off)
#endif

namespace teuk {

namespace {

struct dd {
    double hi, lo;
};

__device__ __forceinline__ dd two_sum(double a, double b)
{
    const double s = a + b;
    const double bb = s - a;
    return {s, (a - (s - bb)) + (b - bb)};
}

// |a| >= |b| (or a = 0)
__device__ __forceinline__ dd fast_two_sum(double a, double b)
{
    const double s = a + b;
    return {s, b - (s - a)};
}

__device__ __forceinline__ dd two_prod(double a, double b)
{
    const double p = a * b;
    return {p, fma(a, b, -p)};
}

__device__ __forceinline__ dd dd_add(dd x, dd y)
{
    const dd s = two_sum(x.hi, y.hi);
    const dd t = two_sum(x.lo, y.lo);
    const dd v = fast_two_sum(s.hi, s.lo + t.hi);
    return fast_two_sum(v.hi, t.lo + v.lo);
}

__device__ __forceinline__ dd dd_neg(dd x) { return {-x.hi, -x.lo}; }
__device__ __forceinline__ dd dd_sub(dd x, dd y) { return dd_add(x, dd_neg(y)); }
// exact scaling by a power of two
__device__ __forceinline__ dd dd_scale(dd x, double p2) { return {x.hi * p2, x.lo * p2}; }

__device__ __forceinline__ dd dd_add_d(dd x, double y)
{
    const dd s = two_sum(x.hi, y);
    return fast_two_sum(s.hi, x.lo + s.lo);
}

__device__ __forceinline__ dd dd_mul_d(dd x, double y)
{
    const dd c = two_prod(x.hi, y);
    return fast_two_sum(c.hi, fma(x.lo, y, c.lo));
}

__device__ __forceinline__ dd dd_mul(dd x, dd y)
{
    const dd c = two_prod(x.hi, y.hi);
    const double tl1 = fma(x.hi, y.lo, x.lo * y.lo);
    const double cl2 = fma(x.lo, y.hi, tl1);
    return fast_two_sum(c.hi, c.lo + cl2);
}

// 1/y: t = 1/y.hi to a unit or two of its last place (hardware estimate and two Newton
// steps), e = 1 - y t (1 - y.hi t is exact to 2u^2), 1/y = t (1 + e + e^2 + ...)
__device__ __forceinline__ dd dd_recip(dd y)
{
    double t = __builtin_amdgcn_rcp(y.hi);
    t = fma(t, fma(-y.hi, t, 1.0), t);
    t = fma(t, fma(-y.hi, t, 1.0), t);
    const double e = fma(-y.lo, t, fma(-y.hi, t, 1.0));
    return fast_two_sum(t, t * fma(e, e, e));
}

__device__ __forceinline__ double sqd(double v) { return v * v; }

// x y + z w
__device__ __forceinline__ dd two_products(dd x, dd y, dd z, dd w) { return dd_add(dd_mul(x, y), dd_mul(z, w)); }

struct DDK {
    dd inv_dx, ih1, ih2, ca, cb, sixth, c13_3, d[3];
};

// Mixed weights (Sec. 3.1.3): the stencil rounded to double, IS_k, alpha_k,
// omega_0 and omega_1 in double exactly as printed (f^+_{j+1/2} from
// g = f_{j-2..j+2}).
__device__ __forceinline__ void w64_plus(const double g[5], double eps, double& w0, double& w1)
{
    const double IS0 = 13.0 / 12.0 * sqd(g[0] - 2.0 * g[1] + g[2]) + 0.25 * sqd(g[0] - 4.0 * g[1] + 3.0 * g[2]);
    const double IS1 = 13.0 / 12.0 * sqd(g[1] - 2.0 * g[2] + g[3]) + 0.25 * sqd(g[1] - g[3]);
    const double IS2 = 13.0 / 12.0 * sqd(g[2] - 2.0 * g[3] + g[4]) + 0.25 * sqd(3.0 * g[2] - 4.0 * g[3] + g[4]);
    const double a0 = (1.0 / 10.0) * sqd(1.0 / (eps + IS0));
    const double a1 = (6.0 / 10.0) * sqd(1.0 / (eps + IS1));
    const double a2 = (3.0 / 10.0) * sqd(1.0 / (eps + IS2));
    const double sum = a0 + a1 + a2;
    w0 = a0 / sum;
    w1 = a1 / sum;
}

// The same for f^-_{j+1/2} from g = f_{j-1..j+3} (omega_0 pairs with the
// right-most stencil g_2..g_4).
__device__ __forceinline__ void w64_minus(const double g[5], double eps, double& w0, double& w1)
{
    const double IS0 = 13.0 / 12.0 * sqd(g[2] - 2.0 * g[3] + g[4]) + 0.25 * sqd(3.0 * g[2] - 4.0 * g[3] + g[4]);
    const double IS1 = 13.0 / 12.0 * sqd(g[1] - 2.0 * g[2] + g[3]) + 0.25 * sqd(g[1] - g[3]);
    const double IS2 = 13.0 / 12.0 * sqd(g[0] - 2.0 * g[1] + g[2]) + 0.25 * sqd(g[0] - 4.0 * g[1] + 3.0 * g[2]);
    const double a0 = (1.0 / 10.0) * sqd(1.0 / (eps + IS0));
    const double a1 = (6.0 / 10.0) * sqd(1.0 / (eps + IS1));
    const double a2 = (3.0 / 10.0) * sqd(1.0 / (eps + IS2));
    const double sum = a0 + a1 + a2;
    w0 = a0 / sum;
    w1 = a1 / sum;
}

// f^+_{j+1/2} from f = f_{j-2..j+2} (the f^- flux is this on the mirrored
// stencil).  With first differences g_i = f_{i+1} - f_i the candidates are
//     6 (q_0 - f_2) = 5 g_1 - 2 g_0,  6 (q_1 - f_2) = g_1 + 2 g_2,  6 (q_2 - f_2) = 4 g_2 - g_3,
// and the smoothness indicators 4 IS_k = (13/3) d_k^2 + e_k^2 with
//     d_0 = g_1 - g_0, d_1 = g_2 - g_1, d_2 = g_3 - g_2,
//     e_0 = 3 g_1 - g_0, e_1 = -(g_1 + g_2), e_2 = g_3 - 3 g_2
// (identities of the printed formulas).  WM = 1: omega_0, omega_1 given in
// double, omega_2 = 1 - omega_0 - omega_1 in double-double.
template <int WM>
__device__ __forceinline__ dd weno(dd f0, dd f1, dd f2, dd f3, dd f4, const DDK& K, double eps, double w0d,
                                   double w1d)
{
    const dd g0 = dd_sub(f1, f0), g1 = dd_sub(f2, f1);
    const dd g2 = dd_sub(f3, f2), g3 = dd_sub(f4, f3);
    const dd A = dd_sub(dd_mul_d(g1, 5.0), dd_scale(g0, 2.0));
    const dd B = dd_add(g1, dd_scale(g2, 2.0));
    const dd C = dd_sub(dd_scale(g2, 4.0), g3);
    dd s6;
    if constexpr (WM == 1) {
        // 6 (f - f_2) = C + omega_0 (A - C) + omega_1 (B - C)
        s6 = dd_add(C, dd_add(dd_mul_d(dd_sub(A, C), w0d), dd_mul_d(dd_sub(B, C), w1d)));
    } else {
        const dd d0 = dd_sub(g1, g0), d1 = dd_sub(g2, g1), d2 = dd_sub(g3, g2);
        const dd e0 = dd_sub(dd_mul_d(g1, 3.0), g0);
        const dd e1 = dd_add(g1, g2);
        const dd e2 = dd_sub(g3, dd_mul_d(g2, 3.0));
        // IS_k = ((13/3) d^2 + e^2) / 4; alpha_k = d_k / (eps + IS_k)^2
        const dd is0 = dd_scale(dd_add(dd_mul(K.c13_3, dd_mul(d0, d0)), dd_mul(e0, e0)), 0.25);
        const dd is1 = dd_scale(dd_add(dd_mul(K.c13_3, dd_mul(d1, d1)), dd_mul(e1, e1)), 0.25);
        const dd is2 = dd_scale(dd_add(dd_mul(K.c13_3, dd_mul(d2, d2)), dd_mul(e2, e2)), 0.25);
        const dd r0 = dd_recip(dd_add_d(is0, eps)), r1 = dd_recip(dd_add_d(is1, eps)), r2 = dd_recip(dd_add_d(is2, eps));
        const dd a0 = dd_mul(K.d[0], dd_mul(r0, r0));
        const dd a1 = dd_mul(K.d[1], dd_mul(r1, r1));
        const dd a2 = dd_mul(K.d[2], dd_mul(r2, r2));
        const dd inv = dd_recip(dd_add(dd_add(a0, a1), a2));
        s6 = dd_add(dd_add(dd_mul(dd_mul(a0, inv), A), dd_mul(dd_mul(a1, inv), B)), dd_mul(dd_mul(a2, inv), C));
    }
    return dd_add(f2, dd_mul(s6, K.sixth));
}

}  // namespace

}  // namespace teuk
