// Device arithmetic shared by the stage kernels (gfx950, wave64): the WENO5
// interface fluxes, the tortoise-chart point coefficients, the right-hand side
// of one point and the small data-movement helpers.
//
// Every kernel that advances a point goes through the functions of this file,
// and their arithmetic is written out operation by operation (fused operations
// spelled as fma, contraction off), so that a point's update has the same bits
// whichever kernel computes it: the launch shape, the batch and the temporal
// blocking never show in the results.
#pragma once

#include <hip/hip_runtime.h>

#include "teuk_coef.h"
#include "teuk_internal.h"

namespace teuk {

namespace {

// Radial chart (TEUK_CHART_*).
constexpr int kChartT = TEUK_CHART_TORTOISE;
constexpr int kChartH = TEUK_CHART_HYPERBOLOIDAL;
// The tortoise chart with fourth-order theta differences (a launch class of
// its own; the ABI's chart field stays TEUK_CHART_TORTOISE).
constexpr int kChartT4 = kChartTortoise4;

constexpr int kWave = 64;

__device__ __forceinline__ double fmad(double a, double b, double c) { return __builtin_fma(a, b, c); }

// 1/x from the hardware estimate refined by one Newton step.
__device__ __forceinline__ double rcp64(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fmad(-x, r, 1.0);
    return fmad(r, e, r);
}

// 1/sqrt(x), x > 0, to full FP64 precision: estimate plus two Newton steps.
__device__ __forceinline__ double rsq64(double x)
{
#pragma clang fp contract(off)
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    y = y * fmad(-h * y, y, 1.5);
    y = y * fmad(-h * y, y, 1.5);
    return y;
}

// The interface flux f^+_{j+1/2} from v0..v4 = f_{j-2..j+2} (Sec. 3.1.2).  The f^-
// flux f^-_{j+1/2} is the same function of the mirrored stencil
// (f_{j+3}, f_{j+2}, f_{j+1}, f_j, f_{j-1}).  `y` is 6 f, or 6 f without 6 v2 where
// kRelative; g1 = v2 - v1 and g2 = v3 - v2 are the first differences with which
// plus_diff / minus_diff put the 6 v2 back into a flux difference.
struct Flux {
    double y, g1, g2;
};

template <int WP>
struct Weno;

// Constants of the flux arithmetic, held for a whole march.  The empty asm keeps
// the multipliers in scalar registers: as literals they would only fit the
// two-operand fmac, whose accumulator then costs a register copy at each use
// (ten copies a row of a stage).
struct WenoK {
    double eps, eps4, c, k3, k6, k9;
};

__device__ __forceinline__ WenoK weno_consts(double eps)
{
    WenoK K{eps, 4.0 * eps, 13.0 / 3.0, 3.0, 6.0, 9.0};
    asm("" : "+s"(K.c), "+s"(K.k3), "+s"(K.k6), "+s"(K.k9));
    return K;
}

// Six stencil differences of the smoothness indicators, 4 IS_k = (13/3) d_k^2 + e_k^2.
struct Differences {
    double d0, d1, d2, e0, e1, e2;
    __device__ __forceinline__ Differences(double v0, double v1, double v2, double v3, double v4, const WenoK& K)
    {
#pragma clang fp contract(off)
        d0 = fmad(-2.0, v1, v0) + v2;
        d1 = fmad(-2.0, v2, v1) + v3;
        d2 = fmad(-2.0, v3, v2) + v4;
        e0 = fmad(K.k3, v2, fmad(-4.0, v1, v0));
        e1 = v1 - v3;
        e2 = fmad(-4.0, v3, K.k3 * v2) + v4;
    }
};

// The candidate part: 6 f = q2 + omega_0 (q0 - q2) + omega_1 (q1 - q2), the
// candidates (times 6) from the same differences
//     q2 = 3 (v2 + v3) - d2,  q1 - q2 = d2 - d1,  q0 = 2 d0 + 9 v2 - 3 v1.
struct Candidates {
    double q2, dq0, dq1;
    __device__ __forceinline__ Candidates(double v1, double v2, double v3, const Differences& q, const WenoK& K)
    {
#pragma clang fp contract(off)
        q2 = fmad(K.k3, v2 + v3, -q.d2);
        dq1 = q.d2 - q.d1;
        dq0 = fmad(2.0, q.d0, fmad(K.k9, v2, -(K.k3 * v1))) - q2;
    }
};

// FP64 weights.  Arithmetic, rearranged by exact identities (only rounding
// differs from the printed formulas):
//  * with the second differences d_k and first differences e_k of IS_k,
//    4 IS_k = (13/3) d_k^2 + e_k^2; eps is scaled by 4 as well, so every
//    t_k = (eps + IS_k)^2 carries the same factor 16, which cancels in omega;
//  * omega_k = alpha_k / sum alpha with alpha_k = d_k / t_k is taken over the
//    common denominator, constants scaled by 10:
//        omega_0 = t1 t2 / D,  omega_1 = 6 t0 t2 / D,  D = t1 t2 + 6 t0 t2 + 3 t0 t1,
//    one reciprocal instead of four divisions;
//  * omega_2 = 1 - omega_0 - omega_1, so the weights sum to one exactly in the
//    combination.
template <>
struct Weno<TEUK_W_FP64> {
    static constexpr bool kRelative = false;
    __device__ __forceinline__ static Flux flux(double v0, double v1, double v2, double v3, double v4, const WenoK& K)
    {
#pragma clang fp contract(off)
        const Differences q(v0, v1, v2, v3, v4, K);
        double t0 = fmad(K.c * q.d0, q.d0, fmad(q.e0, q.e0, K.eps4));
        double t1 = fmad(K.c * q.d1, q.d1, fmad(q.e1, q.e1, K.eps4));
        double t2 = fmad(K.c * q.d2, q.d2, fmad(q.e2, q.e2, K.eps4));
        t0 *= t0;
        t1 *= t1;
        t2 *= t2;
        const double p12 = t1 * t2, p02 = K.k6 * (t0 * t2);
        const double inv = rcp64(fmad(t1, t2, fmad(K.k3, t0 * t1, p02)));
        const Candidates f(v1, v2, v3, q, K);
        return {fmad(inv, fmad(p12, f.dq0, p02 * f.dq1), f.q2), 0.0, 0.0};
    }
};

// FP64 weights in the hyperboloidal chart, on the first differences
// g_i = v_{i+1} - v_i, again by identities of the printed formulas:
//  * (3/4) IS_0 = (g0 - 11/8 g1)^2 + 39/64 g1^2,  (3/4) IS_1 = (g1 - 5/8 g2)^2 + 39/64 g2^2,
//    (3/4) IS_2 = (g3 - 11/8 g2)^2 + 39/64 g2^2: with eps scaled by 3/4 as well, one
//    fma for each linear form a_k, one for each square and the term in g1 or g2
//    shared; the common factor of s_k = (3/4)(eps + IS_k) cancels in omega;
//  * D = t1 t2 + 6 t0 (t2 + t1/2), t_k = s_k^2;
//  * 6 (f - v2) = C + omega_0 (A - C) + omega_1 (B - C) with A = 5 g1 - 2 g0,
//    B = g1 + 2 g2, C = 4 g2 - g3, whose differences reuse the forms:
//    B - C = a1 + a2, A - C = a2 - 2 a0 + 9/4 g1 - 21/8 g2;
//  * the flux difference takes its 6 v2 part from the field difference directly
//    (plus_diff / minus_diff), so that no large value is formed and cancelled.
// 33 operations and one reciprocal a flux against the 42 of the form above.  (The
// tortoise chart keeps that form: its fields are sampled far outside a packet,
// where only the last bits of larger neighbours are left and any other order of
// operations would show.)
constexpr int kWeno64H = 16;

struct WenoKH {
    double e4, k0, k1, kh, k6, ka, kb;
};

template <>
struct Weno<kWeno64H> {
    static constexpr bool kRelative = true;
    __device__ __forceinline__ static Flux flux(double v0, double v1, double v2, double v3, double v4, const WenoKH& K)
    {
#pragma clang fp contract(off)
        const double g0 = v1 - v0, g1 = v2 - v1, g2 = v3 - v2, g3 = v4 - v3;
        const double h1 = fmad(K.kh * g1, g1, K.e4), h2 = fmad(K.kh * g2, g2, K.e4);
        const double a0 = fmad(K.k0, g1, g0), a1 = fmad(K.k1, g2, g1), a2 = fmad(K.k0, g2, g3);
        const double s0 = fmad(a0, a0, h1), s1 = fmad(a1, a1, h2), s2 = fmad(a2, a2, h2);
        const double t0 = s0 * s0, t1 = s1 * s1, t2 = s2 * s2;
        const double z = K.k6 * t0;
        const double n0 = t1 * t2, n1 = z * t2;
        const double inv = rcp64(fmad(z, fmad(0.5, t1, t2), n0));
        const double ac = fmad(K.kb, g2, fmad(K.ka, g1, fmad(-2.0, a0, a2)));
        const double x = fmad(n1, a1 + a2, n0 * ac);
        return {fmad(inv, x, fmad(4.0, g2, -g3)), g1, g2};
    }
};

// ---------------------------------------------------------------- reduced-precision weights
// Sec. 3.1.3: the smoothness indicators and nonlinear weights are computed in a
// lower precision and the weights are made to sum to one in FP64.  Here the six
// stencil differences of IS_k are taken in FP64 (differencing first keeps the
// information the low format would lose to cancellation), converted, and
// IS_k, alpha_k and omega_0, omega_1 are formed in the low format; omega_2 is
// the FP64 complement and the candidate fluxes stay FP64.
//
// The 16-bit weights use the ratio form
//     alpha'_k = d_k (tau_min / tau_k)^2,   tau_k = eps + IS_k,
// which equals alpha_k tau_min^2 (so omega is unchanged in exact arithmetic)
// and keeps every intermediate in [0, 1] whatever the magnitude of the data.
// rho_k = 1 where tau_k equals tau_min (also when both are zero).  FP32 has
// the range for the FP64 form and takes it (Weno<TEUK_W_FP32> below).

// Arithmetic in the low format: every result rounded to it, fma(a, b, c) once.
// taus forms the tau_k = eps + IS_k; which term of IS_k is rounded before their sum,
// 13/12 of the squared second difference or 1/4 of the other square, is the order that
// the format's results have had.
// ratio(a, b) is
// a / b for 0 <= a < b, a true division: after the power-of-two scaling eps
// can underflow to zero, so a flat stencil gives tau_min = 0 next to a tau_k
// below 2^-16 whose reciprocal overflows, and 0 * inf would poison the weights.
struct LowF16 {
    typedef _Float16 T;
    __device__ static T cvt(float x) { return (_Float16)x; }
    __device__ static T rcp(T x) { return (_Float16)1.0 / x; }
    __device__ static T ratio(T a, T b) { return a / b; }
    __device__ static T fma(T a, T b, T c) { return __builtin_fmaf16(a, b, c); }
    // (tau_0 and tau_1 as a pair: scalar operations throughout cost 3 % of a step,
    // 8192 x 256 124 us against 120)
    __device__ static void taus(T D0, T D1, T D2, T E0, T E1, T E2, T ep, T c1312, T c14, T& t0, T& t1, T& t2)
    {
#pragma clang fp contract(off)
        typedef T Two __attribute__((ext_vector_type(2)));
        t2 = ep + fma(c1312, D2 * D2, c14 * (E2 * E2));
        const Two y = {D0, E1}, x = {E0, D1};
        const Two t = __builtin_elementwise_fma(Two{c14, c1312}, x * x, Two{c1312, c14} * (y * y)) + ep;
        t0 = t.x;
        t1 = t.y;
    }
    __device__ static float f(T x) { return (float)x; }
};
// BF16 arithmetic: compute in FP32 and round each result to BF16 (round to
// nearest even).  FP32 carries more than 2p+2 bits for p = 8, so this equals a
// correctly rounded BF16 operation for +, -, * and /; an fma is the FP32 one, rounded.
struct Bf16Val {
    float v;
};
__device__ __forceinline__ float bf16_round(float x)
{
    return (float)(__bf16)x;
}
__device__ __forceinline__ Bf16Val operator+(Bf16Val a, Bf16Val b)
{
#pragma clang fp contract(off)
    return {bf16_round(a.v + b.v)};
}
__device__ __forceinline__ Bf16Val operator*(Bf16Val a, Bf16Val b)
{
#pragma clang fp contract(off)
    return {bf16_round(a.v * b.v)};
}
__device__ __forceinline__ bool operator<(Bf16Val a, Bf16Val b) { return a.v < b.v; }
__device__ __forceinline__ bool operator==(Bf16Val a, Bf16Val b) { return a.v == b.v; }
struct LowBF16 {
    typedef Bf16Val T;
    __device__ static T cvt(float x) { return {bf16_round(x)}; }
    // A quotient of two 8-bit significands lies at least 2^-16.9 (relative) from every
    // midpoint between BF16 values, so a times the 1 ulp reciprocal (error below
    // 2^-21) rounds to what the true quotient rounds to, in 2 instructions instead
    // of 10.  Where the reciprocal could overflow, a true division.  (Quotients
    // below 2^-126, whose significands are shorter, vanish when squared.)
    __device__ static T rcp(T x) { return {bf16_round(__builtin_amdgcn_rcpf(x.v))}; }
    __device__ static T fma(T a, T b, T c) { return {bf16_round(__builtin_fmaf(a.v, b.v, c.v))}; }
    __device__ static void taus(T D0, T D1, T D2, T E0, T E1, T E2, T ep, T c1312, T c14, T& t0, T& t1, T& t2)
    {
        t0 = ep + fma(D0 * D0, c1312, c14 * (E0 * E0));
        t1 = ep + fma(D1 * D1, c1312, c14 * (E1 * E1));
        t2 = ep + fma(D2 * D2, c1312, c14 * (E2 * E2));
    }
    __device__ static T ratio(T a, T b)
    {
#pragma clang fp contract(off)
        return {bf16_round(b.v >= 0x1p-120f ? a.v * __builtin_amdgcn_rcpf(b.v) : a.v / b.v)};
    }
    __device__ static float f(T x) { return x.v; }
};

template <class L, bool kScale>
__device__ __forceinline__ void low_weights(double d0, double d1, double d2, double e0, double e1, double e2,
                                            double eps, double* w0, double* w1)
{
#pragma clang fp contract(off)
    typedef typename L::T T;
    float fd0 = (float)d0, fd1 = (float)d1, fd2 = (float)d2;
    float fe0 = (float)e0, fe1 = (float)e1, fe2 = (float)e2;
    float feps = (float)eps;
    if (kScale) {
        // Scale by an exact power of two so that the largest of the differences
        // and sqrt(eps) is O(1): IS' = sigma^2 IS and eps' = sigma^2 eps leave the
        // weights unchanged and keep a 16-bit format away from overflow.
        float m = fmaxf(fmaxf(fmaxf(fabsf(fd0), fabsf(fd1)), fmaxf(fabsf(fd2), fabsf(fe0))),
                        fmaxf(fmaxf(fabsf(fe1), fabsf(fe2)), sqrtf(feps)));
        const int ex = __builtin_amdgcn_frexp_expf(m);
        fd0 = ldexpf(fd0, -ex); fd1 = ldexpf(fd1, -ex); fd2 = ldexpf(fd2, -ex);
        fe0 = ldexpf(fe0, -ex); fe1 = ldexpf(fe1, -ex); fe2 = ldexpf(fe2, -ex);
        feps = ldexpf(feps, -2 * ex);
    }
    const T c1312 = L::cvt(13.0f / 12.0f), c14 = L::cvt(0.25f);
    const T D0 = L::cvt(fd0), D1 = L::cvt(fd1), D2 = L::cvt(fd2);
    const T E0 = L::cvt(fe0), E1 = L::cvt(fe1), E2 = L::cvt(fe2);
    const T ep = L::cvt(feps);
    T t0, t1, t2;
    L::taus(D0, D1, D2, E0, E1, E2, ep, c1312, c14, t0, t1, t2);
    T tm = t0 < t1 ? t0 : t1;
    tm = t2 < tm ? t2 : tm;
    const T one = L::cvt(1.0f);
    const T r0 = t0 == tm ? one : L::ratio(tm, t0);
    const T r1 = t1 == tm ? one : L::ratio(tm, t1);
    const T r2 = t2 == tm ? one : L::ratio(tm, t2);
    const T q0 = r0 * r0;
    const T a0 = L::cvt(0.1f) * q0, a1 = L::cvt(0.6f) * (r1 * r1);
    const T inv = L::rcp(L::fma(L::cvt(0.3f), r2 * r2, L::fma(L::cvt(0.1f), q0, a1)));   // 1 / (a0 + a1 + a2)
    *w0 = (double)L::f(a0 * inv);
    *w1 = (double)L::f(a1 * inv);
}

// 6 f from the two low-format weights.
__device__ __forceinline__ double combine_weights(const Candidates& f, double w0, double w1)
{
#pragma clang fp contract(off)
    return f.q2 + fmad(w0, f.dq0, w1 * f.dq1);
}

template <class L, bool kScale>
struct WenoLow {
    static constexpr bool kRelative = false;
    __device__ __forceinline__ static Flux flux(double v0, double v1, double v2, double v3, double v4, const WenoK& K)
    {
        const Differences q(v0, v1, v2, v3, v4, K);
        double w0, w1;
        low_weights<L, kScale>(q.d0, q.d1, q.d2, q.e0, q.e1, q.e2, K.eps, &w0, &w1);
        return {combine_weights(Candidates(v1, v2, v3, q, K), w0, w1), 0.0, 0.0};
    }
};

// FP32 weights take one common denominator as the FP64 ones do,
//     omega_0 = t1 t2 / D,  omega_1 = 6 t0 t2 / D,  D = t1 t2 + 6 t0 t2 + 3 t0 t1,
// with t_k = (4 eps + 4 IS_k)^2 and one reciprocal (v_rcp_f32, 1 ulp), evaluated
// in FP32 from the six FP64 stencil differences, omega_2 the FP64 complement.
// FP32 has the range for it over most of the data: the denominator is at least
// 2560 eps^4 and stays finite for differences up to about 1e4.  It must also
// stay well above the subnormals, where the reciprocal overflows to inf (and
// 0 * inf is a NaN) or loses its precision: below 2^-100 -- every flat stencil
// once eps is under about 4e-9 -- and above 3e38 the lane takes the FP64 weights
// instead.  From 2^-100 on, a product that is subnormal or flushed to zero moves
// its weight by at most 2^-26 absolute.
template <>
struct Weno<TEUK_W_FP32> {
    static constexpr bool kRelative = false;
    __device__ __forceinline__ static Flux flux(double v0, double v1, double v2, double v3, double v4, const WenoK& K)
    {
#pragma clang fp contract(off)
        const Differences q(v0, v1, v2, v3, v4, K);
        const float D0 = (float)q.d0, D1 = (float)q.d1, D2 = (float)q.d2;
        const float E0 = (float)q.e0, E1 = (float)q.e1, E2 = (float)q.e2;
        constexpr float c = 13.0f / 3.0f;
        const float eps4 = (float)(4.0 * K.eps);
        float t0 = __builtin_fmaf(c * D0, D0, __builtin_fmaf(E0, E0, eps4));
        float t1 = __builtin_fmaf(c * D1, D1, __builtin_fmaf(E1, E1, eps4));
        float t2 = __builtin_fmaf(c * D2, D2, __builtin_fmaf(E2, E2, eps4));
        t0 *= t0;
        t1 *= t1;
        t2 *= t2;
        const float p12 = t1 * t2, p02 = 6.0f * (t0 * t2);
        const float den = __builtin_fmaf(t1, t2, __builtin_fmaf(3.0f, t0 * t1, p02));
        if (!(den >= 0x1p-100f && den <= 3.0e38f)) return Weno<TEUK_W_FP64>::flux(v0, v1, v2, v3, v4, K);
        const float inv = __builtin_amdgcn_rcpf(den);
        return {combine_weights(Candidates(v1, v2, v3, q, K), (double)(p12 * inv), (double)(p02 * inv)), 0.0, 0.0};
    }
};
template <>
struct Weno<TEUK_W_FP16> : WenoLow<LowF16, true> {};
template <>
struct Weno<TEUK_W_BF16> : WenoLow<LowBF16, true> {};

template <int WP>
__device__ __forceinline__ auto weno_consts_for(double eps)
{
    if constexpr (WP == kWeno64H) {
        WenoKH K{0.75 * eps, -1.375, -0.625, 39.0 / 64.0, 6.0, 2.25, -2.625};
        asm("" : "+s"(K.k0), "+s"(K.k1), "+s"(K.kh), "+s"(K.k6), "+s"(K.ka), "+s"(K.kb));
        return K;
    } else {
        return weno_consts(eps);
    }
}

// 6 dx times the derivative at j from this lane's flux at j - 1/2 and the next
// lane's flux value `yn` at j + 1/2: of f^+ fluxes (v2 = f_{j-1}, so the next
// lane's v2 is g2 further), and of f^- fluxes (v2 = f_j, mirrored).
template <int WP, class Consts>
__device__ __forceinline__ double plus_diff(const Consts& K, const Flux& f, double yn)
{
#pragma clang fp contract(off)
    return Weno<WP>::kRelative ? fmad(K.k6, f.g2, yn - f.y) : yn - f.y;
}
template <int WP, class Consts>
__device__ __forceinline__ double minus_diff(const Consts& K, const Flux& f, double yn)
{
#pragma clang fp contract(off)
    return Weno<WP>::kRelative ? fmad(-K.k6, f.g1, yn - f.y) : yn - f.y;
}

// ---------------------------------------------------------------- tortoise-chart points
// The radial factors of teuk_coef.h at one point, held for a whole march.
struct Radial {
    double t[kNRT];
};

__device__ __forceinline__ double ldb(const double* base, unsigned off);

__device__ __forceinline__ Radial load_radial(const StageArgs& A, unsigned oc)
{
    Radial r;
#pragma unroll
    for (int i = 0; i < kNRT; ++i) r.t[i] = ldb(A.rtab + (size_t)i * A.nr, oc);
    return r;
}

// The polar factors of one theta row (uniform over the wave: scalar loads).
struct Polar {
    double sn2, cs, cot, th;
};

__device__ __forceinline__ Polar load_polar(const StageArgs& A, int k)
{
    const __attribute__((address_space(4))) double* t =
        (const __attribute__((address_space(4))) double*)A.ttab;
    return {t[kSn2 * A.nth + k], t[kCs * A.nth + k], t[kCot * A.nth + k], t[kTh * A.nth + k]};
}

__device__ __forceinline__ double point_vsig(const Radial& r, double sn2)
{
    return rsq64(fmad(-r.t[kQ], sn2, r.t[kP]));
}

// point_coef of teuk_coef.h, v = 1/Sigma.
__device__ __forceinline__ PointCoef point_coef_t(const Radial& r, const Polar& p, double v)
{
#pragma clang fp contract(off)
    const double* t = r.t;
    const double w = v * v;
    PointCoef c;
    c.b = t[kRa2] * v;
    c.ath = t[kDl] * w;
    c.bth = c.ath * p.cot;
    c.btr = w * t[kT0];
    c.bti = w * fmad(t[kT2], p.cs, t[kT1]);
    c.cr = w * fmad(-t[kDl], p.th, t[kA0]);
    c.ci = w * t[kA1];
    c.m3r = fmad(c.b, c.btr, w * fmad(-w, fmad(-t[kG2], p.sn2, t[kG1]), t[kH0]));
    c.m3i = fmad(c.b, c.bti, -(w * t[kX1]));
    return c;
}

// Centred theta differences of one plane (not yet scaled): second order, and
// fourth order, from Phi on the rows k + 1, k - 1 (k + 2, k - 2).
struct Theta {
    double d1, d2;
};
__device__ __forceinline__ Theta theta2(double ph, double up, double dn)
{
#pragma clang fp contract(off)
    return {up - dn, fmad(-2.0, ph, up) + dn};
}
__device__ __forceinline__ Theta theta4(double ph, double up, double dn, double up2, double dn2)
{
#pragma clang fp contract(off)
    return {fmad(8.0, up - dn, -(up2 - dn2)), fmad(16.0, up + dn, -(30.0 * ph)) - (up2 + dn2)};
}

struct Four {
    double v[4];
};

// F(u) of one point: dPh*, dPi* the radial derivatives times 6 dx, xR, xI the
// theta differences of Phi, ih1 the scale of the first (negated by a caller that
// took it backwards).
//     d_t Phi = pi - b d_x Phi
//     d_t pi  = b d_x pi - m3 d_x Phi + B~t pi + A~thth Phi_thth + B~th Phi_th + C~ Phi
// kBtFirst: which product of Im(B~t pi) is fused into the other's rounding.  It
// shows in the last bit only, but far outside a pulse the field is the
// difference of much larger neighbours and the last bits are all of it, so each
// weight precision and integrator keeps the order that its results have had.
template <int WP>
constexpr bool bt_first() { return WP == TEUK_W_FP64 || WP == TEUK_W_BF16; }

template <bool kBtFirst>
__device__ __forceinline__ Four rhs_t(const StageArgs& A, double ih1, const PointCoef& c, double dPhR, double dPhI, double dPiR,
                                      double dPiI, double phR, double phI, double piR, double piI, const Theta& xR,
                                      const Theta& xI)
{
#pragma clang fp contract(off)
    dPhR *= A.inv6dx;
    dPhI *= A.inv6dx;
    dPiR *= A.inv6dx;
    dPiI *= A.inv6dx;
    double sR = fmad(c.b, dPiR, -fmad(c.m3r, dPhR, -(c.m3i * dPhI)));
    double sI = fmad(c.b, dPiI, -fmad(c.m3i, dPhR, c.m3r * dPhI));
    sR += fmad(c.btr, piR, -(c.bti * piI));
    sI += kBtFirst ? fmad(c.btr, piI, c.bti * piR) : fmad(c.bti, piR, c.btr * piI);
    sR = fmad(c.ath, xR.d2 * A.ih2, sR);
    sI = fmad(c.ath, xI.d2 * A.ih2, sI);
    sR = fmad(c.bth, xR.d1 * ih1, sR);
    sI = fmad(c.bth, xI.d1 * ih1, sI);
    sR += fmad(c.cr, phR, -(c.ci * phI));
    sI += fmad(c.ci, phR, c.cr * phI);
    return {{fmad(-c.b, dPhR, piR), fmad(-c.b, dPhI, piI), sR, sI}};
}

// F(u) of one point in the hyperboloidal chart: ten coefficients hc from the
// table, dPh*, dPi* the radial derivatives, up / dn Phi on the rows k + 1 / k - 1.
//     d_t Phi = pi - lam1 d_x Phi
//     d_t pi  = -lam2 d_x pi - m3 d_x Phi + B~t pi + A~thth Phi_thth + B~th Phi_th + C~ Phi
__device__ __forceinline__ Four rhs_h(const double (&hc)[kNCH], double ih1, double ih2, double dPhR, double dPhI,
                                      double dPiR, double dPiI, double phR, double phI, double piR, double piI,
                                      double upR, double upI, double dnR, double dnI)
{
#pragma clang fp contract(off)
    const double a2 = hc[kHAth] * ih2, a1 = hc[kHBth] * ih1;
    const double lapR = fmad(-2.0, phR, upR + dnR), lapI = fmad(-2.0, phI, upI + dnI);
    double sR = -(hc[kHLam2] * dPiR);
    sR = fmad(-hc[kHM3r], dPhR, sR);
    sR = fmad(hc[kHM3i], dPhI, sR);
    sR = fmad(hc[kHBtr], piR, sR);
    sR = fmad(-hc[kHBti], piI, sR);
    sR = fmad(a2, lapR, sR);
    sR = fmad(a1, upR - dnR, sR);
    sR = fmad(hc[kHCr], phR, sR);
    sR = fmad(-hc[kHCi], phI, sR);
    double sI = -(hc[kHLam2] * dPiI);
    sI = fmad(-hc[kHM3r], dPhI, sI);
    sI = fmad(-hc[kHM3i], dPhR, sI);
    sI = fmad(hc[kHBtr], piI, sI);
    sI = fmad(hc[kHBti], piR, sI);
    sI = fmad(a2, lapI, sI);
    sI = fmad(a1, upI - dnI, sI);
    sI = fmad(hc[kHCr], phI, sI);
    sI = fmad(hc[kHCi], phR, sI);
    Four F;
    F.v[0] = fmad(-hc[kHLam1], dPhR, piR);
    F.v[1] = fmad(-hc[kHLam1], dPhI, piI);
    F.v[2] = sR;
    F.v[3] = sI;
    return F;
}

// u + dt F and the stage combination ca u^n + cb v.
__device__ __forceinline__ double euler(double u, double dt, double F) { return fmad(dt, F, u); }
__device__ __forceinline__ double combine(double ca, double un, double cb, double v)
{
#pragma clang fp contract(off)
    return fmad(ca, un, cb * v);
}

// x of lane l + 1 (0 in lane 63), by a DPP wavefront shift: no LDS round trip,
// unlike __shfl_down.  Used wherever a lane takes the interface flux of the lane
// after it; lane 63 never uses what it gets.
__device__ __forceinline__ double next_lane(double x)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Barrier that orders LDS only.  __syncthreads() is also a workgroup fence on
// global memory, which makes every wave drain its outstanding global loads
// (s_waitcnt vmcnt(0)) before the barrier: that would serialise the row
// prefetch below with the arithmetic it is meant to overlap.
__device__ __forceinline__ void lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders LDS between the lanes of one wave: what a lane wrote before it is what the
// others read after it.  (The wave barrier alone is no memory operation to the compiler,
// which may move a read of another lane's value over the write that it cannot see it
// needs; the hardware runs a wave's LDS operations in order, so the fences cost nothing.)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Load a double at a byte offset from a uniform base: the 32-bit offset lets
// the compiler use the scalar-base addressing form (no 64-bit address math),
// and the global address space keeps it from flat accesses where the base came
// out of memory (the members' descriptors of a batched launch).
typedef const __attribute__((address_space(1))) char* GlobalBytes;
__device__ __forceinline__ double ldb(const double* base, unsigned off)
{
    return *(const __attribute__((address_space(1))) double*)((GlobalBytes)base + off);
}
__device__ __forceinline__ void stb(double* base, unsigned off, double v)
{
    *(__attribute__((address_space(1))) double*)((__attribute__((address_space(1))) char*)base + off) = v;
}

// Ranks are dealt so that each XCD (which receives every eighth workgroup id)
// owns a contiguous block of ranks, i.e. whole strips and their neighbours.
__device__ __forceinline__ int xcd_rank(int bid, int G)
{
    const int xcd = bid & 7, loc = bid >> 3;
    const int q8 = G >> 3, r8 = G & 7;
    return xcd * q8 + (xcd < r8 ? xcd : r8) + loc;
}

}  // namespace

}  // namespace teuk
