// Double-double stage kernel (tortoise chart): the paper's quad-precision
// baseline of Sec. 3.1.3, with every state value carried as an unevaluated sum
// hi + lo of two doubles (106 significant bits) and the WENO weights either in
// double-double or, as in the paper's mixed variant, in double.
//
// Arithmetic (all of it in this file is rounded exactly as written: the
// pragma below turns off multiply-add contraction; fused operations are
// spelled out as fma):
//   - error-free transformations: TwoSum (Knuth), FastTwoSum (Dekker), TwoProd
//     by one FMA;
//   - double-word sum, products and reciprocal after Joldes, Muller and
//     Popescu, "Tight and rigorous error bounds for basic building blocks of
//     double-word arithmetic" (ACM TOMS 2017): AccurateDWPlusDW (relative error
//     <= 3u^2), DWPlusFP (2u^2), DWTimesFP3 (2u^2), DWTimesDW3 (4u^2), u = 2^-53;
//     the reciprocal is the double reciprocal corrected by one Newton step
//     carried to second order in the residual.
// Work layout: one workgroup of four waves per (63-point radial strip, theta
// row), one wave for each of the four planes; workgroups go strip by strip through a
// row, each XCD through rows of its own (row by row through a strip was 2 % slower on
// grids that HBM feeds).  Lane l of a strip owns point
// j = 63 strip + l and computes the interface flux of its wave's plane at
// j - 1/2; the flux at j + 1/2 comes from lane l + 1.  The Phi waves then form the
// theta differences and hand them and their radial derivatives to the pi waves,
// which form the coupled sums meanwhile and wait once.  Values are (hi, lo) pairs
// stored as double2, [4][ntheta][nr], radial index fastest.
//
// Bound: FP64 VALU issue, 2 to 20 instructions for each operation, about 3000 a
// strip-row with double-double weights (4310 with accurate sums, IEEE reciprocals and
// normalised products everywhere).  How many waves a SIMD gets one after the other
// decides small grids: with all four planes in one wave, 2048 x 64 gave some SIMDs
// three of them and most two.  2048 x 64 with double-double weights 82.4 -> 49.3 us a
// step, with FP64 weights 57.5 -> 44.3; 100 x 20 32.5 -> 13.5; 8192 x 256 898 -> 690
// and 614 -> 609.
#include <hip/hip_runtime.h>

#include "teuk_dd_tables.h"
#include "teuk_device.h"
#include "teuk_internal.h"

#pragma clang fp contract(off)

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

// x + y with an error of u^2 (|x| + |y|) instead of 3u^2 |x + y|: for terms of one
// sign, and where the operands' own errors are as large
__device__ __forceinline__ dd dd_add_s(dd x, dd y)
{
    const dd s = two_sum(x.hi, y.hi);
    return fast_two_sum(s.hi, s.lo + (x.lo + y.lo));
}
__device__ __forceinline__ dd dd_sub_s(dd x, dd y) { return dd_add_s(x, dd_neg(y)); }

// x^2 and x y as pairs whose low words are not normalised (a few u of the high one)
__device__ __forceinline__ dd sq_raw(dd x)
{
    const dd c = two_prod(x.hi, x.hi);
    return {c.hi, fma(x.hi + x.hi, x.lo, fma(x.lo, x.lo, c.lo))};
}
__device__ __forceinline__ dd mul_raw(dd x, double y)
{
    const dd c = two_prod(x.hi, y);
    return {c.hi, fma(x.lo, y, c.lo)};
}

__device__ __forceinline__ dd mul_raw(dd x, dd y)
{
    const dd c = two_prod(x.hi, y.hi);
    return {c.hi, fma(x.hi, y.lo, fma(x.lo, y.hi, fma(x.lo, y.lo, c.lo)))};
}

// A running sum of products: the high words summed by TwoSum, everything below
// them in one low word, normalised once at the end.  Its error is a few u^2 of the
// sum of the terms' sizes, as is that of products rounded one by one.
struct Acc {
    double s, l;
    __device__ __forceinline__ void add(dd x)
    {
        const dd t = two_sum(s, x.hi);
        s = t.hi;
        l += t.lo + x.lo;
    }
    __device__ __forceinline__ dd get() const { return fast_two_sum(s, l); }
};
__device__ __forceinline__ Acc acc(dd x) { return {x.hi, x.lo}; }

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

// A pair of a row whose address is uniform over the wave (kept in scalar registers, so
// that an access costs no address arithmetic), at a byte offset within it.
typedef __attribute__((address_space(1))) char* GlobalChar;
typedef double Pair __attribute__((ext_vector_type(2)));
__device__ __forceinline__ GlobalChar scalar(const double2* p)
{
    GlobalChar g = (GlobalChar)const_cast<double2*>(p);
    asm("" : "+s"(g));
    return g;
}
__device__ __forceinline__ dd ld(const double2* row, unsigned off)
{
    const Pair v = *(__attribute__((address_space(1))) const Pair*)(scalar(row) + off);
    return {v.x, v.y};
}
__device__ __forceinline__ void st(double2* row, unsigned off, dd v)
{
    *(__attribute__((address_space(1))) Pair*)(scalar(row) + off) = Pair{v.hi, v.lo};
}

__device__ __forceinline__ dd shfl_down1(dd v)
{
    return {__shfl_down(v.hi, 1, 64), __shfl_down(v.lo, 1, 64)};
}

// x y + z w
__device__ __forceinline__ dd two_products(dd x, dd y, dd z, dd w) { return dd_add(dd_mul(x, y), dd_mul(z, w)); }

struct DDK {
    dd inv_dx, ih1, ih2, ca, cb, sixth, eps12;
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
//     e_0 = 3 g_1 - g_0 = d_0 + 2 g_1, e_1 = g_1 + g_2, e_2 = g_3 - 3 g_2 = d_2 - 2 g_2
// (identities of the printed formulas; e_1 enters squared).  With double-double
// weights the differences of the g_i are formed by the short sum: an error of u^2 |g|
// in them is one of u^2 in IS_k, whose square root is at least of the size of the g_i
// that enter it, and the candidates carry as much from the g_i themselves.  WM = 1: omega_0, omega_1 given in double, omega_2 = 1 - omega_0 -
// omega_1 in double-double.
template <int WM>
__device__ __forceinline__ dd weno(dd f0, dd f1, dd f2, dd f3, dd f4, const DDK& K, double w0d, double w1d)
{
    const dd g0 = dd_sub(f1, f0), g1 = dd_sub(f2, f1);
    const dd g2 = dd_sub(f3, f2), g3 = dd_sub(f4, f3);
    if constexpr (WM == 1) {
        const dd A = dd_sub(mul_raw(g1, 5.0), dd_scale(g0, 2.0));
        const dd B = dd_add(g1, dd_scale(g2, 2.0));
        const dd C = dd_sub(dd_scale(g2, 4.0), g3);
        // 6 (f - f_2) = C + omega_0 (A - C) + omega_1 (B - C)
        const dd s6 = dd_add(C, dd_add(mul_raw(dd_sub(A, C), w0d), mul_raw(dd_sub(B, C), w1d)));
        return dd_add(f2, mul_raw(s6, K.sixth));
    } else {
        const dd d0 = dd_sub_s(g1, g0), d2 = dd_sub_s(g3, g2);
        const dd e0 = dd_add_s(d0, dd_scale(g1, 2.0));
        const dd e1 = dd_add_s(g1, g2);
        const dd e2 = dd_sub_s(d2, dd_scale(g2, 2.0));
        const dd A = dd_sub_s(dd_scale(e0, 2.0), g1);
        const dd B = dd_add_s(e1, g2);
        const dd C = dd_sub_s(g2, e2);
        const dd d1 = dd_sub_s(g2, g1);
        // 1 / (12 (eps + IS_k)), 12 IS_k = 13 d^2 + 3 e^2
        auto recip_b = [&](dd d, dd e) {
            Acc b = acc(mul_raw(sq_raw(d), 13.0));
            b.add(mul_raw(sq_raw(e), 3.0));
            b.add(K.eps12);
            return dd_recip(b.get());
        };
        // weights times a common factor: alpha = (1, 6, 3) / (12 (eps + IS_k))^2
        const dd a0 = sq_raw(recip_b(d0, e0));
        const dd a1 = mul_raw(sq_raw(recip_b(d1, e1)), 6.0);
        const dd a2 = mul_raw(sq_raw(recip_b(d2, e2)), 3.0);
        Acc sum = acc(a0);
        sum.add(a1);
        sum.add(a2);
        const dd num = dd_add(two_products(a0, A, a1, B), mul_raw(a2, C));
        return dd_add(f2, mul_raw(num, dd_recip(dd_mul_d(sum.get(), 6.0))));
    }
}

// Workgroups of one launch (the threads of a grid are counted in 32 bits).
constexpr long long kMaxTiles = (1LL << 24) - 1;

template <int WM>
__global__ __launch_bounds__(256) void dd_stage_kernel(DDStageArgs a, int stage)
{
    __shared__ double2 shared[6][64];             // D of the Phi planes, theta parts and C Phi of the pi planes
    const int lane = threadIdx.x & 63;
    const int p = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int q = p & 1;                          // 0 real, 1 imaginary
    const unsigned tile = (unsigned)xcd_rank((int)blockIdx.x, (int)gridDim.x);
    const int k = __builtin_amdgcn_readfirstlane((int)(tile / (unsigned)a.nstrips));
    const int strip = (int)(tile - (unsigned)k * (unsigned)a.nstrips);
    const int nr = a.nr;
    const int j = strip * kStripPoints + lane;
    const bool inside = lane < kStripPoints && j < nr;
    const long long plane = a.plane;
    const long long row = (long long)k * nr;
    const unsigned at = (unsigned)min(j, nr - 1) * 16u;          // rows are < 2^27 points
    DDK K;
    K.inv_dx = {a.inv_dx[0], a.inv_dx[1]};
    K.ih1 = {a.ih1[0], a.ih1[1]};
    K.ih2 = {a.ih2[0], a.ih2[1]};
    K.ca = {a.ca[0], a.ca[1]};
    K.cb = {a.cb[0], a.cb[1]};
    K.sixth = {a.sixth[0], a.sixth[1]};
    K.eps12 = two_prod(a.eps, 12.0);
    auto state = [&](int r) { return (const double2*)a.uk + (r * plane + row); };
    auto coef = [&](int r) { return ld((const double2*)a.ctab + (r * plane + row), at); };

    // the radial derivative of plane p: f^+ on the Phi rows (speed b > 0, f^+_{j-1/2} from
    // f_{j-3..j+1}), f^- on the pi rows (speed -b, f^-_{j-1/2} from f_{j+2..j-2}: the f^+
    // form on the mirrored stencil)
    dd D, own;
    {
        const double2* P = state(p);
        dd w[5];
        if (strip > 0 && (strip + 1) * kStripPoints + 2 < nr) {     // no clamps
#pragma unroll
            for (int t = 0; t < 5; ++t) w[t] = ld(P, at + (p < 2 ? t - 3 : 2 - t) * 16);
        } else {
#pragma unroll
            for (int t = 0; t < 5; ++t) w[t] = ld(P, (unsigned)min(max(p < 2 ? j - 3 + t : j + 2 - t, 0), nr - 1) * 16u);
        }
        own = p < 2 ? w[3] : w[2];
        double w0 = 0.0, w1 = 0.0;
        if constexpr (WM == 1) {
            if (p < 2) {
                const double g[5] = {w[0].hi, w[1].hi, w[2].hi, w[3].hi, w[4].hi};
                w64_plus(g, a.eps, w0, w1);
            } else {
                const double g[5] = {w[4].hi, w[3].hi, w[2].hi, w[1].hi, w[0].hi};
                w64_minus(g, a.eps, w0, w1);
            }
        }
        const dd flux = weno<WM>(w[0], w[1], w[2], w[3], w[4], K, w0, w1);
        D = dd_mul(dd_sub(shfl_down1(flux), flux), K.inv_dx);
    }
    // of a complex product z w the real part is zr wr - zi wi, the imaginary part
    // zr wi + zi wr, and wave q holds w_q
    const double sg = q ? 1.0 : -1.0;
    dd F;
    if (p < 2) {
        // theta differences of this Phi plane with the pole ghosts, and C Phi (the pi waves'
        // work without it is about as much); F = pi - b D
        const double2* P = state(p);
        const dd c = own;
        const dd ghost = a.parity < 0 ? dd_neg(c) : c;
        const dd m = k > 0 ? ld(P - nr, at) : ghost;
        const dd pp = k < a.nth - 1 ? ld(P + nr, at) : ghost;
        const dd d1 = dd_mul(dd_sub(pp, m), K.ih1);
        const dd d2 = dd_mul(dd_add(dd_sub(pp, dd_scale(c, 2.0)), m), K.ih2);
        const dd T = two_products(coef(kDAth), d2, coef(kDBth), d1);
        const dd cp = two_products(coef(kDCr), own, dd_scale(coef(kDCi), sg), ld(state(1 - q), at));
        shared[q][lane] = make_double2(D.hi, D.lo);
        shared[2 + q][lane] = make_double2(T.hi, T.lo);
        shared[4 + q][lane] = make_double2(cp.hi, cp.lo);
        lds_sync();
        F = dd_sub(ld(state(2 + q), at), dd_mul(coef(kDB), D));
    } else {
        // F = b D - m3 D_Phi + Bt pi + theta part + C Phi (-lam2 d_x pi = b d_x pi in the
        // tortoise chart)
        const dd bp = two_products(coef(kDBtr), own, dd_scale(coef(kDBti), sg), ld(state(3 - q), at));
        F = dd_mul(coef(kDB), D);
        const dd m3r = coef(kDM3r), m3i = coef(kDM3i);
        lds_sync();
        const double2 Dq = shared[q][lane], Do = shared[1 - q][lane], T = shared[2 + q][lane], C = shared[4 + q][lane];
        const dd md = two_products(m3r, {Dq.x, Dq.y}, dd_scale(m3i, sg), {Do.x, Do.y});
        F = dd_add(dd_add(dd_add(dd_sub(F, md), bp), {T.x, T.y}), {C.x, C.y});
    }
    if (!inside) return;
    dd v;
    if (stage == 0) {
        v = F;
    } else {
        v = dd_add(own, dd_mul_d(F, a.dt));
        if (stage > 1) v = dd_add(dd_mul(K.ca, ld((const double2*)a.un + (p * plane + row), at)), dd_mul(K.cb, v));
    }
    st((double2*)a.out + (p * plane + row), at, v);
}

__global__ void dd_extract_kernel(const double2* u, long long plane, int nr, int nth, int j_e, double2* slot)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nth) return;
    slot[2 * k + 0] = u[(long long)k * nr + j_e];
    slot[2 * k + 1] = u[plane + (long long)k * nr + j_e];
}

// (hi, lo) -> TwoSum(hi, lo): the normalised pair of the same value.
__global__ void dd_normalise_kernel(double2* u, long long n)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 v = u[i];
    const dd s = two_sum(v.x, v.y);
    u[i] = make_double2(s.hi, s.lo);
}

}  // namespace

int launch_dd_stage(const DDStageArgs& a, int stage, int weight_prec, void* stream)
{
    if (a.nr < 1 || a.nth < 1 || a.nstrips < 1) return (int)hipErrorInvalidValue;
    const long long tiles = (long long)a.nstrips * a.nth;
    if (tiles > kMaxTiles) return (int)hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles);
    if (weight_prec == TEUK_W_FP64)
        hipLaunchKernelGGL(dd_stage_kernel<1>, grid, dim3(256), 0, (hipStream_t)stream, a, stage);
    else
        hipLaunchKernelGGL(dd_stage_kernel<0>, grid, dim3(256), 0, (hipStream_t)stream, a, stage);
    return (int)hipGetLastError();
}

int launch_dd_extract(const double* u, long long plane, int nr, int nth, int j_e, double* slot, void* stream)
{
    if (j_e < 0 || j_e >= nr) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(dd_extract_kernel, dim3((nth + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       (const double2*)u, plane, nr, nth, j_e, (double2*)slot);
    return (int)hipGetLastError();
}

int launch_dd_normalise(double* u, long long n, void* stream)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(dd_normalise_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       (double2*)u, n);
    return (int)hipGetLastError();
}

}  // namespace teuk
