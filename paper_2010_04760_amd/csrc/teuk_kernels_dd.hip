// Double-double stage kernel (tortoise chart): the paper's quad-precision
// baseline of Sec. 3.1.3, with every state value carried as an unevaluated sum
// hi + lo of two doubles (106 significant bits) and the WENO weights either in
// double-double or, as in the paper's mixed variant, in double.
//
// Arithmetic: teuk_dd_math.h (all of it rounded exactly as written: the pragma below
// turns off multiply-add contraction; fused operations are spelled out as fma).
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
// Bound: FP64 VALU issue, 3 to 20 instructions for each operation, about 4000 a
// strip-row with double-double weights and 2730 with FP64 ones.  How many waves a SIMD
// gets one after the other decides small grids: with all four planes in one wave,
// 2048 x 64 gave some SIMDs three of them and most two.  2048 x 64 with double-double
// weights 82.2 -> 60.9 us a step, with FP64 weights 57.5 -> 44.3; 100 x 20 32.9 -> 15.7;
// 8192 x 256 880 -> 852 and 603 -> 604.
#include <hip/hip_runtime.h>

#include "teuk_dd_math.h"
#include "teuk_dd_tables.h"
#include "teuk_device.h"
#include "teuk_internal.h"

#pragma clang fp contract(off)

namespace teuk {

namespace {

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
    K.c13_3 = {a.c13_3[0], a.c13_3[1]};
#pragma unroll
    for (int i = 0; i < 3; ++i) K.d[i] = {a.d[i][0], a.d[i][1]};
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
        const dd flux = weno<WM>(w[0], w[1], w[2], w[3], w[4], K, a.eps, w0, w1);
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
