// Temporal blocking: one whole SSP-RK(3,3) step per launch.  The three stages
// of a tile are computed in one workgroup, the intermediate states u(1) and
// u(2) never leave LDS, and HBM sees one read of u^n and one write of u^{n+1} per
// point (64 B instead of 256 B per point-step).  The price is recomputation at
// the tile edges: a stage needs three radial neighbours and one theta neighbour
// of its input on each side.  (Device code and its launchers, a part of
// teuk_kernels.hip.)
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "teuk_coef.h"
#include "teuk_device.h"
#include "teuk_internal.h"

namespace teuk {

namespace {

// Radially a tile spans 127 points q = 0 .. 126, point q standing for
// j = 114 strip - 6 + q in all three stages, held by two waves: wave 0 points
// 0 .. 63, wave 1 points 63 .. 126.  The two overlap by one point so that every
// point but the last of each wave finds its j + 1/2 flux in the next lane of its
// own wave; point 63 is computed by wave 1 (wave 0's copy, lacking that flux, is
// never stored).  Stage 1 is valid on points 0 .. 125, stage 2 on 3 .. 122 and
// stage 3 (the output) on 6 .. 119: 114 outputs per 128 lanes.
constexpr int kBW = kBlockedPoints;      // output points per tile
constexpr int kBPts = 2 * kWave - 1;     // points of a tile (the waves share one)
constexpr int kBStage = kBPts + 6;       // staged u^n positions: q - 3 .. q + 3 of every point
constexpr int kBHalf = 2 * kWave;        // threads of one half
constexpr int kBThreads = 2 * kBHalf;    // two halves
constexpr int blocked_lead(int stages) { return 3 * (stages - 1); }            // first output point of a tile
constexpr int blocked_width(int stages) { return kBPts - 1 - 2 * blocked_lead(stages); }
static_assert(blocked_width(3) == kBW, "tile geometry");

// What the stages of a launch do.
enum BlockedKind : int {
    kBStep = 0,      // the three of an SSP-RK(3,3) step
    kBEuler3 = 1,    // three of the form v + dt F(v)
    kBLast2 = 2,     // one of that form and one that combines with u^n: out = ca u^n + cb (v + dt F(v)),
                     // and out2 = ca2 u^n + cb2 (...) if there is an out2, either of which may be u^n's own
                     // buffer (u^n is read at the own point only)
};

// Along theta a tile of rows [k0, k1) is marched by two such pairs of waves from
// its middle row kb outwards: half 1 takes kb, kb + 1, ... and half 0 kb - 1,
// kb - 2, ....  At step i a half stages its u^n row i + 1 (LDS, three-slot ring),
// computes u(1) at its row i, u(2) at i - 1 and u^{n+1} at i - 2.  Where the two
// meet, each finds the other's u(1) and u(2) rows in LDS one step after they
// were computed, so only the far ends recompute rows that belong to the
// neighbouring tiles (u(1) on two rows beyond, u(2) on one; a pole takes the
// parity ghost of the stage's own input): half the recomputation of a tile
// marched from one end, for the same rows per wave.
//
// One barrier a step orders all LDS traffic: every row read in step i was written
// in an earlier step, into a slot whose previous row was last read in an earlier
// step (three slots in each ring).
//
// A workgroup takes an equal share of the grid's strip-rows (strip by strip, the
// rows of a strip in order), in one tile per strip that its share touches, so
// that the last round of tiles does not leave part of the GPU idle: on
// 16384 x 512 whole tiles per strip would keep 432 of 512 workgroup slots busy.
//
// The arithmetic of each point and stage is the stage kernels', operation by
// operation; the per-point coefficients of a row are built once, by stage 1, and
// reused by stages 2 and 3 (a lane keeps its radial point through all three).
//
// Bound: FP64 VALU issue (HBM sees 75 B per point-step; 2.92e7 wave instructions a
// step of 8192 x 256, the SIMDs issuing them 80 % of the time at the 1.8 GHz that
// this load leaves).  The march is unrolled by three so that the values rolling
// over three rows (coefficients, u^n) and the three-slot rings keep fixed registers
// and addresses: with the copies, one-ended marches and 1024 one-tile workgroups
// of the form before it the step took 3.57e7 instructions and 87.5 us, now 74.9.
//
// Issue priority: the two waves of a SIMD belong to different workgroups, and a
// wave alone issues FP64 work at half the rate of two, so a stall of either costs
// its full length.  A wave's priority drops to 0 once the fluxes of its stage 1 are
// formed and rises stage by stage to 3 over the barrier into the next step: the two
// settle half a step apart, one computing while the other meets its barrier and
// its first LDS reads (8192 x 256 77.5 -> 74.9 us a step, 16384 x 512 302 -> 284,
// 4099 x 131 with FP32 weights 32.0 -> 29.7, chart H 16384 x 64 49.4 -> 46.2; steps
// down along the march, as in the stage kernel, 77.3, 295, 31.6 and 46.0).
//
// Hyperboloidal chart: the ten coefficients of a point are read once a step (loaded
// one row ahead) instead of once a stage, 144 B a point-step against 496, and a
// row's fluxes are taken on the side of its own speed: 16384 x 64 in 46.2 us where
// three launches of the stage kernel take 87.8 at 5.9 TB/s.
constexpr int kBS1 = 2 * 4 * 3 * kBStage;            // u(1) rings
constexpr int kBS2 = 2 * 4 * 3 * kBPts;              // u(2) rings, from the u(1) rings on

typedef const volatile __attribute__((address_space(3))) double* LdsLoad;
typedef __attribute__((address_space(3))) double* LdsDouble;
__device__ __forceinline__ LdsDouble lds_at(double* p)
{
    LdsDouble a = (LdsDouble)p;
    asm("" : "+v"(a));
    return a;
}
__device__ __forceinline__ double lds_get(LdsDouble p, int i) { return ((LdsLoad)p)[i]; }

// A value of a uniform row pointer, which is kept in scalar registers (the loop
// would otherwise carry it, and add to it, in vector registers).
typedef __attribute__((address_space(1))) char* GlobalChar;
__device__ __forceinline__ GlobalChar scalar(const double* p)
{
    GlobalChar g = (GlobalChar)const_cast<double*>(p);
    asm("" : "+s"(g));
    return g;
}
__device__ __forceinline__ double row_get(const double* row, unsigned off)
{
    return *(__attribute__((address_space(1))) const double*)(scalar(row) + off);
}
__device__ __forceinline__ void row_put(double* row, unsigned off, double v)
{
    *(__attribute__((address_space(1))) double*)(scalar(row) + off) = v;
}

// The four launches of an SSP-RK(10,4) step are made of the same parts: stages 1-3
// and 6-8 in one launch each (kBEuler3: three stages without u^n in them), 4-5 and
// 9-10 in one each (kBLast2: two stages, 120 outputs per tile, u^n read from memory
// for the second).  The split 3 + 2 + 3 + 2 lets the combining stages be the last of
// their launch, so that u^n is read at the own point alone and q = (u^n + 9 u(5)) / 25
// can take its buffer.  Ten stage launches took 188 us a step of 4096 x 256, these
// four 152; 1000 x 100 51 -> 40, 150 x 8 37 -> 27, 16384 x 180 475 -> 374, chart H
// 4096 x 256 289 -> 166, FP32 weights 4099 x 131 124 -> 104.  (The two-stage launch at
// three waves per SIMD, which its LDS would allow, spills 108 B a lane: 171 us.)
//
// Rows [k0, k1) of radial strip `strip` of one solve.  (Every wave of the workgroup
// calls it with the same arguments.)
template <int WP, bool kBtFirst, bool kHyp, int kKind = kBStep>
__device__ __forceinline__ void blocked_tile(const StageArgs& A, double* lds, int strip, int k0, int k1)
{
    constexpr int kStages = kKind == kBLast2 ? 2 : 3;
    constexpr int kWidth = blocked_width(kStages), kLead = blocked_lead(kStages);
    const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kBHalf);
    const int tid = (int)threadIdx.x - half * kBHalf;
    const int l = tid - (tid >= kWave ? 1 : 0);          // point of this lane in the tile
    const bool dup = tid == kWave - 1;                    // wave 0's copy of point 63
    const int nr = A.nr, nth = A.nth;
    const long long P = A.plane;
    constexpr int W = kHyp && WP == TEUK_W_FP64 ? kWeno64H : WP;
    const auto K = weno_consts_for<W>(A.eps);
    const double* ukp[4] = {A.uk, A.uk + P, A.uk + 2 * P, A.uk + 3 * P};
    double* outp[4] = {A.out, A.out + P, A.out + 2 * P, A.out + 3 * P};
    const int dir = half ? 1 : -1;
    const double ih1 = half ? A.ih1 : -A.ih1;
    // the middle row, with at least one grid row on either side of it
    int kb = (k0 + k1) >> 1;
    if (kb == 0) kb = 1;
    const int n0 = kb - k0, n1 = k1 - kb;             // rows of the halves (one may be 0)
    const int n = half ? n1 : n0;
    const int first = half ? kb : kb - 1;
    const int lim = half ? nth - kb : kb;             // grid rows from `first` on, in this half's direction
    const int N1 = min(n + kStages - 1, lim), N2 = min(n + kStages - 2, lim), NS = min(N1 + 1, lim);
    const int steps = max(n0, n1) + kStages - 1;

    const int p0 = strip * kWidth - kLead;            // grid point of tile point 0
    const int j = p0 + l;
    const unsigned oc = (unsigned)clampi(j, 0, nr - 1) * 8u;
    const unsigned oa = (unsigned)clampi(p0 - 3 + tid, 0, nr - 1) * 8u;            // staged position tid
    const unsigned ob = (unsigned)clampi(p0 - 3 + kBHalf + tid, 0, nr - 1) * 8u;   // position 128 + tid
    const bool halo = tid < kBStage - kBHalf;
    // radial ghosts of u(1), u(2): the end values, by clamping to the points inside the grid
    const int lo = clampi(-p0, 0, kBPts - 1), hi = clampi(nr - 1 - p0, 0, kBPts - 1);
    LdsDouble q[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) q[t] = lds_at(lds + kBS1 + half * 4 * 3 * kBPts + clampi(l - 3 + t, lo, hi));
    const LdsDouble own = lds_at(lds + kBS1 + half * 4 * 3 * kBPts + l);
    const LdsDouble across = lds_at(lds + kBS1 + (half ^ 1) * 4 * 3 * kBPts + l);
    const LdsDouble rows = lds_at(lds + half * 4 * 3 * kBStage + l), put = lds_at(lds + half * 4 * 3 * kBStage + tid);
    const bool out_lane = !dup && l >= kLead && l < kLead + kWidth && j < nr;
    Radial rt;
    if constexpr (!kHyp) rt = load_radial(A, oc);

    struct Row { double a[4], b[4]; };
    auto load_row = [&](Row& x, int i) {
        const size_t row = (size_t)(first + dir * i) * nr;
#pragma unroll
        for (int p = 0; p < 4; ++p) x.a[p] = row_get(ukp[p] + row, oa);
        if (halo) {
#pragma unroll
            for (int p = 0; p < 4; ++p) x.b[p] = row_get(ukp[p] + row, ob);
        }
    };
    auto store_row = [&](const Row& x, int b) {
#pragma unroll
        for (int p = 0; p < 4; ++p) put[(p * 3 + b) * kBStage] = x.a[p];
        if (halo) {
#pragma unroll
            for (int p = 0; p < 4; ++p) put[(p * 3 + b) * kBStage + kBHalf] = x.b[p];
        }
    };

    // The point's factors on one row.
    struct Point {
        PointCoef t;             // tortoise chart, built by stage 1
        double hc[kNCH];         // hyperboloidal chart, from the table
    };
    // One stage at one row for this lane, from the window w[p][t] (input of plane p
    // at j - 3 + t): the fluxes first, in the block that reads the window, so that
    // a plane's flux starts as its values arrive and covers the reads of the next;
    // then the rest with the input Phi at the own point on the rows ahead and behind.
    // (hyperboloidal chart: each plane on the side of its own speed at the point, both
    // sides in a wave whose lanes disagree; c holds the row's coefficients)
    struct Diffs { double d[4]; };
    auto fluxes = [&](auto read, double (&w)[4][6], const Point& c) {
        Diffs r;
        if constexpr (!kHyp) {
            Flux f[4];
            double fn[4];
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int t = p >> 1; t < 5 + (p >> 1); ++t) w[p][t] = read(p, t);
#pragma unroll
            for (int p = 0; p < 2; ++p) f[p] = Weno<W>::flux(w[p][0], w[p][1], w[p][2], w[p][3], w[p][4], K);
#pragma unroll
            for (int p = 2; p < 4; ++p) f[p] = Weno<W>::flux(w[p][5], w[p][4], w[p][3], w[p][2], w[p][1], K);
#pragma unroll
            for (int p = 0; p < 4; ++p) fn[p] = next_lane(f[p].y);
#pragma unroll
            for (int p = 0; p < 2; ++p) r.d[p] = plus_diff<W>(K, f[p], fn[p]);
#pragma unroll
            for (int p = 2; p < 4; ++p) r.d[p] = minus_diff<W>(K, f[p], fn[p]);
        } else {
            const bool up[2] = {c.hc[kHLam1] >= 0.0, c.hc[kHLam2] >= 0.0};
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                r.d[2 * q] = r.d[2 * q + 1] = 0.0;
                if (__any(up[q])) {
#pragma unroll
                    for (int p = 2 * q; p < 2 * q + 2; ++p) {
#pragma unroll
                        for (int t = 0; t < 5; ++t) w[p][t] = read(p, t);
                        const Flux f = Weno<W>::flux(w[p][0], w[p][1], w[p][2], w[p][3], w[p][4], K);
                        const double d = plus_diff<W>(K, f, next_lane(f.y));
                        if (up[q]) r.d[p] = d;
                    }
                }
                if (__any(!up[q])) {
#pragma unroll
                    for (int p = 2 * q; p < 2 * q + 2; ++p) {
#pragma unroll
                        for (int t = 1; t < 6; ++t) w[p][t] = read(p, t);
                        const Flux f = Weno<W>::flux(w[p][5], w[p][4], w[p][3], w[p][2], w[p][1], K);
                        const double d = minus_diff<W>(K, f, next_lane(f.y));
                        if (!up[q]) r.d[p] = d;
                    }
                }
                r.d[2 * q] *= A.inv6dx;
                r.d[2 * q + 1] *= A.inv6dx;
            }
        }
        return r;
    };
    auto finish = [&](const Diffs& r, const double (&w)[4][6], double ahR, double ahI, double bhR, double bhI,
                      const Point& c) {
        Four F;
        if constexpr (kHyp) {
            // symmetric in the rows ahead and behind but for the sign of ih1
            F = rhs_h(c.hc, ih1, A.ih2, r.d[0], r.d[1], r.d[2], r.d[3], w[0][3], w[1][3], w[2][3], w[3][3], ahR, ahI,
                      bhR, bhI);
        } else {
            // second differences as (up - 2 own) + down; a branch, as selects would
            // cost sixteen instructions
            Theta xR, xI;
            if (half) {
                xR = theta2(w[0][3], ahR, bhR);
                xI = theta2(w[1][3], ahI, bhI);
                asm volatile("" : "+v"(xR.d2));
            } else {
                xR = theta2(w[0][3], bhR, ahR);
                xI = theta2(w[1][3], bhI, ahI);
                asm volatile("" : "+v"(xI.d2));
            }
            xR.d1 = ahR - bhR;
            xI.d1 = ahI - bhI;
            F = rhs_t<kBtFirst>(A, ih1, c.t, r.d[0], r.d[1], r.d[2], r.d[3], w[0][3], w[1][3], w[2][3], w[3][3], xR, xI);
        }
        Four v;
#pragma unroll
        for (int p = 0; p < 4; ++p) v.v[p] = euler(w[p][3], A.dt, F.v[p]);
        return v;
    };

    Point pc[3];
    double un[3][4];                     // u^n at the own point, rows i, i - 1, i - 2
    double b0R, b0I;                     // Phi of u^n on row i - 1
    double a1R = 0, a1I = 0;             // Phi of u(1) on row i (its parity ghost beyond a pole)
    double b1R = 0, b1I = 0;             // ... on row i - 2
    double a2R = 0, a2I = 0;             // Phi of u(2) on row i - 1
    double b2R = 0, b2I = 0;             // ... on row i - 3
    // hyperboloidal chart: the coefficients of the next row, loaded one row ahead
    double hn[kNCH];
    auto load_coefs = [&](int i) {
        const double* c = A.ctab + (size_t)(first + dir * i) * nr;
#pragma unroll
        for (int q2 = 0; q2 < kNCH; ++q2) hn[q2] = row_get(c + (size_t)q2 * P, oc);
    };
    if constexpr (kHyp) load_coefs(0);
    // every load of the first rows is under way before the first is waited for (rows
    // past the last staged one are read again and not stored)
    Row ahead;
    {
        Row r0, r1;
        load_row(r0, 0);
        load_row(r1, min(1, NS - 1));
        load_row(ahead, min(2, NS - 1));
        const size_t row = (size_t)(first - dir) * nr;
        b0R = row_get(ukp[0] + row, oc);
        b0I = row_get(ukp[1] + row, oc);
        store_row(r0, 0);
        if (NS > 1) store_row(r1, 1);
    }

    auto step = [&](auto phase, int i) {
        constexpr int c0 = decltype(phase)::value, c1 = (c0 + 1) % 3, c2 = (c0 + 2) % 3;
        lds_sync();
        double un2[4];                   // two-stage launch: u^n at the own point on row i - 1
        const bool last2 = kKind == kBLast2 && i >= 1 && i - 1 < n;
        if (last2 && out_lane) {
            const size_t row = (size_t)(first + dir * (i - 1)) * nr;
#pragma unroll
            for (int p = 0; p < 4; ++p) un2[p] = row_get(A.un + p * P + row, oc);
        }
        if (i < N1) {
            // ---- stage 1 at row i: u(1) = u^n + dt F(u^n)
            __builtin_amdgcn_s_setprio(3);
            double w[4][6];
            double ahR = lds_get(rows, c1 * kBStage + 3), ahI = lds_get(rows, (3 + c1) * kBStage + 3);
            Polar pol;
            if constexpr (!kHyp) pol = load_polar(A, first + dir * i);
            if constexpr (kHyp) {
#pragma unroll
                for (int q2 = 0; q2 < kNCH; ++q2) pc[c0].hc[q2] = hn[q2];
                if (i + 1 < N1) load_coefs(i + 1);
            }
            const Diffs f = fluxes([&](int p, int t) { return lds_get(rows, (p * 3 + c0) * kBStage + t); }, w, pc[c0]);
            __builtin_amdgcn_s_setprio(0);
                if constexpr (!kHyp) pc[c0].t = point_coef_t(rt, pol, point_vsig(rt, pol.sn2));
            if (i + 1 >= lim) {          // a ghost row (the ring holds an older one)
                ahR = A.parity * w[0][3];
                ahI = A.parity * w[1][3];
            }
            const Four o = finish(f, w, ahR, ahI, b0R, b0I, pc[c0]);
            if (!dup) {
#pragma unroll
                for (int p = 0; p < 4; ++p) own[(p * 3 + c0) * kBPts] = o.v[p];
            }
            if constexpr (kKind == kBStep) {
#pragma unroll
                for (int p = 0; p < 4; ++p) un[c0][p] = w[p][3];
            }
            b0R = w[0][3];
            b0I = w[1][3];
            a1R = o.v[0];
            a1I = o.v[1];
        } else {                         // beyond the pole (or no longer needed)
            a1R *= A.parity;
            a1I *= A.parity;
        }
        if (i >= 1 && i - 1 < N2) {
            // ---- stage 2 at row i - 1: u(2) = 3/4 u^n + 1/4 (u(1) + dt F(u(1)))
            __builtin_amdgcn_s_setprio(1);
            if (c0 == 1 && i == 1) {     // across the middle: the other half's row 0
                b1R = lds_get(across, c2 * kBPts);
                b1I = lds_get(across, (3 + c2) * kBPts);
            }
            double w[4][6];
            const Diffs f = fluxes([&](int p, int t) { return lds_get(q[t], (p * 3 + c2) * kBPts); }, w, pc[c2]);
            const Four o = finish(f, w, a1R, a1I, b1R, b1I, pc[c2]);
            if constexpr (kKind == kBLast2) {
                if (out_lane) {
                    const size_t row = (size_t)(first + dir * (i - 1)) * nr;
#pragma unroll
                    for (int p = 0; p < 4; ++p) row_put(outp[p] + row, oc, combine(A.ca, un2[p], A.cb, o.v[p]));
                    if (A.out2) {
#pragma unroll
                        for (int p = 0; p < 4; ++p) row_put(A.out2 + p * P + row, oc, combine(A.ca2, un2[p], A.cb2, o.v[p]));
                    }
                }
            } else {
                Four u2 = o;
                if constexpr (kKind == kBStep) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) u2.v[p] = combine(0.75, un[c2][p], 0.25, o.v[p]);
                }
                if (!dup) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) own[kBS2 + (p * 3 + c2) * kBPts] = u2.v[p];
                }
                a2R = u2.v[0];
                a2I = u2.v[1];
            }
            b1R = w[0][3];
            b1I = w[1][3];
        } else {
            a2R *= A.parity;
            a2I *= A.parity;
        }
        if (kStages == 3 && i >= 2 && i - 2 < n) {
            // ---- stage 3 at row i - 2: u^{n+1} = 1/3 u^n + 2/3 (u(2) + dt F(u(2)))
            __builtin_amdgcn_s_setprio(2);
            if (c0 == 2 && i == 2) {
                b2R = lds_get(across, kBS2 + c1 * kBPts);
                b2I = lds_get(across, kBS2 + (3 + c1) * kBPts);
            }
            double w[4][6];
            const Diffs f = fluxes([&](int p, int t) { return lds_get(q[t], kBS2 + (p * 3 + c1) * kBPts); }, w, pc[c1]);
            const Four o = finish(f, w, a2R, a2I, b2R, b2I, pc[c1]);
            if (out_lane) {
                const size_t row = (size_t)(first + dir * (i - 2)) * nr;
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    row_put(outp[p] + row, oc, kKind == kBStep ? combine(1.0 / 3.0, un[c1][p], 2.0 / 3.0, o.v[p]) : o.v[p]);
            }
            b2R = w[0][3];
            b2I = w[1][3];
        }
        // row i + 2 into the slot of row i - 1
        if (i + 2 < NS) {
            store_row(ahead, c2);
            if (i + 3 < NS) load_row(ahead, i + 3);
        }
    };
    int i = 0;
    for (;;) {
        step(std::integral_constant<int, 0>{}, i);
        if (++i >= steps) break;
        step(std::integral_constant<int, 1>{}, i);
        if (++i >= steps) break;
        step(std::integral_constant<int, 2>{}, i);
        if (++i >= steps) break;
    }
}

// per half and plane, three-row rings of u^n (position s = point p0 - 3 + s) and
// of u(1) and u(2) (one value per point).  The planes are more than 255 values
// apart and the accesses go through opaque addresses plus immediate offsets:
// pairs of reads merged by the compiler would need an address of their own
// each (20 VALU instructions a step).
constexpr int kBLds = 2 * 4 * 3 * (kBStage + 2 * kBPts);
constexpr int kBLds2 = 2 * 4 * 3 * (kBStage + kBPts);      // two stages

// Strip-rows [at, end) of a rank: `share`, and one more for the first `extra` ranks
// (a grid has at most 2^34 / 114 + 2^16 strip-rows, a launch less than 2^31).
__device__ __forceinline__ void share_of(unsigned share, unsigned extra, unsigned& at, unsigned& end)
{
    const unsigned rank = (unsigned)xcd_rank((int)blockIdx.x, (int)gridDim.x);
    at = rank * share + min(rank, extra);
    end = at + share + (rank < extra ? 1u : 0u);
}

template <int WP, bool kBtFirst, bool kHyp>
__global__ __launch_bounds__(kBThreads, 2) void blocked_step_kernel(StageArgs A, unsigned share, unsigned extra)
{
    __shared__ double lds[kBLds];
    unsigned at, end;
    share_of(share, extra, at, end);
    while (at < end) {                                    // uniform over the workgroup
        const int strip = (int)(at / (unsigned)A.nth);
        const int k0 = (int)(at - (unsigned)strip * (unsigned)A.nth);
        const int k1 = min(k0 + (int)(end - at), A.nth);
        at += (unsigned)(k1 - k0);
        blocked_tile<WP, kBtFirst, kHyp>(A, lds, strip, k0, k1);
        lds_sync();   // before the next tile's rows go into the rings
    }
}

// Stages of an SSP-RK(10,4) step (the same walk over the strip-rows).
template <int WP, bool kHyp, int kKind>
__global__ __launch_bounds__(kBThreads, 2) void blocked_part_kernel(StageArgs A, unsigned share, unsigned extra)
{
    __shared__ double lds[kKind == kBLast2 ? kBLds2 : kBLds];
    unsigned at, end;
    share_of(share, extra, at, end);
    while (at < end) {
        const int strip = (int)(at / (unsigned)A.nth);
        const int k0 = (int)(at - (unsigned)strip * (unsigned)A.nth);
        const int k1 = min(k0 + (int)(end - at), A.nth);
        at += (unsigned)(k1 - k0);
        blocked_tile<WP, bt_first<WP>(), kHyp, kKind>(A, lds, strip, k0, k1);
        lds_sync();
    }
}

// The same step of several independent solves in one launch: member m owns the
// strip-rows [start[m], start[m + 1]) of the launch, which its workgroups share
// equally whatever solve they belong to, so that small solves together fill the
// GPU and no solve waits for another's last tiles.
template <int WP, bool kBtFirst, bool kHyp>
__global__ __launch_bounds__(kBThreads, 2) void group_blocked_kernel(const StageArgs* __restrict__ args,
                                                                     const unsigned* __restrict__ start, int nmem,
                                                                     unsigned share, unsigned extra)
{
    __shared__ double lds[kBLds];
    unsigned at, end;
    share_of(share, extra, at, end);
    while (at < end) {
        int lo = 0, hi = nmem - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (start[mid] <= at) lo = mid;
            else hi = mid - 1;
        }
        const StageArgs A = args[lo];
        const unsigned local = at - start[lo];
        const int strip = (int)(local / (unsigned)A.nth);
        const int k0 = (int)(local - (unsigned)strip * (unsigned)A.nth);
        const int k1 = min(k0 + (int)(end - at), A.nth);
        at += (unsigned)(k1 - k0);
        blocked_tile<WP, kBtFirst, kHyp>(A, lds, strip, k0, k1);
        lds_sync();
    }
}

}  // namespace

int blocked_grid(int weight_prec, int chart)
{
    static ResidentCache cache[4][2];
    int dev = 0;
    const bool hyp = chart == TEUK_CHART_HYPERBOLOIDAL;
    if (weight_prec < 0 || weight_prec > 3 || (chart != TEUK_CHART_TORTOISE && !hyp) || hipGetDevice(&dev) != hipSuccess)
        return 0;
    return cache[weight_prec][hyp].get(dev, [&] {
        int cus = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        const void* fn = nullptr;
#define TEUK_BGRID(W, F)                                                                                          \
    if (weight_prec == W)                                                                                         \
        fn = hyp ? (const void*)blocked_step_kernel<W, F, true> : (const void*)blocked_step_kernel<W, F, false>;
        TEUK_BGRID(TEUK_W_FP64, bt_first<TEUK_W_FP64>())
        TEUK_BGRID(TEUK_W_FP32, bt_first<TEUK_W_FP32>())
        TEUK_BGRID(TEUK_W_FP16, bt_first<TEUK_W_FP16>())
        TEUK_BGRID(TEUK_W_BF16, bt_first<TEUK_W_BF16>())
#undef TEUK_BGRID
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBThreads, 0);
        return e != hipSuccess || per_cu < 1 ? 0 : cus * per_cu;
    });
}

int launch_blocked_step(const StageArgs& a, int weight_prec, int chart, bool own_order, void* stream)
{
    if (a.nr < 1 || a.nth < 2 || a.nstrips < 1 || a.grid < 1 || (long long)a.grid > (long long)a.nstrips * a.nth ||
        (long long)a.nstrips * kBW < a.nr || (long long)a.nstrips * a.nth > (1LL << 31) - 1 || a.uk == a.out)
        return (int)hipErrorInvalidValue;
    (void)hipGetLastError();
    const dim3 grid((unsigned)a.grid), block(kBThreads);
    hipStream_t st = (hipStream_t)stream;
    const unsigned rows = (unsigned)((long long)a.nstrips * a.nth), g = (unsigned)a.grid;
    const bool hyp = chart == TEUK_CHART_HYPERBOLOIDAL;
    bool done = false;
#define TEUK_BLAUNCH(W, F)                                                                                     \
    if (!done && weight_prec == W && (W != TEUK_W_FP64 || hyp || own_order != F)) {                              \
        if (hyp) hipLaunchKernelGGL((blocked_step_kernel<W, F, true>), grid, block, 0, st, a, rows / g, rows % g); \
        else hipLaunchKernelGGL((blocked_step_kernel<W, F, false>), grid, block, 0, st, a, rows / g, rows % g);  \
        done = true;                                                                                             \
    }
    TEUK_BLAUNCH(TEUK_W_FP64, bt_first<TEUK_W_FP64>())
    TEUK_BLAUNCH(TEUK_W_FP32, bt_first<TEUK_W_FP32>())
    TEUK_BLAUNCH(TEUK_W_FP16, bt_first<TEUK_W_FP16>())
    TEUK_BLAUNCH(TEUK_W_BF16, bt_first<TEUK_W_BF16>())
    if (!done && weight_prec == TEUK_W_FP64) {
        hipLaunchKernelGGL((blocked_step_kernel<TEUK_W_FP64, !bt_first<TEUK_W_FP64>(), false>), grid, block, 0, st, a, rows / g,
                           rows % g);
        done = true;
    }
#undef TEUK_BLAUNCH
    if (!done) return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

// The kernel of a part, or null.
static const void* part_kernel(int stages, int weight_prec, int chart)
{
#define TEUK_PART(W, H)                                                                        \
    if (weight_prec == W && chart == (H ? TEUK_CHART_HYPERBOLOIDAL : TEUK_CHART_TORTOISE))     \
        return stages == 3 ? (const void*)blocked_part_kernel<W, H, kBEuler3>                  \
                           : (const void*)blocked_part_kernel<W, H, kBLast2>;
    TEUK_PART(TEUK_W_FP64, false)
    TEUK_PART(TEUK_W_FP64, true)
    TEUK_PART(TEUK_W_FP32, false)
    TEUK_PART(TEUK_W_FP32, true)
#undef TEUK_PART
    return nullptr;
}

int part_grid(int stages, int weight_prec, int chart)
{
    static ResidentCache cache[2][2][2];
    int dev = 0;
    const void* fn = stages == 2 || stages == 3 ? part_kernel(stages, weight_prec, chart) : nullptr;
    if (!fn || hipGetDevice(&dev) != hipSuccess) return 0;
    return cache[stages - 2][weight_prec == TEUK_W_FP32][chart == TEUK_CHART_HYPERBOLOIDAL].get(dev, [&] {
        int cus = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBThreads, 0) != hipSuccess)
            return 0;
        return cus * per_cu;
    });
}

int launch_blocked_part(StageArgs a, int stages, int weight_prec, int chart, void* stream)
{
    const int resident = part_grid(stages, weight_prec, chart);
    if (resident < 1 || a.nr < 1 || a.nth < 2 || a.uk == a.out || a.uk == a.out2) return (int)hipErrorInvalidValue;
    a.nstrips = (a.nr + blocked_width(stages) - 1) / blocked_width(stages);
    const long long rows = (long long)a.nstrips * a.nth;
    if (rows > (1LL << 31) - 1) return (int)hipErrorInvalidValue;
    a.grid = (int)(rows < resident ? rows : resident);
    unsigned share = (unsigned)rows / (unsigned)a.grid, extra = (unsigned)rows % (unsigned)a.grid;
    void* args[] = {&a, &share, &extra};
    (void)hipGetLastError();
    return (int)hipLaunchKernel(part_kernel(stages, weight_prec, chart), dim3((unsigned)a.grid), dim3(kBThreads), args, 0,
                                (hipStream_t)stream);
}

int launch_group_blocked(const StageArgs* args, const unsigned* start, int nmem, long long rows, int weight_prec,
                         int chart, void* stream)
{
    if (nmem < 1 || rows < 1 || rows > (1LL << 31) - 1) return (int)hipErrorInvalidValue;
    const int resident = blocked_grid(weight_prec, chart);
    if (resident < 1) return (int)hipErrorInvalidValue;
    const unsigned g = (unsigned)(rows < resident ? rows : resident), r = (unsigned)rows;
    const dim3 grid(g), block(kBThreads);
    hipStream_t st = (hipStream_t)stream;
    (void)hipGetLastError();
    const bool hyp = chart == TEUK_CHART_HYPERBOLOIDAL;
    bool done = false;
#define TEUK_GBLAUNCH(W, H)                                                                                         \
    if (weight_prec == W && hyp == H) {                                                                             \
        hipLaunchKernelGGL((group_blocked_kernel<W, bt_first<W>(), H>), grid, block, 0, st, args, start, nmem, r / g, r % g); \
        done = true;                                                                                                \
    }
    TEUK_GBLAUNCH(TEUK_W_FP64, false)
    TEUK_GBLAUNCH(TEUK_W_FP64, true)
    TEUK_GBLAUNCH(TEUK_W_FP32, false)
    TEUK_GBLAUNCH(TEUK_W_FP32, true)
    TEUK_GBLAUNCH(TEUK_W_FP16, false)
    TEUK_GBLAUNCH(TEUK_W_FP16, true)
    // (BF16 weights in the tortoise chart: groups step by stage launches)
    TEUK_GBLAUNCH(TEUK_W_BF16, true)
#undef TEUK_GBLAUNCH
    if (!done) return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

}  // namespace teuk
