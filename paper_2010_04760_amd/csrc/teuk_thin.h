// The temporally blocked SSP-RK(3,3) step for grids that leave the GPU nearly
// empty: one wave per theta row of a small tile, all rows of a stage at once.
// (Device code and its launcher, a part of teuk_kernels.hip.)
#pragma once

#include <hip/hip_runtime.h>

#include "teuk_blocked.h"
#include "teuk_coef.h"
#include "teuk_device.h"
#include "teuk_internal.h"

namespace teuk {

namespace {

// A tile is `rows` output rows of 51 output points.  Wave w of its rows + 4 waves
// owns grid row k0 - 2 + w through all three stages: u(1) on every row of the tile,
// u(2) on all but the first and last, u^{n+1} on the rows between.  Its lane l
// stands for point 51 strip - 6 + l: stage 1 is valid on points 0 .. 62 (the flux at
// j + 1/2 comes from the next lane), stage 2 on 3 .. 59, stage 3 on 6 .. 56.
//
// A stage's radial window comes from the wave's own row, which it wrote to LDS
// itself; only the theta neighbours come from other waves.  So the fluxes of a stage
// are formed before the barrier and the waves meet while each has work.
//
// Bound: the chain of three stages, each some 230 FP64 instructions that a wave alone
// on its SIMD issues at one per eight cycles (0.83 us), between a launch and the latency
// of the first loads (3 us).  The march of blocked_tile runs six stages one after the
// other even for a single row.  200 x 12 took 7.9 us a step by it and takes 5.4 here.
// The arithmetic of each point and stage is the same.
// Fourth-order theta differences take two rows more on each side of a stage, two-stage
// launches (kBLast2) one stage's rows and points less.
constexpr int kThinWaves = 16;                      // most rows of a tile, all stages'
constexpr int thin_lead(int stages) { return 3 * (stages - 1); }
constexpr int thin_points(int stages) { return kWave - 1 - 2 * thin_lead(stages); }
constexpr int thin_halo(int stages, int theta_order) { return (stages - 1) * (theta_order / 2); }
static_assert(thin_points(3) == 51 && thin_lead(3) == 6, "tile geometry");
constexpr int kThinStage = kWave + 6;               // staged u^n positions: point - 3 .. point + 3
constexpr int kThinPlane = kThinStage;              // LDS values per plane and row

template <int WP, int kChart, int kKind>
__global__ __launch_bounds__(kThinWaves * kWave, 4) void thin_step_kernel(StageArgs A, int rows)
{
    constexpr bool kHyp = kChart == kChartH, kTheta4 = kChart == kChartT4;
    constexpr int kStages = kKind == kBLast2 ? 2 : 3;
    constexpr int kReach = kTheta4 ? 2 : 1;                         // theta rows that a stage needs on either side
    constexpr int kHalo = kReach * (kStages - 1);
    constexpr int kPoints = thin_points(kStages), kLead = thin_lead(kStages);
    // a ring row of u^n and one of u(1) per wave; u(2) takes the place of u^n, whose last
    // reader has passed the barrier before it is written
    extern __shared__ double lds[];
    constexpr int W = kHyp && WP == TEUK_W_FP64 ? kWeno64H : WP;
    const auto K = weno_consts_for<W>(A.eps);
    const int nw = rows + 2 * kHalo;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int l = (int)threadIdx.x & (kWave - 1);
    const int nr = A.nr, nth = A.nth;
    const long long P = A.plane;
    const unsigned tiles = ((unsigned)nth + (unsigned)rows - 1) / (unsigned)rows;
    const unsigned rank = (unsigned)xcd_rank((int)blockIdx.x, (int)gridDim.x);
    const int strip = (int)(rank / tiles), k0 = (int)(rank - (unsigned)strip * tiles) * rows;
    const int k = k0 - kHalo + w;                   // this wave's row
    const bool in_grid = k >= 0 && k < nth;
    const int kc = clampi(k, 0, nth - 1);
    const int p0 = strip * kPoints - kLead;
    const int j = p0 + l;
    const unsigned oc = (unsigned)clampi(j, 0, nr - 1) * 8u;
    const unsigned oa = (unsigned)clampi(p0 - 3 + l, 0, nr - 1) * 8u;
    const unsigned ob = (unsigned)clampi(p0 - 3 + kWave + l, 0, nr - 1) * 8u;
    const size_t row = (size_t)kc * nr;

    // every load is under way before the first is waited for
    double xa[4], xb[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) xa[p] = row_get(A.uk + p * P + row, oa);
    if (l < kThinStage - kWave) {
#pragma unroll
        for (int p = 0; p < 4; ++p) xb[p] = row_get(A.uk + p * P + row, ob);
    }
    // Phi of u^n on the rows beyond the tile: e[0] at distance 1, e[1] at 2 (to the side
    // that the tile lacks; a tile has more than 2 kReach rows)
    double e[kReach][2];
#pragma unroll
    for (int d = 1; d <= kReach; ++d) {
        e[d - 1][0] = e[d - 1][1] = 0.0;
        if (w < d || w >= nw - d) {
            const size_t r2 = (size_t)clampi(w < d ? k - d : k + d, 0, nth - 1) * nr;
            e[d - 1][0] = row_get(A.uk + r2, oc);
            e[d - 1][1] = row_get(A.uk + P + r2, oc);
        }
    }
    const bool final = w >= kHalo && w < nw - kHalo && in_grid;
    const bool out_lane = l >= kLead && l < kLead + kPoints && j < nr;
    double un[4];
    if constexpr (kKind == kBLast2) {
        if (final && out_lane) {
#pragma unroll
            for (int p = 0; p < 4; ++p) un[p] = row_get(A.un + p * P + row, oc);
        }
    }
    PointCoef ct;
    double hc[kNCH];
    Radial rt;
    Polar pol;
    if constexpr (kHyp) {
#pragma unroll
        for (int q = 0; q < kNCH; ++q) hc[q] = row_get(A.ctab + (size_t)q * P + row, oc);
    } else {
        rt = load_radial(A, oc);
        pol = load_polar(A, kc);
    }

    double* r0 = lds + w * 4 * kThinPlane;                          // own row of u^n
    double* r1 = lds + (nw + w) * 4 * kThinPlane;                   // ... of u(1)
    double* r2 = r0;                                                // ... of u(2)
#pragma unroll
    for (int p = 0; p < 4; ++p) r0[p * kThinPlane + l] = xa[p];
    if (l < kThinStage - kWave) {
#pragma unroll
        for (int p = 0; p < 4; ++p) r0[p * kThinPlane + kWave + l] = xb[p];
    }
    wave_sync();

    const int lo = clampi(-p0, 0, kWave - 1), hi = clampi(nr - 1 - p0, 0, kWave - 1);
    double own[4], d[4];
    auto fluxes = [&](auto read) {
        if constexpr (!kHyp) {
            double v[4][6];
            Flux f[4];
            double fn[4];
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int t = p >> 1; t < 5 + (p >> 1); ++t) v[p][t] = read(p, t);
#pragma unroll
            for (int p = 0; p < 2; ++p) f[p] = Weno<W>::flux(v[p][0], v[p][1], v[p][2], v[p][3], v[p][4], K);
#pragma unroll
            for (int p = 2; p < 4; ++p) f[p] = Weno<W>::flux(v[p][5], v[p][4], v[p][3], v[p][2], v[p][1], K);
#pragma unroll
            for (int p = 0; p < 4; ++p) fn[p] = next_lane(f[p].y);
#pragma unroll
            for (int p = 0; p < 2; ++p) d[p] = plus_diff<W>(K, f[p], fn[p]);
#pragma unroll
            for (int p = 2; p < 4; ++p) d[p] = minus_diff<W>(K, f[p], fn[p]);
#pragma unroll
            for (int p = 0; p < 4; ++p) own[p] = v[p][3];
        } else {
            const bool up[2] = {hc[kHLam1] >= 0.0, hc[kHLam2] >= 0.0};
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                double v[6], x = 0.0;
#pragma unroll
                for (int t = 0; t < 6; ++t) v[t] = read(p, t);
                if (__any(up[p >> 1])) {
                    const Flux f = Weno<W>::flux(v[0], v[1], v[2], v[3], v[4], K);
                    const double y = plus_diff<W>(K, f, next_lane(f.y));
                    if (up[p >> 1]) x = y;
                }
                if (__any(!up[p >> 1])) {
                    const Flux f = Weno<W>::flux(v[5], v[4], v[3], v[2], v[1], K);
                    const double y = minus_diff<W>(K, f, next_lane(f.y));
                    if (!up[p >> 1]) x = y;
                }
                d[p] = x * A.inv6dx;
                own[p] = v[3];
            }
        }
    };
    // v + dt F(v) from the derivatives and the neighbours' Phi (nb[0] at k + 1, nb[1] at k - 1,
    // nb[2], nb[3] at k + 2, k - 2; Re and Im); beyond a pole row -1 - m is parity times row m
    auto finish = [&](double (&nb)[2 * kReach][2]) {
        if (k == nth - 1 || k == 0) {
            const int u = k == 0 ? 1 : 0, d = 1 - u;         // u: the side beyond the pole
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                nb[u][c] = A.parity * own[c];
                if constexpr (kTheta4) nb[2 + u][c] = A.parity * nb[d][c];
            }
        }
        if constexpr (kTheta4) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (k == nth - 2) nb[2][c] = A.parity * nb[0][c];
                if (k == 1) nb[3][c] = A.parity * nb[1][c];
            }
        }
        Four F;
        if constexpr (kHyp) {
            F = rhs_h(hc, A.ih1, A.ih2, d[0], d[1], d[2], d[3], own[0], own[1], own[2], own[3], nb[0][0], nb[0][1],
                      nb[1][0], nb[1][1]);
        } else {
            Theta x[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if constexpr (kTheta4) x[c] = theta4(own[c], nb[0][c], nb[1][c], nb[2][c], nb[3][c]);
                else x[c] = theta2(own[c], nb[0][c], nb[1][c]);
            }
            F = rhs_t<bt_first<WP>()>(A, A.ih1, ct, d[0], d[1], d[2], d[3], own[0], own[1], own[2], own[3], x[0], x[1]);
        }
        Four v;
#pragma unroll
        for (int p = 0; p < 4; ++p) v.v[p] = euler(own[p], A.dt, F.v[p]);
        return v;
    };
    constexpr int kRow = 4 * kThinPlane;
    // the neighbours' Phi at value `at` of the rows around r
    auto neighbours = [&](const double* r, int at, double (&nb)[2 * kReach][2]) {
#pragma unroll
        for (int m = 0; m < kReach; ++m)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                nb[2 * m][c] = r[(m + 1) * kRow + c * kThinPlane + at];
                nb[2 * m + 1][c] = r[-(m + 1) * kRow + c * kThinPlane + at];
            }
    };

    // ---- stage 1
    fluxes([&](int p, int t) { return r0[p * kThinPlane + l + t]; });
    if constexpr (!kHyp) ct = point_coef_t(rt, pol, point_vsig(rt, pol.sn2));
    if constexpr (kKind == kBStep) {
#pragma unroll
        for (int p = 0; p < 4; ++p) un[p] = own[p];
    }
    lds_sync();
    {
        double nb[2 * kReach][2];
#pragma unroll
        for (int m = 0; m < kReach; ++m)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                nb[2 * m][c] = nb[2 * m + 1][c] = e[m][c];
                if (w < nw - 1 - m) nb[2 * m][c] = r0[(m + 1) * kRow + c * kThinPlane + l + 3];
                if (w > m) nb[2 * m + 1][c] = r0[-(m + 1) * kRow + c * kThinPlane + l + 3];
            }
        const Four v = finish(nb);
#pragma unroll
        for (int p = 0; p < 4; ++p) r1[p * kThinPlane + l] = v.v[p];
    }
    wave_sync();
    int q[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) q[t] = clampi(l - 3 + t, lo, hi);

    // ---- stage 2
    const bool two = w >= kReach && w < nw - kReach && in_grid;
    if (two) fluxes([&](int p, int t) { return r1[p * kThinPlane + q[t]]; });
    lds_sync();
    if (two) {
        double nb[2 * kReach][2];
        neighbours(r1, l, nb);
        const Four v = finish(nb);
        if constexpr (kKind == kBLast2) {
            if (out_lane) {
#pragma unroll
                for (int p = 0; p < 4; ++p) row_put(A.out + p * P + row, oc, combine(A.ca, un[p], A.cb, v.v[p]));
                if (A.out2) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) row_put(A.out2 + p * P + row, oc, combine(A.ca2, un[p], A.cb2, v.v[p]));
                }
            }
        } else {
#pragma unroll
            for (int p = 0; p < 4; ++p)
                r2[p * kThinPlane + l] = kKind == kBStep ? combine(0.75, un[p], 0.25, v.v[p]) : v.v[p];
        }
    }
    if constexpr (kStages == 3) {
        wave_sync();

        // ---- stage 3
        if (final) fluxes([&](int p, int t) { return r2[p * kThinPlane + q[t]]; });
        lds_sync();
        if (final) {
            double nb[2 * kReach][2];
            neighbours(r2, l, nb);
            const Four v = finish(nb);
            if (out_lane) {
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    row_put(A.out + p * P + row, oc,
                            kKind == kBStep ? combine(1.0 / 3.0, un[p], 2.0 / 3.0, v.v[p]) : v.v[p]);
            }
        }
    }
}

}  // namespace

// Output rows of a tile, or 0 for a grid that the marched launch takes.  A compute
// unit runs one such workgroup (of up to 16 waves) at a time, and its time grows
// little with its rows, so the tiles are as low as they can be with all of them under
// way at once: 512 x 32 in tiles of 1, 2 and 4 rows takes 6.9, 5.8 and 6.2 us a step
// (352, 176 and 88 tiles on 256 compute units), 1024 x 64 in tiles of 5, 6 and 8 rows 11.8,
// 7.6 and 8.1.  Where 12 rows are too few for that, two rounds of tiles still beat the
// marched launch (its workgroups have a few rows each, and 3 to 4 more to recompute),
// three do not always: us a step, marched launch against this one, FP64 weights unless
// named: one round 200 x 12 7.9 and 5.4, 512 x 32 8.05 and 5.8 (FP32 9.5 and 6.25), 1024 x 64
// 11.5 and 7.55, 1200 x 90 11.6 and 9.2 (BF16 21.6 and 17.6), chart H 1500 x 80 15.8 and
// 9.3; two rounds 1500 x 120 15.4 and 14.0, 2600 x 118 21.3 and 18.6 (BF16 44.6 and 35.2),
// chart H 600 x 300 16.0 and 14.3, SSP-RK(10,4) 150 x 8 26.9 and 18.4, 1000 x 100 40 and 32;
// three rounds 3000 x 100 21.3 and 20.0, 3000 x 150 25.0
// and 25.9, FP16 2000 x 150 28.6 and 31.4.  Fourth-order theta differences (tiles of at
// most 8 rows) have stage launches instead: 200 x 12 12.7 and 6.55, 1024 x 64 16.2 and 9.0,
// two rounds 1500 x 80 17.6 and 15.5, FP32 600 x 200 18.5 and 16.3.
int thin_rows(int nr, int nth, int theta_order)
{
    static ResidentCache cache;
    int dev = 0;
    if (nr < 1 || hipGetDevice(&dev) != hipSuccess) return 0;
    const int cus = cache.get(dev, [&] {
        int n = 0;
        return hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess ? n : 0;
    });
    const long long strips = ((long long)nr + thin_points(3) - 1) / thin_points(3);
    for (int rounds = 1; rounds <= 2; ++rounds) {
        const long long bands = (long long)cus * rounds / strips;    // tiles that a strip may have
        if (bands < 1) continue;
        const long long rows = (nth + bands - 1) / bands;
        if (rows <= kThinWaves - 2 * thin_halo(3, theta_order)) return (int)rows;
    }
    return 0;
}

long long thin_tiles(int nr, int nth, int rows, int stages)
{
    const int points = thin_points(stages);
    return ((long long)nr + points - 1) / points * (((long long)nth + rows - 1) / rows);
}

// stages and kind as in launch_blocked_part
static int launch_thin(const StageArgs& a, int rows, int stages, const void* fn, int theta_order, void* stream)
{
    const int waves = rows + 2 * thin_halo(stages, theta_order);
    if (!fn || rows < 1 || waves > kThinWaves || a.nr < 1 || a.nth < 2 || a.uk == a.out || a.uk == a.out2)
        return (int)hipErrorInvalidValue;
    const long long tiles = thin_tiles(a.nr, a.nth, rows, stages);
    if (tiles > (1LL << 21)) return (int)hipErrorInvalidValue;
    StageArgs b = a;
    void* args[] = {&b, &rows};
    (void)hipGetLastError();
    return (int)hipLaunchKernel(fn, dim3((unsigned)tiles), dim3((unsigned)waves * kWave), args,
                                sizeof(double) * 2 * 4 * kThinPlane * (size_t)waves, (hipStream_t)stream);
}

int launch_thin_step(const StageArgs& a, int rows, int weight_prec, int chart, void* stream)
{
    const void* fn = nullptr;
#define TEUK_THIN(W)                                                                        \
    if (weight_prec == W)                                                                   \
        fn = chart == kChartH    ? (const void*)thin_step_kernel<W, kChartH, kBStep>        \
             : chart == kChartT4 ? (const void*)thin_step_kernel<W, kChartT4, kBStep>       \
             : chart == kChartT  ? (const void*)thin_step_kernel<W, kChartT, kBStep>        \
                                 : nullptr;
    TEUK_THIN(TEUK_W_FP64)
    TEUK_THIN(TEUK_W_FP32)
    TEUK_THIN(TEUK_W_FP16)
    TEUK_THIN(TEUK_W_BF16)
#undef TEUK_THIN
    return launch_thin(a, rows, 3, fn, chart == kChartT4 ? 4 : 2, stream);
}

int launch_thin_part(const StageArgs& a, int rows, int stages, int weight_prec, int chart, void* stream)
{
    const void* fn = nullptr;
#define TEUK_THIN(W, C)                                                                     \
    if (weight_prec == W && chart == C)                                                     \
        fn = stages == 3 ? (const void*)thin_step_kernel<W, C, kBEuler3> : (const void*)thin_step_kernel<W, C, kBLast2>;
    TEUK_THIN(TEUK_W_FP64, kChartT)
    TEUK_THIN(TEUK_W_FP64, kChartH)
    TEUK_THIN(TEUK_W_FP32, kChartT)
    TEUK_THIN(TEUK_W_FP32, kChartH)
#undef TEUK_THIN
    return launch_thin(a, rows, stages, fn, 2, stream);
}

}  // namespace teuk
