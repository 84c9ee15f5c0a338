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
constexpr int kThinPoints = 51;
constexpr int kThinLead = 6;
constexpr int kThinRows = 12;                       // most output rows of a tile (16 waves)
constexpr int kThinStage = kWave + 6;               // staged u^n positions: point - 3 .. point + 3
constexpr int kThinPlane = kThinStage;              // LDS values per plane and row

template <int WP, bool kHyp>
__global__ __launch_bounds__((kThinRows + 4) * kWave, 4) void thin_step_kernel(StageArgs A, int rows)
{
    // a ring row of u^n and one of u(1) per wave; u(2) takes the place of u^n, whose last
    // reader has passed the barrier before it is written
    extern __shared__ double lds[];
    constexpr int W = kHyp && WP == TEUK_W_FP64 ? kWeno64H : WP;
    const auto K = weno_consts_for<W>(A.eps);
    const int nw = rows + 4;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int l = (int)threadIdx.x & (kWave - 1);
    const int nr = A.nr, nth = A.nth;
    const long long P = A.plane;
    const unsigned tiles = ((unsigned)nth + (unsigned)rows - 1) / (unsigned)rows;
    const unsigned rank = (unsigned)xcd_rank((int)blockIdx.x, (int)gridDim.x);
    const int strip = (int)(rank / tiles), k0 = (int)(rank - (unsigned)strip * tiles) * rows;
    const int k = k0 - 2 + w;                       // this wave's row
    const bool in_grid = k >= 0 && k < nth;
    const int kc = clampi(k, 0, nth - 1);
    const int p0 = strip * kThinPoints - kThinLead;
    const int j = p0 + l;
    const unsigned oc = (unsigned)clampi(j, 0, nr - 1) * 8u;
    const unsigned oa = (unsigned)clampi(p0 - 3 + l, 0, nr - 1) * 8u;
    const unsigned ob = (unsigned)clampi(p0 - 3 + kWave + l, 0, nr - 1) * 8u;
    const size_t row = (size_t)kc * nr;
    const bool first = w == 0, last = w == nw - 1;

    // every load is under way before the first is waited for
    double xa[4], xb[4], eR = 0.0, eI = 0.0;
#pragma unroll
    for (int p = 0; p < 4; ++p) xa[p] = row_get(A.uk + p * P + row, oa);
    if (l < kThinStage - kWave) {
#pragma unroll
        for (int p = 0; p < 4; ++p) xb[p] = row_get(A.uk + p * P + row, ob);
    }
    if (first || last) {                            // Phi of u^n beyond the tile
        const size_t r2 = (size_t)clampi(first ? k - 1 : k + 1, 0, nth - 1) * nr;
        eR = row_get(A.uk + r2, oc);
        eI = row_get(A.uk + P + r2, oc);
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
    __builtin_amdgcn_wave_barrier();

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
    // v + dt F(v) from the derivatives and the neighbours' Phi at the own point
    auto finish = [&](double upR, double upI, double dnR, double dnI) {
        if (k == nth - 1) {
            upR = A.parity * own[0];
            upI = A.parity * own[1];
        }
        if (k == 0) {
            dnR = A.parity * own[0];
            dnI = A.parity * own[1];
        }
        Four F;
        if constexpr (kHyp)
            F = rhs_h(hc, A.ih1, A.ih2, d[0], d[1], d[2], d[3], own[0], own[1], own[2], own[3], upR, upI, dnR, dnI);
        else
            F = rhs_t<bt_first<WP>()>(A, A.ih1, ct, d[0], d[1], d[2], d[3], own[0], own[1], own[2], own[3],
                                      theta2(own[0], upR, dnR), theta2(own[1], upI, dnI));
        Four v;
#pragma unroll
        for (int p = 0; p < 4; ++p) v.v[p] = euler(own[p], A.dt, F.v[p]);
        return v;
    };
    constexpr int kRow = 4 * kThinPlane;

    // ---- stage 1
    double un[4];
    fluxes([&](int p, int t) { return r0[p * kThinPlane + l + t]; });
    if constexpr (!kHyp) ct = point_coef_t(rt, pol, point_vsig(rt, pol.sn2));
#pragma unroll
    for (int p = 0; p < 4; ++p) un[p] = own[p];
    lds_sync();
    {
        double upR = eR, upI = eI, dnR = eR, dnI = eI;
        if (!last) upR = r0[kRow + l + 3], upI = r0[kRow + kThinPlane + l + 3];
        if (!first) dnR = r0[-kRow + l + 3], dnI = r0[-kRow + kThinPlane + l + 3];
        const Four v = finish(upR, upI, dnR, dnI);
#pragma unroll
        for (int p = 0; p < 4; ++p) r1[p * kThinPlane + l] = v.v[p];
    }
    __builtin_amdgcn_wave_barrier();
    int q[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) q[t] = clampi(l - 3 + t, lo, hi);

    // ---- stage 2
    const bool two = w >= 1 && w < nw - 1 && in_grid, three = w >= 2 && w < nw - 2 && in_grid;
    if (two) fluxes([&](int p, int t) { return r1[p * kThinPlane + q[t]]; });
    lds_sync();
    if (two) {
        const Four v = finish(r1[kRow + l], r1[kRow + kThinPlane + l], r1[-kRow + l], r1[-kRow + kThinPlane + l]);
#pragma unroll
        for (int p = 0; p < 4; ++p) r2[p * kThinPlane + l] = combine(0.75, un[p], 0.25, v.v[p]);
    }
    __builtin_amdgcn_wave_barrier();

    // ---- stage 3
    if (three) fluxes([&](int p, int t) { return r2[p * kThinPlane + q[t]]; });
    lds_sync();
    if (three) {
        const Four v = finish(r2[kRow + l], r2[kRow + kThinPlane + l], r2[-kRow + l], r2[-kRow + kThinPlane + l]);
        if (l >= kThinLead && l < kThinLead + kThinPoints && j < nr) {
#pragma unroll
            for (int p = 0; p < 4; ++p)
                row_put(A.out + p * P + row, oc, combine(1.0 / 3.0, un[p], 2.0 / 3.0, v.v[p]));
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
// chart H 600 x 300 16.0 and 14.3; three rounds 3000 x 100 21.3 and 20.0, 3000 x 150 25.0
// and 25.9, FP16 2000 x 150 28.6 and 31.4.
int thin_rows(int nr, int nth)
{
    static ResidentCache cache;
    int dev = 0;
    if (nr < 1 || hipGetDevice(&dev) != hipSuccess) return 0;
    const int cus = cache.get(dev, [&] {
        int n = 0;
        return hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess ? n : 0;
    });
    const long long strips = ((long long)nr + kThinPoints - 1) / kThinPoints;
    for (int rounds = 1; rounds <= 2; ++rounds) {
        const long long bands = (long long)cus * rounds / strips;    // tiles that a strip may have
        if (bands < 1) continue;
        const long long rows = (nth + bands - 1) / bands;
        if (rows <= kThinRows) return (int)rows;
    }
    return 0;
}

int launch_thin_step(const StageArgs& a, int rows, int weight_prec, int chart, void* stream)
{
    if (rows < 1 || rows > kThinRows || a.nr < 1 || a.nth < 2 || a.uk == a.out) return (int)hipErrorInvalidValue;
    const long long strips = ((long long)a.nr + kThinPoints - 1) / kThinPoints;
    const long long tiles = strips * (((long long)a.nth + rows - 1) / rows);
    if (tiles > (1LL << 21)) return (int)hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block((unsigned)(rows + 4) * kWave);
    const size_t shm = sizeof(double) * 2 * 4 * kThinPlane * (size_t)(rows + 4);
    hipStream_t st = (hipStream_t)stream;
    const bool hyp = chart == TEUK_CHART_HYPERBOLOIDAL;
    (void)hipGetLastError();
#define TEUK_THIN(W)                                                                                        \
    if (weight_prec == W) {                                                                                 \
        if (hyp) hipLaunchKernelGGL((thin_step_kernel<W, true>), grid, block, shm, st, a, rows);            \
        else hipLaunchKernelGGL((thin_step_kernel<W, false>), grid, block, shm, st, a, rows);               \
        return (int)hipGetLastError();                                                                      \
    }
    TEUK_THIN(TEUK_W_FP64)
    TEUK_THIN(TEUK_W_FP32)
    TEUK_THIN(TEUK_W_FP16)
    TEUK_THIN(TEUK_W_BF16)
#undef TEUK_THIN
    return (int)hipErrorInvalidValue;
}

}  // namespace teuk
