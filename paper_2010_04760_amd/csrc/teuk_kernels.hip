// Device kernels of libteuk for gfx950 (CDNA4, wave64).
//
// Hot path: one fused kernel per SSP-RK(3,3) stage (paper Sec. 3.2) that
// evaluates F(u) = -(M d_x u + L u + A u) of eq. evln and combines it with u^n:
//   - WENO5 interface fluxes per real plane (Sec. 3.1.2): Phi_R, Phi_I with the
//     f^+ treatment (speed +b), pi_R, pi_I with the f^- treatment (speed -b);
//   - flux differences (f_{j+1/2} - f_{j-1/2}) / dx;
//   - second-order centred theta differences of Phi (Sec. 3.1);
//   - complex 2x2 blocks of M, A, L with per-point coefficients rebuilt from
//     radial and polar tables;
//   - u^(k+1) = ca u^n + cb (u^(k) + dt F).
//
// Work decomposition.  A workgroup is one wave of 64 lanes.  It owns a radial
// strip of 63 points and marches over a chunk of theta rows.  Per row the wave
// stages the strip plus a 3/2-cell halo of the four planes in LDS (coalesced
// along the radial index), each lane computes the four fluxes of the interface
// just left of its point, and takes the flux of the interface on its right from
// the next lane, so every interface flux is computed once.  The Phi values of
// the rows above and below the own point stay in registers across the march,
// as do the thirteen radial coefficient factors; the polar factors of a row
// are uniform across the wave.  Tiles are ordered theta-chunk fastest and
// dealt to the eight XCDs in contiguous ranges, so neighbouring chunks (which
// share boundary rows) run on the same L2.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "teuk_blocked.h"
#include "teuk_thin.h"
#include "teuk_coef.h"
#include "teuk_device.h"
#include "teuk_internal.h"

namespace teuk {

namespace {

constexpr int kRow = kWave + 5;   // staged positions j0-3 .. j0+65

// What a stage launch writes.
constexpr int kStageFirst = 0;    // out = u + dt F(u)
constexpr int kStageLater = 1;    // out = ca u^n + cb (u^(k) + dt F(u^(k)))
constexpr int kRhsOnly = 2;       // out = F(u)
constexpr int kStageDual = 3;     // v = u^(k) + dt F(u^(k)): out = ca u^n + cb v, out2 = ca2 u^n + cb2 v
// stage modes that read u^n at the own point
template <int kMode>
constexpr bool reads_un() { return kMode == kStageLater || kMode == kStageDual; }

// ---------------------------------------------------------------- chart-T row pipeline
// The tortoise-chart stage streams each theta row of the four planes straight
// from HBM into a four-row LDS ring with LDS-DMA loads (global_load_lds: every
// lane moves one dword, no VGPRs involved), three rows ahead of the row being
// computed.  The compiler does not model these loads, so they and the u^n
// loads are issued from inline assembly and waited for with explicit vmcnt
// counts.  Each count covers only the loads issued here; any other memory
// operation the compiler places in between can only make a wait stricter.
constexpr int kRowP = 72;                                   // LDS row stride (doubles)
constexpr int kRing = 4;                                    // rows in the LDS ring
constexpr unsigned kPlaneBytes = kRowP * 8;                 // 576
constexpr unsigned kSlotBytes = 4 * kPlaneBytes;            // 2304

// One LDS-DMA dword per lane: LDS[m0 + 4 lane] = global[sbase + voff].  The
// LDS address reaches m0 through an operand constrained to that register, so
// the compiler writes m0 itself and knows the instruction reads it.
__device__ __forceinline__ void dma_dword(unsigned voff, const double* sbase, unsigned lds)
{
    asm volatile("global_load_lds_dword %0, %1" : : "v"(voff), "s"(sbase), "{m0}"(lds) : "memory");
}

// A double from global memory whose arrival is waited for explicitly: the
// register holds the value only after the vm_wait that takes it as an operand.
// Until then no instruction may read, copy or reuse it; the compiler sees the
// value as ready at once, so this is checked in the built assembly (every
// wait names its operands in a comment for that check).
__device__ __forceinline__ double ld_async(unsigned voff, const double* sbase)
{
    double v;
    asm volatile("global_load_dwordx2 %0, %1, %2 ; async-load" : "=&v"(v) : "v"(voff), "s"(sbase) : "memory");
    return v;
}

// Wait until at most N vector-memory operations are outstanding.
template <int N>
__device__ __forceinline__ void vm_wait()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
// The same, also making four values depend on the wait (so that no use of
// them can be scheduled before it).
template <int N>
__device__ __forceinline__ void vm_wait(double& a, double& b, double& c, double& d)
{
    asm volatile("s_waitcnt vmcnt(%4) ; async-wait %0 %1 %2 %3" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N) : "memory");
}

// Agent-coherent forms of the row traffic (the sc1 cache policy that the
// compiler gives agent-scope atomics: not served from a non-coherent cache
// line, and stores written through), for the pipelined step, whose workgroups
// on any CU or XCD exchange tiles without cache write-back or invalidation.
// With kCoh false they are the plain forms above.
template <bool kCoh>
__device__ __forceinline__ double ldb_c(const double* base, unsigned off)
{
    if constexpr (kCoh) {
        const unsigned long long* q =
            reinterpret_cast<const unsigned long long*>(reinterpret_cast<const char*>(base) + off);
        return __longlong_as_double((long long)__hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    } else {
        return ldb(base, off);
    }
}
template <bool kCoh>
__device__ __forceinline__ void stb_c(double* base, unsigned off, double v)
{
    if constexpr (kCoh) {
        unsigned long long* q = reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(base) + off);
        __hip_atomic_store(q, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        stb(base, off, v);
    }
}
template <bool kCoh>
__device__ __forceinline__ void dma_dword_c(unsigned voff, const double* sbase, unsigned lds)
{
    if constexpr (kCoh)
        asm volatile("global_load_lds_dword %0, %1 sc1" : : "v"(voff), "s"(sbase), "{m0}"(lds) : "memory");
    else
        dma_dword(voff, sbase, lds);
}
template <bool kCoh>
__device__ __forceinline__ double ld_async_c(unsigned voff, const double* sbase)
{
    if constexpr (kCoh) {
        double v;
        asm volatile("global_load_dwordx2 %0, %1, %2 sc1 ; async-load" : "=&v"(v) : "v"(voff), "s"(sbase) : "memory");
        return v;
    } else {
        return ld_async(voff, sbase);
    }
}

// The results of one point: what the launch's mode writes, from F(u^(k)), the
// point's own values and (stages 2, 3 and the dual stage) those of u^n.
template <int kMode, bool kCoh = false>
__device__ __forceinline__ void write_point(const StageArgs& A, size_t row, unsigned oc, const Four& F, double phR,
                                            double phI, double piR, double piI, double n0, double n1, double n2,
                                            double n3)
{
    const double own[4] = {phR, phI, piR, piI}, un[4] = {n0, n1, n2, n3};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        double* out = A.out + p * A.plane + row;
        const double v = euler(own[p], A.dt, F.v[p]);
        if (kMode == kRhsOnly) stb_c<kCoh>(out, oc, F.v[p]);
        else if (kMode == kStageFirst) stb_c<kCoh>(out, oc, v);
        else stb_c<kCoh>(out, oc, combine(A.ca, un[p], A.cb, v));
        if (kMode == kStageDual) stb_c<kCoh>(A.out2 + p * A.plane + row, oc, combine(A.ca2, un[p], A.cb2, v));
    }
}

// Hyperboloidal chart: one radial strip [j0, j0 + 63) marched over the theta
// rows [k0, k1), upward (dir = +1, from k0) or downward (dir = -1, from
// k1 - 1).  Rows are staged in a two-row LDS ring: while row k is computed
// from LDS, the loads of row k + 2 dir and of u^n at row k are already in
// flight and are consumed at the end of the iteration, so each wave always has
// its next rows' memory traffic overlapping its arithmetic.  The ten
// coefficients of the point are read from the per-point table, and each row
// takes the flux side of the sign of its own speed at the point (speed >= 0:
// f^+, speed < 0: f^-); a wave whose lanes disagree computes both sides and
// each lane differences its own.
template <int WP, int kMode>
__device__ __forceinline__ void march_strip_h(const StageArgs& A, double (*s)[4][kRow], int strip, int k0, int k1,
                                              int dir)
{
    const int l = threadIdx.x;
    const int nr = A.nr, nth = A.nth;
    const long long P = A.plane;
    const int j0 = strip * kStripPoints;
    const int j = j0 + l;
    const bool active = (l < kStripPoints) && (j < nr);
    const int jc = min(j, nr - 1);
    // byte offsets within a row (rows are < 2^27 doubles, so these fit in 32 bits)
    const unsigned oa = (unsigned)clampi(j0 - 3 + l, 0, nr - 1) * 8u;    // LDS index l
    const unsigned ob = (unsigned)clampi(j0 + 61 + l, 0, nr - 1) * 8u;   // LDS index 64 + l, l < 5
    const unsigned oc = (unsigned)jc * 8u;                                 // own point
    const bool halo = l < 5;
    const double* __restrict__ ukp[4] = {A.uk, A.uk + P, A.uk + 2 * P, A.uk + 3 * P};
    const double* unp[4] = {A.un, A.un + P, A.un + 2 * P, A.un + 3 * P};   // read where reads_un<kMode>()

    constexpr int HW = WP == TEUK_W_FP64 ? kWeno64H : WP;
    const auto K = weno_consts_for<HW>(A.eps);

    const int n = k1 - k0;
    const int first = dir > 0 ? k0 : k1 - 1;
    // Phi at the own point on the row behind the first one (pole ghost past
    // either pole).
    double bhR, bhI;
    {
        const int kb = first - dir;
        if (kb >= 0 && kb < nth) {
            bhR = ldb(ukp[0] + (size_t)kb * nr, oc);
            bhI = ldb(ukp[1] + (size_t)kb * nr, oc);
        } else {
            bhR = A.parity * ldb(ukp[0] + (size_t)first * nr, oc);
            bhI = A.parity * ldb(ukp[1] + (size_t)first * nr, oc);
        }
    }

    // Rows staged: first + dir i for i = 0 .. nst-1, i.e. every computed row
    // plus the one ahead of the last (its theta neighbour) unless that is past
    // a pole.
    const int ahead_last = first + dir * n;
    const int nst = (ahead_last >= 0 && ahead_last < nth) ? n + 1 : n;
    double xa[4], xb[4];
    auto load_row = [&](int k) {
        const size_t row = (size_t)k * nr;
#pragma unroll
        for (int p = 0; p < 4; ++p) xa[p] = ldb(ukp[p] + row, oa);
        if (halo) {
#pragma unroll
            for (int p = 0; p < 4; ++p) xb[p] = ldb(ukp[p] + row, ob);
        }
    };
    auto store_row = [&](int buf) {
#pragma unroll
        for (int p = 0; p < 4; ++p) s[buf][p][l] = xa[p];
        if (halo) {
#pragma unroll
            for (int p = 0; p < 4; ++p) s[buf][p][kWave + l] = xb[p];
        }
    };
    load_row(first);
    store_row(0);
    if (nst > 1) {
        load_row(first + dir);
        store_row(1);
    }

    for (int i = 0; i < n; ++i) {
        const int k = first + dir * i;
        const int b = i & 1;
        const size_t row = (size_t)k * nr;
        // next rows' traffic, consumed at the end of this iteration
        const bool pre = i + 2 < nst;
        if (pre) load_row(k + 2 * dir);
        double n0 = 0.0, n1 = 0.0, n2 = 0.0, n3 = 0.0;
        if (reads_un<kMode>()) {
            n0 = ldb(unp[0] + row, oc);
            n1 = ldb(unp[1] + row, oc);
            n2 = ldb(unp[2] + row, oc);
            n3 = ldb(unp[3] + row, oc);
        }
        double hc[kNCH];
#pragma unroll
        for (int q = 0; q < kNCH; ++q) hc[q] = ldb(A.ctab + (size_t)q * P + row, oc);
        lds_sync();

        double dPhR, dPhI, dPiR, dPiI;
        {
            // upwind side per lane and row: speed >= 0 -> f^+, speed < 0 -> f^-
            const bool up1 = hc[kHLam1] >= 0.0, up2 = hc[kHLam2] >= 0.0;
            auto deriv = [&](int p, bool up, bool any_up, bool any_dn) {
                double d = 0.0;
                if (any_up) {
                    const Flux f = Weno<HW>::flux(s[b][p][l], s[b][p][l + 1], s[b][p][l + 2], s[b][p][l + 3], s[b][p][l + 4], K);
                    const double dp = plus_diff<HW>(K, f, next_lane(f.y));
                    if (up) d = dp;
                }
                if (any_dn) {
                    const Flux f = Weno<HW>::flux(s[b][p][l + 5], s[b][p][l + 4], s[b][p][l + 3], s[b][p][l + 2], s[b][p][l + 1], K);
                    const double dm = minus_diff<HW>(K, f, next_lane(f.y));
                    if (!up) d = dm;
                }
                return d * A.inv6dx;
            };
            const bool up1_any = __any(active && up1), dn1_any = __any(active && !up1);
            const bool up2_any = __any(active && up2), dn2_any = __any(active && !up2);
            dPhR = deriv(0, up1, up1_any, dn1_any);
            dPhI = deriv(1, up1, up1_any, dn1_any);
            dPiR = deriv(2, up2, up2_any, dn2_any);
            dPiI = deriv(3, up2, up2_any, dn2_any);
        }
        const double phR = s[b][0][l + 3], phI = s[b][1][l + 3];
        const double piR = s[b][2][l + 3], piI = s[b][3][l + 3];
        double ahR, ahI;   // Phi on the row ahead (k + dir)
        if (i + 1 < nst) {
            ahR = s[b ^ 1][0][l + 3];
            ahI = s[b ^ 1][1][l + 3];
        } else {
            ahR = A.parity * phR;
            ahI = A.parity * phI;
        }

        if (active) {
            // rows k+1 and k-1
            const double upR = dir > 0 ? ahR : bhR, upI = dir > 0 ? ahI : bhI;
            const double dnR = dir > 0 ? bhR : ahR, dnI = dir > 0 ? bhI : ahI;
            const Four F = rhs_h(hc, A.ih1, A.ih2, dPhR, dPhI, dPiR, dPiI, phR, phI, piR, piI, upR, upI, dnR, dnI);

            write_point<kMode>(A, row, oc, F, phR, phI, piR, piI, n0, n1, n2, n3);
        }
        bhR = phR;
        bhI = phI;
        lds_sync();               // every lane is done reading s[b] (row k)
        if (pre) store_row(b);    // row k + 2 dir takes its place
    }
}

// Chart-T march of one strip over rows [k0, k1) with the LDS-DMA row pipeline.
// Row i of the march (k = first + dir i) lives in ring slot i mod 4; the
// rows first, first + dir, first + 2 dir are issued before the loop and row
// i + 3 at the top of iteration i.  Where the march has no such row, one
// cache line is loaded into the free slot instead, so that every iteration
// issues the same operations and the wait counts are constants:
//     per iteration: [u^n of row i: 4 loads (later stages)] [row i + 3: 12 DMA];
//     before reading rows i and i + 1: everything up to row i + 1 has landed,
//         i.e. vmcnt <= (12 + it) at i = 0 and vmcnt <= 2 it for i >= 1,
//         it = loads per iteration (16 later stages, 12 otherwise);
//     before the stores: u^n of row i has landed, vmcnt <= 12.
// kTh4 (fourth-order theta differences) also reads Phi on row i + 2, so it
// waits for everything up to row i + 2 (vmcnt <= it at every i), keeps the
// two rows behind in registers, and stages up to two rows past the segment.
// Beyond a pole, ghost row -1 - g is parity x row g (and row nth + g is
// parity x row nth - 1 - g): the ahead rows then come from the rows already
// at hand (row k + 2 dir mirrors k + dir when only it is a ghost, and k - dir
// when both are).
template <int WP, int kMode, bool kLevel, bool kCoh = false, bool kTh4 = false>
__device__ __forceinline__ void march_strip_t(const StageArgs& A, char* ring, int strip, int k0, int k1, int dir)
{
    const int l = threadIdx.x;
    const int nr = A.nr, nth = A.nth;
    const long long P = A.plane;
    const int j0 = strip * kStripPoints;
    const int j = j0 + l;
    const bool active = (l < kStripPoints) && (j < nr);
    const int jc = min(j, nr - 1);
    const unsigned oc = (unsigned)jc * 8u;                                 // own point
    // staged dword d = 64 c + l of a row holds half (d & 1) of position j0 - 3 + d/2
    unsigned od[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int d = 64 * c + l;
        od[c] = (unsigned)clampi(j0 - 3 + (d >> 1), 0, nr - 1) * 8u + (unsigned)(d & 1) * 4u;
    }
    const unsigned lds0 = (unsigned)(size_t)ring;          // LDS byte address of the ring
    const double* ukp[4] = {A.uk, A.uk + P, A.uk + 2 * P, A.uk + 3 * P};
    const double* unp[4] = {A.un, A.un + P, A.un + 2 * P, A.un + 3 * P};

    const Radial rt = load_radial(A, oc);
    const WenoK K = weno_consts(A.eps);

    const int n = k1 - k0;
    const int first = dir > 0 ? k0 : k1 - 1;
    // Phi on the rows behind (k - dir, and k - 2 dir for kTh4), pole ghosts mirrored
    auto behind = [&](int kb, double& vR, double& vI) {
        const bool ghost = kb < 0 || kb >= nth;
        const int km = kb < 0 ? -1 - kb : (kb >= nth ? 2 * nth - 1 - kb : kb);
        vR = ldb_c<kCoh>(ukp[0] + (size_t)km * nr, oc);
        vI = ldb_c<kCoh>(ukp[1] + (size_t)km * nr, oc);
        if (ghost) {
            vR *= A.parity;
            vI *= A.parity;
        }
    };
    double bhR, bhI, bh2R = 0.0, bh2I = 0.0;
    behind(first - dir, bhR, bhI);
    if constexpr (kTh4) behind(first - 2 * dir, bh2R, bh2I);
    // rows staged: the segment's n rows and the rows past it that lie in the grid
    const int ahead_last = first + dir * n;
    int nst = (ahead_last >= 0 && ahead_last < nth) ? n + 1 : n;
    if constexpr (kTh4) {
        const int ahead2 = ahead_last + dir;
        if (nst > n && ahead2 >= 0 && ahead2 < nth) ++nst;
    }

    // 12 DMA operations: march row i into its slot, or, where the march has no
    // row i, the first dword of each plane (one cache line, read by every lane)
    // into the free slot
    auto issue_row = [&](int i) {
        const bool real = i < nst;
        const size_t row = real ? (size_t)(first + dir * i) * nr : 0;
        const unsigned slot = lds0 + (unsigned)(i & (kRing - 1)) * kSlotBytes;
        const unsigned o0 = real ? od[0] : 0u, o1 = real ? od[1] : 0u, o2 = real ? od[2] : 0u;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double* base = ukp[p] + row;
            dma_dword_c<kCoh>(o0, base, slot + p * kPlaneBytes);
            dma_dword_c<kCoh>(o1, base, slot + p * kPlaneBytes + 256u);
            if (l < 10) dma_dword_c<kCoh>(o2, base, slot + p * kPlaneBytes + 512u);
        }
    };
    issue_row(0);
    issue_row(1);
    issue_row(2);

    const double (*sr)[4][kRowP] = reinterpret_cast<const double (*)[4][kRowP]>(ring);
    for (int i = 0; i < n; ++i) {
        // Waves of one SIMD issue oldest first.  When every workgroup of the
        // launch is resident from the start (kLevel: the single-solve launch),
        // the oldest wave of a SIMD would end its segment long before the
        // youngest (measured: 15 us against 30 us), leaving the SIMD with one
        // or two waves for the last third of the launch.  Lowering a wave's
        // priority as it advances lets the younger waves keep up, and the
        // segments end closer together.  A launch whose tiles are dispatched
        // as slots free up (the batched launch) measured slower with it.
        if constexpr (kLevel) {
            if (i == 0) __builtin_amdgcn_s_setprio(3);
            else if (i == 2) __builtin_amdgcn_s_setprio(2);
            else if (i == 4) __builtin_amdgcn_s_setprio(1);
            else if (i == 6) __builtin_amdgcn_s_setprio(0);
        }
        const int k = first + dir * i;
        const size_t row = (size_t)k * nr;
        const Polar pol = load_polar(A, k);
        double n0 = 0.0, n1 = 0.0, n2 = 0.0, n3 = 0.0;
        if (reads_un<kMode>()) {
            n0 = ld_async_c<kCoh>(oc, unp[0] + row);
            n1 = ld_async_c<kCoh>(oc, unp[1] + row);
            n2 = ld_async_c<kCoh>(oc, unp[2] + row);
            n3 = ld_async_c<kCoh>(oc, unp[3] + row);
        }
        // 1/Sigma of the point.  In the single-solve launch its dependent chain
        // (reciprocal square root and two Newton steps) is started here, where
        // it overlaps the row's loads (the empty asm keeps the compiler from
        // sinking it to its use); the batched launch, whose tiles start as
        // slots free up, measured 0.7 % slower on C4 with that, and leaves the
        // placement to the compiler.
        const double vsig = point_vsig(rt, pol.sn2);
        if constexpr (kLevel) asm volatile("" : : "v"(vsig));
        issue_row(i + 3);
        constexpr int it = reads_un<kMode>() ? 16 : 12;
        if constexpr (kTh4) vm_wait<it>();
        else if (i == 0) vm_wait<12 + it>();
        else vm_wait<2 * it>();
        const int b = i & (kRing - 1), bn = (i + 1) & (kRing - 1);

        const Flux fR = Weno<WP>::flux(sr[b][0][l], sr[b][0][l + 1], sr[b][0][l + 2], sr[b][0][l + 3], sr[b][0][l + 4], K);
        const Flux fI = Weno<WP>::flux(sr[b][1][l], sr[b][1][l + 1], sr[b][1][l + 2], sr[b][1][l + 3], sr[b][1][l + 4], K);
        const Flux gR = Weno<WP>::flux(sr[b][2][l + 5], sr[b][2][l + 4], sr[b][2][l + 3], sr[b][2][l + 2], sr[b][2][l + 1], K);
        const Flux gI = Weno<WP>::flux(sr[b][3][l + 5], sr[b][3][l + 4], sr[b][3][l + 3], sr[b][3][l + 2], sr[b][3][l + 1], K);
        const double phR = sr[b][0][l + 3], phI = sr[b][1][l + 3];
        const double piR = sr[b][2][l + 3], piI = sr[b][3][l + 3];
        double ahR, ahI;   // Phi on the row ahead (k + dir)
        if (i + 1 < nst) {
            ahR = sr[bn][0][l + 3];
            ahI = sr[bn][1][l + 3];
        } else {
            ahR = A.parity * phR;
            ahI = A.parity * phI;
        }
        double ah2R = 0.0, ah2I = 0.0;   // Phi on row k + 2 dir (kTh4)
        if constexpr (kTh4) {
            if (i + 2 < nst) {
                const int bn2 = (i + 2) & (kRing - 1);
                ah2R = sr[bn2][0][l + 3];
                ah2I = sr[bn2][1][l + 3];
            } else if (i + 1 < nst) {
                ah2R = A.parity * ahR;
                ah2I = A.parity * ahI;
            } else {
                ah2R = A.parity * bhR;
                ah2I = A.parity * bhI;
            }
        }
        // the interface flux of the next lane: by DPP in the single-solve
        // launch; the batched launch measured 1.2 % slower on C4 with the DPP
        // moves (VALU work) than with ds_bpermute (LDS work)
        const double fR1 = kLevel ? next_lane(fR.y) : __shfl_down(fR.y, 1);
        const double fI1 = kLevel ? next_lane(fI.y) : __shfl_down(fI.y, 1);
        const double gR1 = kLevel ? next_lane(gR.y) : __shfl_down(gR.y, 1);
        const double gI1 = kLevel ? next_lane(gI.y) : __shfl_down(gI.y, 1);

        if (reads_un<kMode>()) vm_wait<12>(n0, n1, n2, n3);
        if (active) {
            const PointCoef c = point_coef_t(rt, pol, vsig);
            const double upR = dir > 0 ? ahR : bhR, upI = dir > 0 ? ahI : bhI;
            const double dnR = dir > 0 ? bhR : ahR, dnI = dir > 0 ? bhI : ahI;
            Theta xR, xI;
            if constexpr (kTh4) {
                xR = theta4(phR, upR, dnR, dir > 0 ? ah2R : bh2R, dir > 0 ? bh2R : ah2R);
                xI = theta4(phI, upI, dnI, dir > 0 ? ah2I : bh2I, dir > 0 ? bh2I : ah2I);
            } else {
                xR = theta2(phR, upR, dnR);
                xI = theta2(phI, upI, dnI);
            }
            const Four F = rhs_t<bt_first<WP>()>(A, A.ih1, c, plus_diff<WP>(K, fR, fR1), plus_diff<WP>(K, fI, fI1), minus_diff<WP>(K, gR, gR1),
                                 minus_diff<WP>(K, gI, gI1), phR, phI, piR, piI, xR, xI);
            write_point<kMode, kCoh>(A, row, oc, F, phR, phI, piR, piI, n0, n1, n2, n3);
        }
        if constexpr (kTh4) {
            bh2R = bhR;
            bh2I = bhI;
        }
        bhR = phR;
        bhI = phI;
    }
    vm_wait<0>();   // nothing of this strip may still be landing in the ring
}

// Launch layout: every radial strip is cut into the same number `segs` of theta
// segments (an even number when there is more than one), workgroup
// rank = strip * segs + i owns segment i of its strip, and even segments march
// upward, odd ones downward.  Two segments that share a boundary row then read
// it at the same moment (both start there, or both end there), and segment i
// of neighbouring strips -- which share the radial halo -- march the same rows
// in step, so the shared lines are read from HBM once and hit in L2 for the
// second reader.
// LDS of one stage workgroup: the four-row DMA ring (chart T) or the two-row
// staging ring (chart H).
constexpr unsigned kLdsBytes = kRing * kSlotBytes;   // 9216 >= 2 * 4 * kRow * 8

template <int WP, int kMode, int kChart, bool kLevel = false, bool kCoh = false>
__device__ __forceinline__ void march(const StageArgs& A, char* lds, int strip, int k0, int k1, int dir)
{
    if constexpr (kChart == kChartT || kChart == kChartT4)
        march_strip_t<WP, kMode, kLevel, kCoh, kChart == kChartT4>(A, lds, strip, k0, k1, dir);
    else
        march_strip_h<WP, kMode>(A, reinterpret_cast<double (*)[4][kRow]>(lds), strip, k0, k1, dir);
}

template <int WP, int kMode, int kChart>
__device__ __forceinline__ void run_tile(const StageArgs& A, char* lds, int rank)
{
    const int strip = rank / A.segs;
    const int seg = rank - strip * A.segs;
    const int k0 = (int)((long long)A.nth * seg / A.segs);
    const int k1 = (int)((long long)A.nth * (seg + 1) / A.segs);
    if (k1 > k0) march<WP, kMode, kChart, true>(A, lds, strip, k0, k1, ((seg ^ A.flip) & 1) ? -1 : 1);
}

template <int WP, int kMode, int kChart>
__global__ __launch_bounds__(kWave) void stage_kernel(StageArgs A)
{
    __shared__ __attribute__((aligned(16))) char lds[kLdsBytes];
    run_tile<WP, kMode, kChart>(A, lds, xcd_rank((int)blockIdx.x, (int)gridDim.x));
}

// One stage of several independent solves in one launch.  Member m is cut
// into tiles of one radial strip by one theta segment (args[m].segs segments
// per strip) and owns the tile numbers [start[m], start[m+1]), numbered
// segment by segment with the strip index fastest; args[m] holds its buffers,
// tables, grid and dt.  Workgroup `rank` takes the tiles rank, rank + G,
// rank + 2G, ...: at any moment the workgroups in flight hold consecutive
// tiles, i.e. neighbouring strips of the same theta segment, which march the
// same rows together -- their reads of a row are one contiguous stretch of
// each plane, and the radial halo they share is read once into L2.  Even
// segments march upward and odd ones downward, so the two tiles that share a
// boundary row meet there at the end of their march.  By default G equals the
// tile count (one tile per workgroup, dispatched in tile order by the
// hardware as slots free up), which measured faster than fewer workgroups
// looping over tiles.  A tile runs exactly the single-solve code.
template <int WP, int kMode, int kChart>
__global__ __launch_bounds__(kWave, WP == TEUK_W_BF16 ? 3 : 4) void group_stage_kernel(const StageArgs* __restrict__ args,
                                                            const long long* __restrict__ start, int nmem,
                                                            long long tiles)
{
    __shared__ __attribute__((aligned(16))) char lds[kLdsBytes];
    const int G = (int)gridDim.x;
    for (long long t = xcd_rank((int)blockIdx.x, G); t < tiles; t += G) {
        int lo = 0, hi = nmem - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (start[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        const StageArgs A = args[lo];
        const int local = (int)(t - start[lo]);
        const int seg = local / A.nstrips;
        const int strip = local - seg * A.nstrips;
        const int k0 = (int)((long long)A.nth * seg / A.segs);
        const int k1 = (int)((long long)A.nth * (seg + 1) / A.segs);
        if (k1 > k0) march<WP, kMode, kChart>(A, lds, strip, k0, k1, ((seg ^ A.flip) & 1) ? -1 : 1);
    }
}

// ---------------------------------------------------------------- pipelined steps
// Several SSP-RK(3,3) steps in one cooperative launch (tortoise chart).  The
// work items are the tiles of every stage of every step -- tile (strip,
// segment) of stage S, the tiles of the single-solve stage launch -- numbered
// stage by stage, and workgroup w takes items w, w + G, w + 2G, ... in order.
// A tile's stage S reads the stage S-1 results of its own tile and of the
// tiles around it (the radial halo from the neighbouring strips, the theta row
// across a segment boundary, and the corners of both), so it waits for those
// nine tiles only, not for the whole grid: waves drift apart, and the memory
// traffic of some overlaps the arithmetic of others across stage boundaries,
// where stage-by-stage launches drain and refill the GPU three times a step.
// Every other hazard (a stage overwriting values that a neighbour's earlier
// stage still reads: u(1) by the next step's stage 1, u^n by stage 3 in place)
// is ordered through these waits by induction, because a neighbour's stage
// S-1 itself waited for the stage S-2 of its own neighbours.
// Progress: the earliest unfinished item waits only on earlier items, which
// have finished, and its workgroup has finished its own earlier items, so it is
// working on that item; this needs every workgroup resident at once, which the
// cooperative launch guarantees.
// Counters: done[tile] = stages the tile has completed since the state was set
// (absolute, so launches need no reset).  The tiles' rows are read and written
// with agent-coherent accesses (the sc1 forms of the row loads, LDS-DMA loads
// and stores), so no cache needs writing back or invalidating: a workgroup
// waits for its stores to complete and then writes its tile's count; a reader
// polls the neighbours' counts with agent-scope loads and issues its coherent
// loads only after seeing them.
// A wait longer than spin_ticks of the 100 MHz real-time counter sets *err and
// goes on, so a fault of this scheme shows up as an error, never as a hang.
struct PipeArgs {
    StageArgs st[3];       // stage 1, 2, 3 arguments (segs, nstrips equal in all three)
    long long* done;       // [nstrips * segs] stages completed per tile
    int* err;              // set to 1 by a wait that timed out
    long long s0;          // stages completed before this launch (3 x steps)
    int nsteps;            // steps in this launch
    int tiles;             // nstrips * segs
    long long spin_ticks;  // wait limit
};

__device__ __forceinline__ void pipe_wait(const PipeArgs& P, int strip, int seg, long long need)
{
    const int l = threadIdx.x;
    const int nstrips = P.st[0].nstrips, segs = P.st[0].segs;
    const long long* c = nullptr;
    if (l < 9) {
        const int s2 = strip + l / 3 - 1, g2 = seg + l % 3 - 1;
        if (s2 >= 0 && s2 < nstrips && g2 >= 0 && g2 < segs) c = P.done + (size_t)s2 * segs + g2;
    }
    const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
    for (;;) {
        const bool ok = !c || __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= need;
        if (__all(ok)) break;
        // after one timed-out wait anywhere, no wait blocks any more
        const int failed = __hip_atomic_load(P.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (failed) break;
        if ((long long)(__builtin_amdgcn_s_memrealtime() - t0) > P.spin_ticks) {
            if (l == 0) __hip_atomic_store(P.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    // the tile's loads are issued after the counts were seen (the loop exit
    // depends on them) and are coherent loads, so they see the neighbours'
    // completed stores; this keeps the compiler from hoisting them
    asm volatile("" ::: "memory");
}

template <int WP>
__global__ __launch_bounds__(kWave, 4) void pipe_kernel(PipeArgs P)
{
    __shared__ __attribute__((aligned(16))) char lds[kLdsBytes];
    const long long items = 3LL * P.nsteps * P.tiles;
    const int segs = P.st[0].segs;
    for (long long it = blockIdx.x; it < items; it += gridDim.x) {
        const long long S = it / P.tiles;
        const int r = (int)(it - S * P.tiles);
        const int strip = r / segs, seg = r - strip * segs;
        const long long need = P.s0 + S;
        if (need > 0) pipe_wait(P, strip, seg, need);
        const int stage = (int)(S % 3);
        StageArgs A = P.st[stage];
        A.flip = (int)(need & 1);
        const int k0 = (int)((long long)A.nth * seg / segs);
        const int k1 = (int)((long long)A.nth * (seg + 1) / segs);
        const int dir = ((seg ^ A.flip) & 1) ? -1 : 1;
        if (k1 > k0) {
            if (stage == 0) march<WP, kStageFirst, kChartT, false, true>(A, lds, strip, k0, k1, dir);
            else march<WP, kStageLater, kChartT, false, true>(A, lds, strip, k0, k1, dir);
        }
        // publish: every coherent store of the tile has completed before the count is written
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (threadIdx.x == 0)
            __hip_atomic_store(P.done + r, need + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---------------------------------------------------------------- stability bound
// max over points of max(|lam1|, |lam2|)/dx + sqrt(4 A~thth/dtheta^2 + |B~th|/dtheta + |C~|);
// the values are >= 0, so their bit patterns order like unsigned integers and
// the reduction ends in one 64-bit atomic max per workgroup.  Chart T takes the
// coefficients from the radial / polar tables (|lam1| = |lam2| = b), chart H
// from the per-point table (ctab != nullptr).
__global__ __launch_bounds__(256) void dt_bound_kernel(const double* __restrict__ rtab,
                                                       const double* __restrict__ ttab,
                                                       const double* __restrict__ ctab, int nr, int nth,
                                                       double idx, double idth, double c2, double c1,
                                                       unsigned long long* cell)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long n = (long long)nr * nth;
    double val = 0.0;
    if (i < n) {
        double lam, ath, bth, cr, ci;
        if (ctab) {
            lam = fmax(fabs(ctab[kHLam1 * n + i]), fabs(ctab[kHLam2 * n + i]));
            ath = ctab[kHAth * n + i];
            bth = ctab[kHBth * n + i];
            cr = ctab[kHCr * n + i];
            ci = ctab[kHCi * n + i];
        } else {
            const int k = (int)(i / nr), j = (int)(i - (long long)k * nr);
            double rt[kNRT];
            for (int t = 0; t < kNRT; ++t) rt[t] = rtab[(size_t)t * nr + j];
            const double sn2 = ttab[kSn2 * nth + k];
            const PointCoef c = point_coef(rt, sn2, ttab[kCs * nth + k], ttab[kCot * nth + k], ttab[kTh * nth + k],
                                           rsq64(sigma2(rt, sn2)));
            lam = c.b;
            ath = c.ath;
            bth = c.bth;
            cr = c.cr;
            ci = c.ci;
        }
        val = lam * idx + sqrt(c2 * ath * idth * idth + c1 * fabs(bth) * idth + hypot(cr, ci));
    }
    for (int off = 32; off > 0; off >>= 1) val = fmax(val, __shfl_xor(val, off));
    __shared__ double sm[4];
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = val;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double mx = fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3]));
        atomicMax(cell, (unsigned long long)__double_as_longlong(mx));
    }
}

// ---------------------------------------------------------------- non-finite guard
__global__ __launch_bounds__(256) void guard_kernel(const double* __restrict__ u, long long n, int* flag)
{
    bool bad = false;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        bad |= !isfinite(u[i]);
    if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

// ---------------------------------------------------------------- horizon weights
// Weights of the four nodes j0 .. j0 + 3 for the value (w) and the
// rho-derivative (dw, already divided by dx) on the horizon.
struct HorizonWeights {
    double w[4], dw[4];
};

// ---------------------------------------------------------------- ring sample
// One waveform sample (and, in the hyperboloidal chart, one horizon sample)
// into ring slot counter % ring, then counter + 1.  The count lives in device
// memory, so the same launch recorded once into a graph writes each replay's
// samples to the slots that stepping launch by launch would.  One workgroup
// walks the theta rows.
__global__ __launch_bounds__(256) void sample_kernel(const double* __restrict__ u, long long plane, int nr, int nth,
                                                     int j_e, double* __restrict__ wave, double* __restrict__ hwave,
                                                     int j0, HorizonWeights W, long long ring,
                                                     unsigned long long* counter)
{
    __shared__ unsigned long long c;
    if (threadIdx.x == 0) c = *counter;
    __syncthreads();
    const long long slot = (long long)(c % (unsigned long long)ring);
    double* w = wave + (size_t)slot * nth * 2;
    double* hw = hwave ? hwave + (size_t)slot * nth * 4 : nullptr;
    for (int k = threadIdx.x; k < nth; k += blockDim.x) {
        const double* pr = u + (size_t)k * nr;
        const double* pi = pr + plane;
        w[2 * k] = pr[j_e];
        w[2 * k + 1] = pi[j_e];
        if (hw) {
            double vr = 0.0, vi = 0.0, dr = 0.0, di = 0.0;
            for (int q = 0; q < 4; ++q) {
                vr += W.w[q] * pr[j0 + q];
                vi += W.w[q] * pi[j0 + q];
                dr += W.dw[q] * pr[j0 + q];
                di += W.dw[q] * pi[j0 + q];
            }
            hw[4 * k] = vr;
            hw[4 * k + 1] = vi;
            hw[4 * k + 2] = dr;
            hw[4 * k + 3] = di;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) *counter = c + 1;
}

// ---------------------------------------------------------------- coefficient dump
// TEUK_X_COEFFS order: lam1, Re m3, Im m3, Re B~t, Im B~t, Re C~, Im C~, A~thth, B~th, lam2.
__global__ __launch_bounds__(256) void coef_dump_kernel(const double* __restrict__ rtab,
                                                        const double* __restrict__ ttab,
                                                        const double* __restrict__ ctab, int nr, int nth,
                                                        double* __restrict__ out)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long n = (long long)nr * nth;
    if (i >= n) return;
    if (ctab) {
        const int order[TEUK_NCOEF] = {kHLam1, kHM3r, kHM3i, kHBtr, kHBti, kHCr, kHCi, kHAth, kHBth, kHLam2};
        for (int q = 0; q < TEUK_NCOEF; ++q) out[q * n + i] = ctab[order[q] * n + i];
        return;
    }
    const int k = (int)(i / nr), j = (int)(i - (long long)k * nr);
    double rt[kNRT];
    for (int t = 0; t < kNRT; ++t) rt[t] = rtab[(size_t)t * nr + j];
    const double sn2 = ttab[kSn2 * nth + k];
    const PointCoef c = point_coef(rt, sn2, ttab[kCs * nth + k], ttab[kCot * nth + k], ttab[kTh * nth + k],
                                   rsq64(sigma2(rt, sn2)));
    out[0 * n + i] = c.b;
    out[1 * n + i] = c.m3r;
    out[2 * n + i] = c.m3i;
    out[3 * n + i] = c.btr;
    out[4 * n + i] = c.bti;
    out[5 * n + i] = c.cr;
    out[6 * n + i] = c.ci;
    out[7 * n + i] = c.ath;
    out[8 * n + i] = c.bth;
    out[9 * n + i] = -c.b;
}

}  // namespace

static int stage_grid_query(int dev, int weight_prec, bool first, int chart)
{
    // resident workgroups of one stage-kernel instantiation
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    hipError_t e = hipErrorInvalidValue;
#define TEUK_OCC(W, C)                                                                                            \
    if (weight_prec == W && chart == C)                                                                          \
        e = first ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, stage_kernel<W, kStageFirst, C>, kWave, 0) \
                  : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, stage_kernel<W, kStageLater, C>, kWave, 0);
    TEUK_OCC(TEUK_W_FP64, kChartT)
    TEUK_OCC(TEUK_W_FP32, kChartT)
    TEUK_OCC(TEUK_W_FP16, kChartT)
    TEUK_OCC(TEUK_W_BF16, kChartT)
    TEUK_OCC(TEUK_W_FP64, kChartH)
    TEUK_OCC(TEUK_W_FP32, kChartH)
    TEUK_OCC(TEUK_W_FP16, kChartH)
    TEUK_OCC(TEUK_W_BF16, kChartH)
    TEUK_OCC(TEUK_W_FP64, kChartT4)
    TEUK_OCC(TEUK_W_FP32, kChartT4)
    TEUK_OCC(TEUK_W_FP16, kChartT4)
    TEUK_OCC(TEUK_W_BF16, kChartT4)
#undef TEUK_OCC
    if (e != hipSuccess || per_cu < 1) return 0;
    // Whole waves per SIMD: a 17th workgroup (what the LDS of a compute unit
    // holds where the registers allow it) gives one SIMD a fifth wave that the
    // launch then waits for: FP32 weights on 4099 x 131, 49 us a step with 17
    // per unit and 42 with 16.
    if (per_cu > 4) per_cu &= ~3;
    return cus * per_cu;
}

int stage_grid(int weight_prec, bool first, int chart)
{
    static ResidentCache cache[4][2][3];
    int dev = 0;
    if (weight_prec < 0 || weight_prec > 3 || chart < 0 || chart > 2 || hipGetDevice(&dev) != hipSuccess) return 0;
    return cache[weight_prec][first ? 1 : 0][chart].get(dev, [&] { return stage_grid_query(dev, weight_prec, first, chart); });
}

int pipe_grid(int weight_prec)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    hipError_t e = hipErrorInvalidValue;
    if (weight_prec == TEUK_W_FP64) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pipe_kernel<TEUK_W_FP64>, kWave, 0);
    if (weight_prec == TEUK_W_FP32) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pipe_kernel<TEUK_W_FP32>, kWave, 0);
    if (weight_prec == TEUK_W_FP16) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pipe_kernel<TEUK_W_FP16>, kWave, 0);
    if (weight_prec == TEUK_W_BF16) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pipe_kernel<TEUK_W_BF16>, kWave, 0);
    if (e != hipSuccess || per_cu < 1) return 0;
    return cus * per_cu;
}

int launch_pipe(const StageArgs st[3], long long* done, int* err, long long s0, int nsteps, int grid,
                long long spin_ticks, int weight_prec, void* stream)
{
    PipeArgs P;
    for (int i = 0; i < 3; ++i) P.st[i] = st[i];
    P.done = done;
    P.err = err;
    P.s0 = s0;
    P.nsteps = nsteps;
    P.tiles = st[0].nstrips * st[0].segs;
    P.spin_ticks = spin_ticks;
    if (grid < 1 || grid > P.tiles || nsteps < 1) return (int)hipErrorInvalidValue;
    void* args[] = {&P};
    const void* fn = nullptr;
    if (weight_prec == TEUK_W_FP64) fn = (const void*)pipe_kernel<TEUK_W_FP64>;
    if (weight_prec == TEUK_W_FP32) fn = (const void*)pipe_kernel<TEUK_W_FP32>;
    if (weight_prec == TEUK_W_FP16) fn = (const void*)pipe_kernel<TEUK_W_FP16>;
    if (weight_prec == TEUK_W_BF16) fn = (const void*)pipe_kernel<TEUK_W_BF16>;
    if (!fn) return (int)hipErrorInvalidValue;
    (void)hipGetLastError();
    const hipError_t e = hipLaunchCooperativeKernel(fn, dim3((unsigned)grid), dim3(kWave), args, 0, (hipStream_t)stream);
    if (e != hipSuccess) return (int)e;
    return (int)hipGetLastError();
}

int launch_stage(const StageArgs& a, int stage, int weight_prec, int chart, void* stream)
{
    const dim3 grid((unsigned)a.grid), block(kWave);
    hipStream_t st = (hipStream_t)stream;
    (void)hipGetLastError();   // report only what this launch does
    bool done = false;
#define TEUK_LAUNCH(W, C)                                                                      \
    if (weight_prec == W && chart == C) {                                                     \
        if (stage == 1)                                                                       \
            hipLaunchKernelGGL((stage_kernel<W, kStageFirst, C>), grid, block, 0, st, a);     \
        else if (stage == 0)                                                                  \
            hipLaunchKernelGGL((stage_kernel<W, kRhsOnly, C>), grid, block, 0, st, a);        \
        else if (stage == 4)                                                                  \
            hipLaunchKernelGGL((stage_kernel<W, kStageDual, C>), grid, block, 0, st, a);      \
        else                                                                                  \
            hipLaunchKernelGGL((stage_kernel<W, kStageLater, C>), grid, block, 0, st, a);     \
        done = true;                                                                          \
    }
    TEUK_LAUNCH(TEUK_W_FP64, kChartT)
    TEUK_LAUNCH(TEUK_W_FP32, kChartT)
    TEUK_LAUNCH(TEUK_W_FP16, kChartT)
    TEUK_LAUNCH(TEUK_W_BF16, kChartT)
    TEUK_LAUNCH(TEUK_W_FP64, kChartH)
    TEUK_LAUNCH(TEUK_W_FP32, kChartH)
    TEUK_LAUNCH(TEUK_W_FP16, kChartH)
    TEUK_LAUNCH(TEUK_W_BF16, kChartH)
    TEUK_LAUNCH(TEUK_W_FP64, kChartT4)
    TEUK_LAUNCH(TEUK_W_FP32, kChartT4)
    TEUK_LAUNCH(TEUK_W_FP16, kChartT4)
    TEUK_LAUNCH(TEUK_W_BF16, kChartT4)
#undef TEUK_LAUNCH
    if (!done) return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

int launch_group_stage(const StageArgs* args, const long long* start, int nmem, long long tiles, int grid,
                       int stage, int weight_prec, int chart, void* stream)
{
    if (nmem < 1 || tiles < 1 || grid < 1 || stage < 1 || stage > 3) return (int)hipErrorInvalidValue;
    const dim3 g((unsigned)grid), block(kWave);
    hipStream_t st = (hipStream_t)stream;
    (void)hipGetLastError();
    bool done = false;
#define TEUK_GLAUNCH(W, C)                                                                                      \
    if (weight_prec == W && chart == C) {                                                                      \
        if (stage == 1)                                                                                        \
            hipLaunchKernelGGL((group_stage_kernel<W, kStageFirst, C>), g, block, 0, st, args, start, nmem, tiles); \
        else                                                                                                   \
            hipLaunchKernelGGL((group_stage_kernel<W, kStageLater, C>), g, block, 0, st, args, start, nmem, tiles); \
        done = true;                                                                                           \
    }
    TEUK_GLAUNCH(TEUK_W_FP64, kChartT)
    TEUK_GLAUNCH(TEUK_W_FP32, kChartT)
    TEUK_GLAUNCH(TEUK_W_FP16, kChartT)
    TEUK_GLAUNCH(TEUK_W_BF16, kChartT)
    TEUK_GLAUNCH(TEUK_W_FP64, kChartH)
    TEUK_GLAUNCH(TEUK_W_FP32, kChartH)
    TEUK_GLAUNCH(TEUK_W_FP16, kChartH)
    TEUK_GLAUNCH(TEUK_W_BF16, kChartH)
    TEUK_GLAUNCH(TEUK_W_FP64, kChartT4)
    TEUK_GLAUNCH(TEUK_W_FP32, kChartT4)
    TEUK_GLAUNCH(TEUK_W_FP16, kChartT4)
    TEUK_GLAUNCH(TEUK_W_BF16, kChartT4)
#undef TEUK_GLAUNCH
    if (!done) return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

int launch_dt_bound(const double* rtab, const double* ttab, const double* ctab, int nr, int nth, double dx,
                    double dth, int theta_order, unsigned long long* cell, void* stream)
{
    // Largest moduli of the Fourier symbols of dth^2 D2 and dth D1.  Second
    // order: |2 cos xi - 2| <= 4 and |sin xi| <= 1.  Fourth order:
    // |(32 cos xi - 2 cos 2xi - 30)/12| <= 16/3 (at xi = pi), and
    // (8 sin xi - sin 2xi)/6 peaks where 8 cos xi = 2 cos 2xi, i.e. at
    // cos xi = 1 - sqrt(3/2), with the value sin xi (4 - cos xi)/3.
    double c2 = 4.0, c1 = 1.0;
    if (theta_order == 4) {
        const double cx = 1.0 - std::sqrt(1.5);
        c2 = 16.0 / 3.0;
        c1 = std::sqrt(1.0 - cx * cx) * (4.0 - cx) / 3.0;
    }
    (void)hipGetLastError();
    const long long n = (long long)nr * nth;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(dt_bound_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, rtab, ttab, ctab, nr, nth,
                       1.0 / dx, 1.0 / dth, c2, c1, cell);
    return (int)hipGetLastError();
}

int launch_guard(const double* u, long long n, int* flag, void* stream)
{
    (void)hipGetLastError();
    long long blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(guard_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, u, n, flag);
    return (int)hipGetLastError();
}

int launch_sample(const double* u, long long plane, int nr, int nth, int j_e, double* wave, double* hwave, int j0,
                  const double* w, const double* dw, long long ring, unsigned long long* counter, void* stream)
{
    if (j_e < 0 || j_e >= nr || ring < 1) return (int)hipErrorInvalidValue;
    HorizonWeights W{};
    if (hwave) {
        if (j0 < 0 || j0 + 3 > nr - 1) return (int)hipErrorInvalidValue;
        for (int q = 0; q < 4; ++q) {
            W.w[q] = w[q];
            W.dw[q] = dw[q];
        }
    }
    (void)hipGetLastError();
    hipLaunchKernelGGL(sample_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, u, plane, nr, nth, j_e, wave,
                       hwave, j0, W, ring, counter);
    return (int)hipGetLastError();
}

int launch_coef_dump(const double* rtab, const double* ttab, const double* ctab, int nr, int nth, double* out,
                     void* stream)
{
    (void)hipGetLastError();
    const long long n = (long long)nr * nth;
    hipLaunchKernelGGL(coef_dump_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       rtab, ttab, ctab, nr, nth, out);
    return (int)hipGetLastError();
}

}  // namespace teuk
