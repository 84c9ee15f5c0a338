// Rounding error of the double-double WENO5 flux of csrc/teuk_dd_math.h, compiled for
// the host, against binary128, and beside it that of the same flux formed from
// AccurateDWPlusDW sums, DWTimesDW3 / DWTimesFP3 products and IEEE reciprocals
// throughout.  Prints one line per kind of data and weights:
//     kind  weights  rms(ours)/rms(accurate)  the same of the difference of two fluxes
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>

#include <quadmath.h>

#define __device__
#define __forceinline__ inline
// the device's estimate of 1/x, 24 bits of it
static inline double __builtin_amdgcn_rcp(double x)
{
    int e;
    const double m = std::frexp(x, &e);
    return std::ldexp((double)(float)(1.0 / m), -e);
}
using std::fma;
#include "teuk_dd_math.h"

typedef __float128 Q;
using namespace teuk;

namespace ref {
dd sum(dd x, dd y)
{
    const dd s = two_sum(x.hi, y.hi), t = two_sum(x.lo, y.lo);
    const dd v = fast_two_sum(s.hi, s.lo + t.hi);
    return fast_two_sum(v.hi, t.lo + v.lo);
}
dd neg(dd x) { return {-x.hi, -x.lo}; }
dd prod(dd x, dd y)
{
    const double p = x.hi * y.hi, l = fma(x.hi, y.hi, -p);
    return fast_two_sum(p, l + fma(x.lo, y.hi, fma(x.hi, y.lo, x.lo * y.lo)));
}
dd prod(dd x, double y)
{
    const double p = x.hi * y, l = fma(x.hi, y, -p);
    return fast_two_sum(p, fma(x.lo, y, l));
}
dd twice(dd x, double p2) { return {x.hi * p2, x.lo * p2}; }
dd inverse(dd y)
{
    const double t = 1.0 / y.hi;
    const dd p = prod(y, t);
    const double e = (1.0 - p.hi) - p.lo;
    return fast_two_sum(t, t * fma(e, e, e));
}
}  // namespace ref

static dd put(Q v)
{
    const double h = (double)v;
    return {h, (double)(v - h)};
}
static Q get(dd x) { return (Q)x.hi + (Q)x.lo; }
static DDK K;
static double eps;

// 6 q_k - 6 f_2 of the three stencils, from the first differences
template <class T, class Sum, class Neg, class Times>
static void candidates(const T* g, T* q, Sum sum, Neg neg, Times times)
{
    q[0] = sum(times(g[1], 5.0), neg(times(g[0], 2.0)));
    q[1] = sum(g[1], times(g[2], 2.0));
    q[2] = sum(times(g[2], 4.0), neg(g[3]));
}

static dd accurate(const dd* f, int wm, double w0, double w1)
{
    using namespace ref;
    dd g[4], q[3];
    for (int i = 0; i < 4; ++i) g[i] = sum(f[i + 1], neg(f[i]));
    candidates(g, q, sum, neg, [](dd x, double y) { return prod(x, y); });
    dd s;
    if (wm == 1) {
        s = sum(q[2], sum(prod(sum(q[0], neg(q[2])), w0), prod(sum(q[1], neg(q[2])), w1)));
    } else {
        const dd d[3] = {sum(g[1], neg(g[0])), sum(g[2], neg(g[1])), sum(g[3], neg(g[2]))};
        const dd e[3] = {sum(prod(g[1], 3.0), neg(g[0])), sum(g[1], g[2]), sum(g[3], neg(prod(g[2], 3.0)))};
        dd a[3];
        for (int k = 0; k < 3; ++k) {
            const dd is = twice(sum(prod(K.c13_3, prod(d[k], d[k])), prod(e[k], e[k])), 0.25);
            const dd b = two_sum(is.hi, eps);
            const dd r = inverse(fast_two_sum(b.hi, is.lo + b.lo));
            a[k] = prod(K.d[k], prod(r, r));
        }
        const dd inv = inverse(sum(sum(a[0], a[1]), a[2]));
        s = sum(sum(prod(prod(a[0], inv), q[0]), prod(prod(a[1], inv), q[1])), prod(prod(a[2], inv), q[2]));
    }
    return sum(f[2], prod(s, K.sixth));
}

static Q exact(const dd* f, int wm, double w0, double w1)
{
    Q v[5], g[4], q[3], a[3];
    for (int i = 0; i < 5; ++i) v[i] = get(f[i]);
    for (int i = 0; i < 4; ++i) g[i] = v[i + 1] - v[i];
    candidates(g, q, [](Q x, Q y) { return x + y; }, [](Q x) { return -x; }, [](Q x, double y) { return x * (Q)y; });
    if (wm == 1) {
        a[0] = w0;
        a[1] = w1;
        a[2] = (Q)1 - a[0] - a[1];
    } else {
        const Q d[3] = {g[1] - g[0], g[2] - g[1], g[3] - g[2]}, e[3] = {3 * g[1] - g[0], g[1] + g[2], g[3] - 3 * g[2]};
        const int c[3] = {1, 6, 3};
        Q s = 0;
        for (int k = 0; k < 3; ++k) {
            const Q t = (Q)eps + ((Q)13 / 3 * d[k] * d[k] + e[k] * e[k]) / 4;
            s += a[k] = c[k] / (t * t);
        }
        for (int k = 0; k < 3; ++k) a[k] /= s;
    }
    return v[2] + (a[0] * q[0] + a[1] * q[1] + a[2] * q[2]) / 6;
}

int main()
{
    K.sixth = put((Q)1 / 6);
    K.c13_3 = put((Q)13 / 3);
    for (int k = 0; k < 3; ++k) K.d[k] = put((Q)(k == 0 ? 1 : k == 1 ? 6 : 3) / 10);
    struct Kind { const char* name; double width, size, offset, eps; };   // width: packet, else rough data
    const Kind kinds[] = {{"rough", 0, 1, 0, 1e-6},       {"rough-eps-1", 0, 1, 0, 1.0},   {"rough-eps-1e-20", 0, 1, 0, 1e-20},
                          {"rough+1", 0, 1, 1, 1e-6},     {"rough-1e-3", 0, 1e-3, 0, 1e-6}, {"rough-1e-6", 0, 1e-6, 0, 1e-6},
                          {"packet-0.4", 0.4, 1, 0, 1e-6}, {"packet-0.2", 0.2, 1, 0, 1e-6}, {"packet-0.05", 0.05, 1, 0, 1e-6},
                          {"packet-0.01", 0.01, 1, 0, 1e-6}};
    for (const Kind& kd : kinds) {
        eps = kd.eps;
        for (int wm = 0; wm < 2; ++wm) {
            std::mt19937_64 rng(20);
            auto uniform = [&] { return (double)(int64_t)(rng() >> 11) * 0x1p-52 - 1.0; };
            double s[2] = {}, d[2] = {};
            for (int n = 0; n < 100000; ++n) {
                dd f[6];
                double big = 0;
                const Q c = (Q)3 * uniform();
                for (int i = 0; i < 6; ++i) {
                    const Q x = c + (Q)i * kd.width;
                    const Q v = kd.width > 0 ? expq(-x * x) : (Q)uniform() + (Q)uniform() * 0x1p-53;
                    f[i] = put(v * kd.size + kd.offset);
                    big = fmax(big, fabs(f[i].hi));
                }
                Q err[2][2];
                for (int i = 0; i < 2; ++i) {
                    double w0 = 0, w1 = 0;
                    if (wm) {
                        const double g[5] = {f[i].hi, f[i + 1].hi, f[i + 2].hi, f[i + 3].hi, f[i + 4].hi};
                        w64_plus(g, eps, w0, w1);
                    }
                    const dd* v = f + i;
                    const Q x = exact(v, wm, w0, w1);
                    const dd y = wm ? weno<1>(v[0], v[1], v[2], v[3], v[4], K, eps, w0, w1)
                                    : weno<0>(v[0], v[1], v[2], v[3], v[4], K, eps, w0, w1);
                    err[0][i] = (get(y) - x) / big;
                    err[1][i] = (get(accurate(v, wm, w0, w1)) - x) / big;
                }
                for (int m = 0; m < 2; ++m) {
                    const double e0 = (double)(err[m][0] * 0x1p106), e1 = (double)(err[m][1] * 0x1p106);
                    s[m] += e0 * e0 + e1 * e1;
                    d[m] += (e1 - e0) * (e1 - e0);
                }
            }
            std::printf("%s %s %.5f %.5f\n", kd.name, wm ? "fp64" : "dd", std::sqrt(s[0] / s[1]), std::sqrt(d[0] / d[1]));
        }
    }
}
