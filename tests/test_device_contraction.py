"""CPU: the device arithmetic of csrc/teuk_device.h is written out operation by operation,
so what the compiler may fuse does not change it: its gfx950 code has the same operations
with -ffp-contract=fast and -ffp-contract=off.  (Which products it fuses could otherwise
differ from kernel to kernel, and a point's bits with the launch that computes it.)"""
import collections
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROBE = """
#include <hip/hip_runtime.h>
#include "teuk_device.h"
using namespace teuk;
template <int W> __device__ void flux(const double* v, double eps, double* o)
{
    const auto K = weno_consts_for<W>(eps);
    const Flux f = Weno<W>::flux(v[0], v[1], v[2], v[3], v[4], K);
    o[0] = plus_diff<W>(K, f, v[5]);
    o[1] = minus_diff<W>(K, f, v[6]);
}
extern "C" __global__ void k_fp64(const double* v, double eps, double* o) { flux<TEUK_W_FP64>(v, eps, o); }
extern "C" __global__ void k_fp64_h(const double* v, double eps, double* o) { flux<kWeno64H>(v, eps, o); }
extern "C" __global__ void k_fp32(const double* v, double eps, double* o) { flux<TEUK_W_FP32>(v, eps, o); }
extern "C" __global__ void k_fp16(const double* v, double eps, double* o) { flux<TEUK_W_FP16>(v, eps, o); }
extern "C" __global__ void k_bf16(const double* v, double eps, double* o) { flux<TEUK_W_BF16>(v, eps, o); }
template <bool kBt> __device__ void rhs(StageArgs A, const double* v, double* o)
{
    const Radial r = load_radial(A, 0);
    const Polar p = load_polar(A, 0);
    const PointCoef c = point_coef_t(r, p, point_vsig(r, p.sn2));
    const Theta x = theta2(v[0], v[1], v[2]), y = theta4(v[0], v[1], v[2], v[3], v[4]);
    const Four F = rhs_t<kBt>(A, A.ih1, c, v[5], v[6], v[7], v[8], v[9], v[10], v[11], v[12], x, y);
    for (int i = 0; i < 4; ++i) o[i] = combine(A.ca, v[13 + i], A.cb, euler(v[17 + i], A.dt, F.v[i]));
}
extern "C" __global__ void k_rhs_a(StageArgs A, const double* v, double* o) { rhs<true>(A, v, o); }
extern "C" __global__ void k_rhs_b(StageArgs A, const double* v, double* o) { rhs<false>(A, v, o); }
extern "C" __global__ void k_rhs_h(StageArgs A, const double* v, double* o)
{
    double hc[kNCH];
    for (int i = 0; i < kNCH; ++i) hc[i] = v[20 + i];
    const Four F = rhs_h(hc, A.ih1, A.ih2, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10], v[11]);
    for (int i = 0; i < 4; ++i) o[i] = F.v[i];
}
"""
KERNELS = ["k_fp64", "k_fp64_h", "k_fp32", "k_fp16", "k_bf16", "k_rhs_a", "k_rhs_b", "k_rhs_h"]


def operations(asm):
    out = {}
    for k in KERNELS:
        body = re.search(rf"^{k}:.*?^\.Lfunc_end", asm, re.S | re.M).group(0)
        ops = re.findall(r"^\s*(v_[a-z0-9_]+?)(?:_e32|_e64|_dpp)?\s", body, re.M)
        out[k] = collections.Counter(o for o in ops if re.search(r"_(f16|bf16|f32|f64)(_|$)", o))
    return out


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_contraction_changes_nothing(tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text(PROBE)
    got = {}
    for mode in ("fast", "off"):
        asm = tmp_path / f"{mode}.s"
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-mcode-object-version=5", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", f"-ffp-contract={mode}", "-w", "-I",
                        os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2010_04760_amd", "csrc"), "-S",
                        "--offload-device-only", str(src), "-o", str(asm)], check=True, capture_output=True)
        got[mode] = operations(asm.read_text())
    for k in KERNELS:
        assert sum(got["fast"][k].values()) >= 10, k
        assert got["fast"][k] == got["off"][k], (k, got["fast"][k] - got["off"][k], got["off"][k] - got["fast"][k])
