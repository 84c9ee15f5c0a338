"""CPU: where the lanes of a wave hand each other values through LDS, the order is a fence of
the wavefront on LDS, not only a barrier that the compiler need not take for a memory
operation: the barrier stands in wave_sync() alone, and its gfx950 code (as LLVM IR) has a
release fence before it and an acquire fence after it, between the write and the read."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_04760_amd", "csrc")
PROBE = """
#include <hip/hip_runtime.h>
#include "teuk_device.h"
extern "C" __global__ void probe(const double* v, double* o)
{
    __shared__ double lds[128];
    const int l = (int)threadIdx.x & 63;
    lds[l] = v[l];
    teuk::wave_sync();
    o[l] = lds[l + 1];
}
"""


def test_no_bare_wave_barrier():
    found = []
    for f in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, f)).read()
        found += [f] * len(re.findall(r"__builtin_amdgcn_wave_barrier\s*\(", text))
    assert found == ["teuk_device.h"]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_wave_sync_is_fenced(tmp_path):
    src, ir = tmp_path / "probe.hip", tmp_path / "probe.ll"
    src.write_text(PROBE)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-w", "-I", os.path.join(ROOT, "include"), "-I",
                    CSRC, "-S", "-emit-llvm", "--offload-device-only", str(src), "-o", str(ir)], check=True,
                   capture_output=True)
    body = re.search(r"define [^\n]*@probe\(.*?^}", ir.read_text(), re.S | re.M).group(0)
    order = [r"store double .*addrspace\(3\)", r"fence syncscope\(\"wavefront[^\"]*\"\) release",
             r"call void @llvm\.amdgcn\.wave\.barrier", r"fence syncscope\(\"wavefront[^\"]*\"\) acquire",
             r"load double, ptr addrspace\(3\)"]
    at = [re.search(p, body) for p in order]
    assert all(at), [p for p, m in zip(order, at) if not m]
    assert [m.start() for m in at] == sorted(m.start() for m in at)
