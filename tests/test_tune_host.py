"""CPU: the tuner's bookkeeping (csrc/teuk_tune.hip with stand-ins for the solver and the GPU,
tests/tune_host.cpp): times paired with the shape that is remembered, the default route timed only
where it is another one, and a failed run that leaves the remembered shape."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2010_04760_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None or shutil.which("g++") is None, reason="needs hipcc and g++")
def test_tuner_bookkeeping(tmp_path):
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    tune, exe = str(tmp_path / "tune.o"), str(tmp_path / "tune_host")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1", "-fPIC", *inc, "-c",
                    os.path.join(CSRC, "teuk_tune.hip"), "-o", tune], check=True)
    subprocess.run(["g++", "-std=gnu++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", *inc,
                    os.path.join(HERE, "tune_host.cpp"), tune, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "failures 0", r.stdout + r.stderr
