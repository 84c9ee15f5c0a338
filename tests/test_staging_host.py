"""CPU: the staged copy to the host (csrc/teuk_staging.h, tests/staging_host.cpp): exact around the
chunk sizes, errors, threads that sleep while nothing has arrived, the pool of chunk sets over
several devices, and the CPUs that a quota leaves; the same under ThreadSanitizer."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("checked", [False, True], ids=["plain", "tsan"])
def test_staged_copy(tmp_path, checked):
    exe = str(tmp_path / "staging_host")
    subprocess.run(["g++", "-std=gnu++17", "-O1", "-g", "-Wall", "-pthread", *(["-fsanitize=thread"] if checked else []),
                    "-I", os.path.join(ROOT, "paper_2010_04760_amd", "csrc"), os.path.join(HERE, "staging_host.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe, str(tmp_path)], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1"))
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout[-2000:] + r.stderr[-3000:]
