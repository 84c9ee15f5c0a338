"""CPU: rounding error of the double-double flux arithmetic (csrc/teuk_dd_math.h, compiled
for the host) against binary128, beside the same flux formed from accurate double-word
sums and products throughout: it may not be larger, on rough data and on packets from
2.5 to 100 points a width.

Bar: a ratio of two rms errors over 200000 fluxes each, whose roundings mostly coincide,
scatters by less than 1/sqrt(200000) = 0.22 %; 1 % is four times that."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_flux_error_is_that_of_accurate_sums(tmp_path):
    exe = str(tmp_path / "dd_flux_error")
    subprocess.run(["g++", "-O2", "-std=gnu++17", "-ffp-contract=off", "-fno-fast-math", "-w",
                    "-I", os.path.join(ROOT, "paper_2010_04760_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "dd_flux_error.cpp"), "-o", exe, "-lquadmath"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True, timeout=300).stdout.split("\n")
    rows = [ln.split() for ln in out if ln]
    assert len(rows) == 20
    for kind, weights, flux, diff in rows:
        print(kind, weights, flux, diff, flush=True)
        assert float(flux) <= 1.01 and float(diff) <= 1.01, (kind, weights, flux, diff)
