"""CPU: the benchmark's roofline of an SSP-RK(3,3) step goes by the launch that the solver takes,
and its share of the VALU issue rate stays one: measured steps of the marched launch (points,
seconds) at each weight precision lie below it."""
import os
import sys
import types

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

T = types.SimpleNamespace(TEUK_STEP_STAGES=0, TEUK_STEP_BLOCKED=1, TEUK_STEP_LOW_TILES=2)


def launch(kind):
    return types.SimpleNamespace(kind=kind)


@pytest.mark.parametrize("weights,points,seconds", [("fp64", 8192 * 256, 70.6e-6), ("fp32", 8192 * 256, 72.6e-6),
                                                    ("fp32", 96173184, 3.2195e-3), ("fp16", 8192 * 256, 121.0e-6)])
def test_issue_share_of_measured_steps(weights, points, seconds):
    r = bench.step_roofline(T, launch(1), points, seconds, weights, None)
    assert r["kernel"].startswith("blocked_step_kernel")
    assert 0.5 < r["valu_issue_frac"] < 1.0, r["valu_issue_frac"]


def test_route_names():
    r = bench.step_roofline(T, launch(0), 1000, 1e-5, "bf16", None)
    assert r["kernel"].startswith("stage_kernel") and "valu_issue_frac" not in r
    assert r["algorithmic_bytes_per_launch"] == pytest.approx(256 * 1000 / 3)
    r = bench.step_roofline(T, launch(2), 1000, 1e-5, "fp64", None)
    assert r["kernel"].startswith("thin_step_kernel") and "valu_issue_frac" not in r
    assert r["algorithmic_bytes_per_launch"] == 64 * 1000
