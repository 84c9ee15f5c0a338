"""GPU: each launch that steps can take, at the edges of its own tiles, on sizes for which
teuk_step_launch says that it is taken, against stage launches (a solver with a budget of
stage workgroups): marched tiles of 114 points (120 in the two-stage launches), low tiles
of 9 to 12 rows, and the extreme stage shapes that a default solver no longer steps by.

The tolerance is zero: every launch writes each point's operations out in the same order."""
import numpy as np
import pytest

import paper_2010_04760_amd as T
import workloads as W

pytestmark = pytest.mark.gpu

T_KW = dict(s=-2, m=1, a=0.9, x_min=-30.0, x_max=50.0)
H_KW = dict(s=-2, m=1, a=0.8, x_min=1.2, x_max=19.0, chart="H")     # inside the horizon: both upwind sides


def compare(nr, nth, runs, kind, rows=None, budget=None, **kw):
    """The default route (of this kind) against stage launches over runs of steps."""
    u0 = W.random_state(nr, nth, seed=nr % 1000 + nth, smooth=True)
    budget = budget or 4 * (-(-nr // 63))
    with T.Solver(T.make_config(nr=nr, ntheta=nth, **kw)) as x, \
            T.Solver(T.make_config(nr=nr, ntheta=nth, workgroups=budget, **kw)) as y:
        lx, ly = x.step_launch(), y.step_launch()
        assert lx.kind == kind and ly.kind == T.TEUK_STEP_STAGES, (lx.kind, ly.kind)
        assert rows is None or lx.rows == rows, lx.rows
        x.set_initial(u0)
        y.set_initial(u0)
        for n in runs:
            x.step(n)
            y.step(n)
            np.testing.assert_array_equal(x.state(), y.state())
        return lx, ly


@pytest.mark.parametrize("wp", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nr", [6042, 6043, 6155, 6156])
def test_marched_tiles(nr, wp):
    """53 whole tiles, one point more, and a last tile of one point less than whole."""
    print("case routes marched", nr, wp, flush=True)
    lx, _ = compare(nr, 53, (2, 3), T.TEUK_STEP_BLOCKED, weight_prec=wp, **T_KW)
    assert lx.launches == 1


@pytest.mark.parametrize("wp", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nr", [6042, 6043])
def test_marched_tiles_hyperboloidal(nr, wp):
    print("case routes marched chart H", nr, wp, flush=True)
    compare(nr, 53, (2, 3), T.TEUK_STEP_BLOCKED, weight_prec=wp, **H_KW)


@pytest.mark.parametrize("wp", ["fp64", "fp32"])
@pytest.mark.parametrize("chart", [T_KW, H_KW], ids=["T", "H"])
@pytest.mark.parametrize("nr", [6000, 6001, 6043])
def test_marched_ssprk104(nr, chart, wp):
    """50 whole tiles of the two-stage launches and one point more; 53 of the three-stage ones."""
    print("case routes marched rk104", nr, wp, flush=True)
    lx, ly = compare(nr, 53, (1, 2), T.TEUK_STEP_BLOCKED, weight_prec=wp, integrator="rk104", **chart)
    assert lx.launches == 4 and ly.launches == 10


@pytest.mark.parametrize("wp,kw", [("fp64", T_KW), ("fp32", T_KW), ("fp16", T_KW), ("bf16", T_KW), ("fp64", H_KW)])
@pytest.mark.parametrize("rows,nth", [(9, 88), (10, 98), (11, 109), (12, 118)])
def test_tall_low_tiles(rows, nth, wp, kw):
    """The last tile is not whole.  (51 strips, 10 tiles of each on 256 compute units.)"""
    print("case routes low tiles", rows, nth, wp, flush=True)
    lx, _ = compare(2600, nth, (2, 3), T.TEUK_STEP_LOW_TILES, rows=rows, weight_prec=wp, **kw)
    assert lx.workgroups == 51 * (-(-nth // rows))


@pytest.mark.parametrize("rows,nth", [(9, 88), (12, 118)])
def test_tall_low_tiles_ssprk104(rows, nth):
    print("case routes low tiles rk104", rows, nth, flush=True)
    compare(2600, nth, (1, 2), T.TEUK_STEP_LOW_TILES, rows=rows, integrator="rk104", **T_KW)


@pytest.mark.parametrize("nr,nth,budget,kind", [(70, 2048, 2 * 2048, T.TEUK_STEP_LOW_TILES),
                                                (70, 2048, 2 * 1024, T.TEUK_STEP_LOW_TILES),
                                                (1 << 19, 4, 8323, T.TEUK_STEP_BLOCKED),
                                                (64, 65536, 2 * 1920, T.TEUK_STEP_BLOCKED)])
def test_extreme_stage_shapes(nr, nth, budget, kind):
    """Segments of one and two rows, one segment per strip on more strips than the GPU holds, the
    most theta rows: these steps by stage launches against the default ones, which have a test
    against the oracle on the same grids."""
    print("case routes stage shapes", nr, nth, budget, flush=True)
    _, ly = compare(nr, nth, (3,), kind, budget=budget, **T_KW)
    assert ly.workgroups == budget


def test_reported_launches():
    """What does not step by temporally blocked launches says so, and a group reports the launch it takes."""
    print("case routes reported", flush=True)
    with T.Solver(T.make_config(nr=6043, ntheta=53, theta_order=4, **T_KW)) as sv:
        assert (sv.step_launch().kind, sv.step_launch().launches) == (T.TEUK_STEP_STAGES, 3)
    with T.Solver(T.make_config(nr=8192, ntheta=130, weight_prec="bf16", **T_KW)) as sv:      # above 2^20 points
        assert sv.step_launch().kind == T.TEUK_STEP_STAGES
    with T.Solver(T.make_config(nr=100, ntheta=20, state="dd", weight_prec="dd", **T_KW)) as sv:
        assert (sv.step_launch().kind, sv.step_launch().workgroups) == (T.TEUK_STEP_STAGES, 2 * 20)
    with T.Solver(T.make_config(nr=900, ntheta=20, integrator="rk3_pipelined", **T_KW)) as sv:
        assert sv.step_launch().kind == T.TEUK_STEP_PIPELINED
    with T.Solver(T.make_config(nr=900, ntheta=20, integrator="rk3_blocked", **T_KW)) as sv:
        assert sv.step_launch().kind == T.TEUK_STEP_BLOCKED and sv.step_launch().workgroups == sv.info().workgroups
    members = [T.Solver(T.make_config(nr=nr, ntheta=3, **T_KW)) for nr in (100, 300)]
    with T.Group(2) as g:
        for sv in members:
            sv.set_initial(W.random_state(sv.cfg.nr, 3, seed=1, smooth=True))
            g.add(sv)
        inf = g.info()
        assert inf.workgroups == inf.tiles == 3 * (1 + 3)      # one strip-row each: fewer than the GPU holds


def test_group_tuning_keeps_a_height_that_makes_no_difference():
    """Members stepped by one blocked launch have no tile heights to choose from."""
    print("case routes group tune", flush=True)
    members = [T.Solver(T.make_config(nr=nr, ntheta=24, **T_KW)) for nr in (500, 700)]
    with T.Group(2) as g:
        for sv in members:
            sv.set_initial(W.random_state(sv.cfg.nr, 24, seed=1, smooth=True))
            g.add(sv)
        for _ in range(3):
            info = g.tune(5)
            assert info.rows_per_tile == info.default_rows_per_tile == 8
            assert info.candidates >= 10 and info.us_per_step <= info.us_per_step_default
