"""GPU: SSP-RK(3,3) stepped by the temporally blocked launch (the default where
that kernel is built) against stage launches (a solver with a budget of stage
workgroups): the same bits, at the edges of the 114-point tiles, from two theta
rows up, with more and fewer strip-rows than workgroups, over runs of one, two,
three and more steps, and where the state has to keep its buffer (graph mode, an
odd chunk; the caller's buffer of teuk_step_noalloc).

The tolerance is zero: both write every operation out in the same order."""
import numpy as np
import pytest

import paper_2010_04760_amd as T
import workloads as W

pytestmark = pytest.mark.gpu


def cfg(nr, nth, wp="fp64", **kw):
    return T.make_config(s=-2, m=1, a=0.9, nr=nr, ntheta=nth, x_min=-30.0, x_max=50.0, weight_prec=wp, **kw)


def pair(nr, nth, wp, **kw):
    strips = -(-nr // 63)
    a, b = T.Solver(cfg(nr, nth, wp, **kw)), T.Solver(cfg(nr, nth, wp, workgroups=4 * strips, **kw))
    u0 = W.random_state(nr, nth, seed=nr + nth, smooth=True)
    a.set_initial(u0)
    b.set_initial(u0)
    return a, b, u0


@pytest.mark.parametrize("wp", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nr,nth", [(7, 2), (64, 3), (114, 2), (115, 7), (127, 5), (228, 4), (229, 33), (1000, 190),
                                    (3000, 61)])
def test_equals_stage_launches(nr, nth, wp):
    a, b, _ = pair(nr, nth, wp, x_extract=5.0, extract_every=3, max_samples=8)
    print("case fused", nr, nth, wp, flush=True)
    for n in (1, 2, 3, 7):
        a.step(n)
        b.step(n)
        np.testing.assert_array_equal(a.state(), b.state())
    ta, wa = a.waveform()
    tb, wb = b.waveform()
    np.testing.assert_array_equal(ta, tb)
    np.testing.assert_array_equal(wa, wb)
    np.testing.assert_array_equal(a.rhs(), b.rhs())
    a.close()
    b.close()


@pytest.mark.parametrize("wp", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nr,nth,a,x_min", [(7, 3, 1.0, 20 / 21), (115, 2, 1.0, 20 / 21), (300, 25, 0.8, 1.2),
                                            (901, 64, 0.8, 1.2)])
def test_hyperboloidal_equals_stage_launches(nr, nth, a, x_min, wp):
    """x_min = 1.2 at a = 0.8 reaches inside the horizon: both upwind sides in one wave."""
    print("case fused chart H", nr, nth, a, wp, flush=True)
    kw = dict(s=-2, m=1, a=a, nr=nr, ntheta=nth, x_min=x_min, x_max=19.0, chart="H", weight_prec=wp, x_extract=5.0,
              extract_every=2, max_samples=8)
    u0 = W.random_state(nr, nth, seed=nr, smooth=True)
    with T.Solver(T.make_config(**kw)) as x, T.Solver(T.make_config(workgroups=2 * (-(-nr // 63)), **kw)) as y:
        x.set_initial(u0)
        y.set_initial(u0)
        for n in (1, 2, 5):
            x.step(n)
            y.step(n)
            np.testing.assert_array_equal(x.state(), y.state())
        for p, q in zip(x.horizon(), y.horizon()):
            np.testing.assert_array_equal(p, q)


@pytest.mark.parametrize("wp", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nr,nth", [(51, 2), (52, 5), (102, 256), (103, 257), (700, 230), (653, 24), (3000, 130),
                                    (8192, 40)])
def test_low_tiles_and_marched_tiles(nr, nth, wp):
    """Around the 51 points of the low tiles, from one row a tile to twelve, with a last
    tile of fewer rows; the last two sizes are marched."""
    a, b, _ = pair(nr, nth, wp)
    print("case fused tiles", nr, nth, wp, flush=True)
    for n in (1, 2):
        a.step(n)
        b.step(n)
        np.testing.assert_array_equal(a.state(), b.state())
    a.close()
    b.close()


@pytest.mark.parametrize("wp", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nr,nth", [(7, 2), (52, 3), (103, 4), (51, 5), (700, 24), (653, 67), (1000, 190)])
def test_fourth_order_theta_low_tiles(nr, nth, wp):
    """Poles that reach two rows into a tile, from one row a tile to eight."""
    a, b, _ = pair(nr, nth, wp, theta_order=4)
    print("case fused theta4", nr, nth, wp, flush=True)
    for n in (1, 2, 3):
        a.step(n)
        b.step(n)
        np.testing.assert_array_equal(a.state(), b.state())
    a.close()
    b.close()


@pytest.mark.parametrize("wp", ["fp64", "fp32"])
@pytest.mark.parametrize("nr,nth,chart", [(7, 2, "T"), (114, 2, "T"), (115, 3, "T"), (120, 5, "T"), (121, 7, "T"),
                                          (500, 200, "T"), (3000, 130, "T"), (900, 24, "T"), (7, 3, "H"), (121, 2, "H"), (300, 25, "H")])
def test_ssprk104_equals_stage_launches(nr, nth, chart, wp):
    """Ten stages in four launches (114 outputs a tile in two of them, 120 in the others)."""
    print("case fused rk104", nr, nth, chart, wp, flush=True)
    kw = dict(s=-2, m=1, a=0.9, nr=nr, ntheta=nth, weight_prec=wp, integrator="rk104", extract_every=2, max_samples=8,
              x_extract=5.0)
    kw.update(dict(x_min=-30.0, x_max=50.0) if chart == "T" else dict(chart="H", a=0.8, x_min=1.2, x_max=19.0))
    u0 = W.random_state(nr, nth, seed=nr, smooth=True)
    with T.Solver(T.make_config(**kw)) as x, T.Solver(T.make_config(workgroups=2 * (-(-nr // 63)), **kw)) as y:
        x.set_initial(u0)
        y.set_initial(u0)
        for n in (1, 2, 4):
            x.step(n)
            y.step(n)
            np.testing.assert_array_equal(x.state(), y.state())
        np.testing.assert_array_equal(x.waveform()[1], y.waveform()[1])


@pytest.mark.parametrize("chunk", [1, 3, 5, 4])
def test_odd_graph_chunks(chunk):
    print("case fused graph", chunk, flush=True)
    a, b, _ = pair(300, 12, "fp64", x_extract=5.0, extract_every=1, max_samples=64)
    a.step(1)                        # the state sits in another buffer when graph mode starts
    b.step(1)
    a.set_graph(chunk)
    for n in (chunk, 2 * chunk + 1, 3, 1, 2, chunk, 7):
        a.step(n)
        b.step(n)
        np.testing.assert_array_equal(a.state(), b.state())
    np.testing.assert_array_equal(a.waveform()[1], b.waveform()[1])
    a.close()
    b.close()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7])
def test_noalloc_keeps_the_callers_buffer(n):
    import torch

    print("case fused noalloc", n, flush=True)
    dt = 0.01
    c = cfg(230, 9, dt=dt)
    u0 = W.random_state(230, 9, seed=n, smooth=True)
    u = torch.from_numpy(u0).cuda()
    T.teuk_step_noalloc(c, u, n)
    with T.Solver(cfg(230, 9, dt=dt, workgroups=8)) as sv:
        sv.set_initial(u0)
        sv.step(n)
        np.testing.assert_array_equal(u.cpu().numpy(), sv.state())


@pytest.mark.parametrize("chunk", [0, 1, 3, 4])
def test_group_members_equal_solves_alone(chunk):
    """One blocked launch over members of both charts and precisions, eagerly and from graphs of odd and
    even chunks, with a member stepped on its own in between (its state keeps its buffer) and one leaving."""
    print("case fused group", chunk, flush=True)
    T1 = dict(x_min=-30.0, x_max=50.0, x_extract=5.0, max_samples=64)
    TH = dict(x_min=20 / 21, x_max=19.0, x_extract=5.0, max_samples=64, chart="H")
    specs = [(130, 5, 0, 1, 0.5, "fp64", 1, T1), (700, 33, -2, 2, 0.9, "fp64", 1, T1), (7, 2, 0, 0, 0.3, "fp64", 0, T1),
             (229, 12, -2, 1, 0.8, "fp32", 1, T1), (300, 9, -2, 0, 1.0, "fp64", 1, TH), (115, 4, 0, 1, 1.0, "fp32", 1, TH)]
    alone, members = [], []
    for i, (nr, nth, s_, m, a, wp, every, kw) in enumerate(specs):
        kw = dict(kw, extract_every=every, max_samples=64 if every else 0)
        c = [T.make_config(s=s_, m=m, a=a, nr=nr, ntheta=nth, weight_prec=wp, workgroups=w, **kw) for w in (0, 4000)]
        u0 = W.random_state(nr, nth, seed=i, smooth=True)
        x, y = T.Solver(c[0]), T.Solver(c[1])
        x.set_initial(u0)
        y.set_initial(u0)
        members.append(x)
        alone.append(y)
    g = T.Group(len(specs))
    for x in members:
        g.add(x)
    if chunk:
        g.set_graph(chunk)
    for n, own in ((3, 3), (4, 1), (7, 2), (1, 5)):
        g.step(n)
        members[1].step(own)
        alone[1].step(own)
        for x, y in zip(members, alone):
            y.step(n)
    g.remove(members[0])
    g.step(5)
    members[0].step(5)
    for x, y in zip(members, alone):
        y.step(5)
        np.testing.assert_array_equal(x.state(), y.state())
        if x.cfg.extract_every:
            np.testing.assert_array_equal(x.waveform()[1], y.waveform()[1])
    g.close()
