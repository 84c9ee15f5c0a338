"""GPU: steps captured by the caller into a graph of its own, replayed several times with
eager steps and synchronisations between the replays, against a solve without graphs:
every replay has to advance the state that the eager steps left, and the eager steps the
state that the replay left, whatever buffer the launches work in.

The tolerance is zero: replays are the same launches."""
import numpy as np
import pytest

import paper_2010_04760_amd as T
import workloads as W

pytestmark = pytest.mark.gpu


def cfg(nr, nth, **kw):
    kw = dict(dict(x_min=-30.0, x_max=50.0), **kw)
    return T.make_config(s=-2, m=1, a=0.9, nr=nr, ntheta=nth, **kw)


def captured(stream, work):
    import torch

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        work()
    return g


def replay(stream, g):
    import torch

    with torch.cuda.stream(stream):
        g.replay()


@pytest.mark.parametrize("before", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("nr,nth,kw", [(200, 12, {}), (6043, 53, {}), (120, 9, dict(integrator="rk104")),
                                       (230, 9, dict(theta_order=4)),
                                       (300, 12, dict(chart="H", a=0.8, x_min=1.2, x_max=19.0))])
def test_solver(nr, nth, kw, n, before):
    import torch

    print("case callers graph", nr, nth, kw, n, before, flush=True)
    s = torch.cuda.Stream()
    kw = dict(kw)
    a = kw.pop("a", 0.9)
    c = cfg(nr, nth, **kw)
    c.a = a
    u0 = W.random_state(nr, nth, seed=nr, smooth=True)
    with T.Solver(c, stream=s) as x, T.Solver(c) as y:
        x.set_initial(u0)
        y.set_initial(u0)
        x.step(before)
        y.step(before)
        g = captured(s, lambda: x.step(n))
        np.testing.assert_array_equal(x.state(), y.state())      # capturing runs nothing
        for eager in (0, 1, 0, 3, 2):
            replay(s, g)
            y.step(n)
            np.testing.assert_array_equal(x.state(), y.state())
            x.step(eager)
            y.step(eager)
            np.testing.assert_array_equal(x.state(), y.state())
        x.set_initial(u0)
        y.set_initial(u0)
        for _ in range(2):
            replay(s, g)
            y.step(n)
        np.testing.assert_array_equal(x.state(), y.state())


@pytest.mark.parametrize("chunk", [0, 3])
@pytest.mark.parametrize("n", [1, 2, 3])
def test_group(n, chunk):
    """Members of both charts; the group steps by its own graphs or eagerly between the replays,
    a member on its own as well."""
    import torch

    print("case callers graph, group", n, chunk, flush=True)
    s = torch.cuda.Stream()
    H = dict(chart="H", x_min=1.2, x_max=19.0)
    cs = [cfg(130, 5), cfg(700, 33), cfg(229, 12, weight_prec="fp32"), cfg(300, 9, **H), cfg(90, 7, theta_order=4)]
    cs[3].a = 0.8
    members, alone = [], []
    for i, c in enumerate(cs):
        u0 = W.random_state(c.nr, c.ntheta, seed=i, smooth=True)
        x, y = T.Solver(c, stream=s), T.Solver(c)
        x.set_initial(u0)
        y.set_initial(u0)
        members.append(x)
        alone.append(y)

    def same():
        for x, y in zip(members, alone):
            np.testing.assert_array_equal(x.state(), y.state())

    def reference(k):
        for y in alone:
            y.step(k)

    with T.Group(len(cs), stream=s) as grp:
        for x in members:
            grp.add(x)
        grp.step(3)                      # the members' states sit in their other buffers
        reference(3)
        g = captured(s, lambda: grp.step(n))
        same()
        if chunk:
            grp.set_graph(chunk)
        for eager in (0, 1, 4, 3, 7):
            replay(s, g)
            reference(n)
            same()
            grp.step(eager)
            reference(eager)
            members[1].step(1)
            alone[1].step(1)
            same()


def test_a_members_own_graph():
    """A graph of one member alone, replayed while the group steps all of them."""
    import torch

    print("case callers graph, one member", flush=True)
    s = torch.cuda.Stream()
    cs = [cfg(130, 5), cfg(300, 12)]
    members, alone = [], []
    for i, c in enumerate(cs):
        u0 = W.random_state(c.nr, c.ntheta, seed=i, smooth=True)
        x, y = T.Solver(c, stream=s), T.Solver(c)
        x.set_initial(u0)
        y.set_initial(u0)
        members.append(x)
        alone.append(y)
    g = captured(s, lambda: members[0].step(3))
    with T.Group(2, stream=s) as grp:
        for x in members:
            grp.add(x)
        for k in (1, 3, 2, 5):
            grp.step(k)
            replay(s, g)
            for y in alone:
                y.step(k)
            alone[0].step(3)
            for x, y in zip(members, alone):
                np.testing.assert_array_equal(x.state(), y.state())
