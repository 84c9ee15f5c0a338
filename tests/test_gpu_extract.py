"""GPU: results that reach the host through the pinned chunks (8 MiB and more) and
the sample rings: exact copies, at the edges of that rule and of the chunks, from
several threads at once, and where the ring wraps."""
import threading

import numpy as np
import pytest

import paper_2010_04760_amd as T
import workloads as W

pytestmark = pytest.mark.gpu


def cfg(nr, nth, **kw):
    return T.make_config(s=-2, m=1, a=0.9, nr=nr, ntheta=nth, x_min=-30.0, x_max=50.0, **kw)


def numbered(nr, nth, first=0.0):
    return (first + np.arange(4 * nth * nr, dtype=np.float64)).reshape(4, nth, nr)


@pytest.mark.parametrize("nr,nth", [(4095, 64), (4096, 64), (4097, 64), (4099, 67), (8192, 256), (9001, 301)])
def test_large_state_is_exact(nr, nth):
    print("case extract", nr, nth, flush=True)
    with T.Solver(cfg(nr, nth)) as s:
        for first in (1.0, -7.0e8):
            u = numbered(nr, nth, first)
            s.set_initial(u)
            np.testing.assert_array_equal(s.state(), u)


def test_copies_from_several_threads():
    """Six at once: more than there are buffer sets."""
    print("case extract threads", flush=True)
    u = [numbered(4099, 70 + i, 1.0e6 * i) for i in range(6)]
    solvers = [T.Solver(cfg(4099, 70 + i)) for i in range(6)]
    for s, v in zip(solvers, u):
        s.set_initial(v)
    bad = []

    def run(i):
        for _ in range(3):
            if not np.array_equal(solvers[i].state(), u[i]):
                bad.append(i)

    threads = [threading.Thread(target=run, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s in solvers:
        s.close()
    assert bad == []


@pytest.mark.parametrize("steps", [4, 5, 6, 13])
def test_ring_in_order_where_it_wraps(steps):
    print("case ring", steps, flush=True)
    u0 = W.random_state(100, 9, seed=3, smooth=True)
    kw = dict(x_extract=5.0, extract_every=1)
    with T.Solver(cfg(100, 9, max_samples=5, **kw)) as a, T.Solver(cfg(100, 9, max_samples=64, **kw)) as b:
        a.set_initial(u0)
        b.set_initial(u0)
        a.step(steps)
        b.step(steps)
        ta, wa = a.waveform()
        tb, wb = b.waveform()
        n = len(ta)
        assert n == min(5, len(tb))
        np.testing.assert_array_equal(ta, tb[-n:])
        np.testing.assert_array_equal(wa, wb[-n:])
