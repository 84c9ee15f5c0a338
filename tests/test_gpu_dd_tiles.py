"""GPU: the double-double stage at the edges of its tiles (63 points, one row),
F(u) and one step against the binary128 oracle.

Tolerance: with u = 2^-53 a stage rounds its result to about 3 u^2 and its F(u), whose
terms are sums of products formed to a few u^2 each, enters times dt F <~ u; three
stages stay well within 80 u^2 = 1e-30 of the largest value, and so does F(u) of its own."""
import numpy as np
import pytest

import paper_2010_04760_amd as T
import workloads as W
from oracle import quad as Q
from oracle import solver as S

pytestmark = pytest.mark.gpu


def err(got, ref):
    d = (got[..., 0] - ref[..., 0]) + (got[..., 1] - ref[..., 1])
    return float(np.max(np.abs(d)) / np.max(np.abs(ref[..., 0])))


@pytest.mark.parametrize("weights", ["quad", "fp64"])
@pytest.mark.parametrize("nr,nth", [(7, 2), (62, 9), (63, 2), (64, 3), (126, 4), (127, 5), (189, 17)])
def test_tile_edges(nr, nth, weights):
    print("case dd tiles", nr, nth, weights, flush=True)
    prob = S.Problem(-2, 1, 0.9, nr, nth, -30.0, 50.0)
    dt = 0.4 * S.TeukOracle(prob).dt_bound(1.0)
    o = Q.TeukOracleQ(prob, weights=weights)
    u0 = Q.promote(W.random_state(nr, nth, seed=nr, smooth=True))
    ref, _ = o.evolve(u0, dt, 1)
    cfg = T.make_config(s=-2, m=1, a=0.9, nr=nr, ntheta=nth, x_min=-30.0, x_max=50.0, dt=dt, state="dd",
                        weight_prec="dd" if weights == "quad" else "fp64")
    with T.Solver(cfg) as sv:
        sv.set_initial(u0)
        assert err(sv.rhs(), o.rhs(u0)) <= 1e-30
        sv.step(1)
        assert err(sv.state(), ref) <= 1e-30
