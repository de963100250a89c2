"""The current sheet on node plane n of a periodic x axis, which is plane 0 (a
row holds n nodes, so that an index of n lies past its end), against the oracle
at the one-step bars, and as plane 0 bit for bit."""
import numpy as np
import pytest

from gpu_common import oracle_from
from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,bc,tol", [
    ("fp32", (0, 0, 0), 2e-5),
    ("fp64", (0, 0, 0), 1e-12),
    ("fp32", (0, W.ABSORBING, W.PEC), 2e-5),
])
def test_last_node_plane_of_a_periodic_axis(precision, bc, tol):
    from paper_2609_16575_amd.sim import Sim
    n, out = (9, 6, 7), []
    for plane in (n[0], 0):
        w = W.Workload("sheet", n, (1.0,) * 3, W.courant_dt((1.0,) * 3), bc, [])
        w.laser = W.LaserInit(a0=1.0, w0=4.0, tau=3.0, t0=0.2, omega0=1.0, yc=3.0, zc=3.0,
                              i_s=plane)
        w.E0, w.B0 = W.random_fields(n, bc, scale=0.05, seed=9)
        g, o = Sim(w, precision=precision), oracle_from(w, w.E0, w.B0)
        E, B, _ = g.fields()
        o.E[...] = E
        o.B[...] = B
        g.step(1)
        o.step(1)
        E, B, _ = g.fields()
        for a, b in ((E, o.E), (B, o.B)):
            assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))
        out.append((E, B))
        g.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
