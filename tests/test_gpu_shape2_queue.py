"""The second-order push's queue of two-part moves (256 per tile), against the
oracle: a tile with more crossing particles than the queue holds (the rest
deposit at once), one with hardly any, two species in one queue, and
per-particle weights.  One step from a common state, at the one-step bar."""
import numpy as np
import pytest

from gpu_common import compare_state, oracle_from
from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vth,count,wpp", [(2.0, 6000, False), (0.02, 4000, True)])
def test_two_part_queue_matches_oracle(vth, count, wpp):
    from paper_2609_16575_amd.sim import Sim
    rng = np.random.default_rng(51)
    n = (16, 16, 8)  # eight tiles
    L = np.asarray(n, dtype=float)
    sp = []
    for q, m in ((-1.0, 1.0), (1.0, 2.0)):
        # most of them in one tile
        pos = rng.random((count, 3)) * L
        pos[: count * 3 // 4] = rng.random((count * 3 // 4, 3)) * np.array([8.0, 8.0, 4.0])
        w1 = (0.5 + rng.random(count)) * 20.0 / count if wpp else None
        sp.append(W.SpeciesInit("s", q, m, 20.0 / count, pos, vth * rng.standard_normal((count, 3)),
                                wpp=w1))
    w = W.Workload("q2", n, (1.0,) * 3, W.courant_dt((1.0,) * 3), (0, 0, 0), sp, sort_every=0)
    w.E0, w.B0 = W.random_fields(n, scale=0.02, seed=52)
    g, o = Sim(w, precision="fp32", shape_order=2), oracle_from(w, w.E0, w.B0, 2)
    E, B, _ = g.fields()
    o.E[...] = E
    o.B[...] = B
    for i in range(2):
        P, U, _ = g.particles_by_id(i)
        o.species[i].pos[...] = P
        o.species[i].u[...] = U
    g.step(1)
    o.step(1)
    compare_state(g, o, w, sp_tol=2e-5, f_tol=2e-5, label="queue %g" % vth)
    g.close()
