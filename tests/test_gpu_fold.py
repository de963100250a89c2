"""The push of thin periodic grids (one or two cells along y) in windows folded
onto the rows that exist, against the oracle: both thicknesses, periodic and
walled x and z with ragged last tiles and grids smaller than a window, per-
particle weights, sparse and dense tiles (one and four particles per thread),
cell crossings in y that wrap, and particles that leave their windows.  One
step from a common state at the one-step bar (2e-5), then six more at 1e-4 as
the other multi-step FP32 tests."""
import numpy as np
import pytest

from gpu_common import compare_state, oracle_from
from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc,count,wpp", [
    ((40, 2, 20), (0, 0, 0), 4000, False),
    ((37, 1, 19), (W.ABSORBING, 0, W.PEC), 3000, True),
    ((9, 2, 5), (0, 0, W.ABSORBING), 6000, True),   # smaller than a window; dense
    ((16, 1, 8), (0, 0, 0), 9000, False),           # one tile, its own neighbour
    ((70, 2, 33), (W.ABSORBING, 0, W.ABSORBING), 60000, False),
])
def test_folded_push_matches_oracle(n, bc, count, wpp):
    from paper_2609_16575_amd.sim import Sim
    rng = np.random.default_rng(31)
    d = (1.0, 0.8, 1.2)
    L = np.asarray(n) * np.asarray(d)
    pos = np.minimum(rng.random((count, 3)) * L, np.nextafter(L, 0.0))
    w1 = (0.5 + rng.random(count)) * 20.0 / count if wpp else None
    sp = W.SpeciesInit("s", -1.0, 1.0, 20.0 / count, pos, 0.7 * rng.standard_normal((count, 3)),
                       wpp=w1)
    w = W.Workload("fold", n, d, W.courant_dt(d), bc, [sp], sort_every=0)
    w.E0, w.B0 = W.random_fields(n, bc=bc, scale=0.02, seed=32)
    for a in range(3):  # tangential E is zero on PEC walls
        for c in range(3):
            if bc[a] == W.PEC and c != a:
                for side in (0, n[a]):
                    sl = [slice(None)] * 3
                    sl[2 - a] = side
                    w.E0[c][tuple(sl)] = 0.0
    g, o = Sim(w, precision="fp32"), oracle_from(w, w.E0, w.B0)
    E, B, _ = g.fields()
    o.E[...] = E
    o.B[...] = B
    P, U, _ = g.particles_by_id(0)
    o.species[0].pos[...] = P
    o.species[0].u[...] = U
    g.step(1)
    o.step(1)
    compare_state(g, o, w, sp_tol=2e-5, f_tol=2e-5, label="fold 1 %s" % (n,))
    g.step(6)
    o.step(6)
    compare_state(g, o, w, sp_tol=1e-4, f_tol=1e-4, label="fold 7 %s" % (n,))
    if n[0] > 30:  # up to 3.5 cells in 7 steps: some left their windows
        assert g.diagnostics()["fallback_particles"] > 0
    g.close()
