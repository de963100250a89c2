"""The current filter's launch rule, against the oracle: filters of up to 4
(FP32) or 2 (FP64) passes per axis run in one launch over 32 x 8 x 4 patches,
wider ones pass by pass (an odd and an even number of passes).  Ragged grids,
grids thinner than a patch's halo, walled and mixed axes.  Tolerances: one
step's (2e-5 FP32, 1e-12 FP64), as in the other filter tests."""
import numpy as np
import pytest

from gpu_common import compare_state, oracle_from
from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(n, bc, filt, prec, tol, seed):
    from paper_2609_16575_amd.sim import Sim
    rng = np.random.default_rng(seed)
    d = (1.0, 0.9, 1.1)
    L = np.asarray(n) * np.asarray(d)
    pos = np.minimum(rng.random((3000, 3)) * L, np.nextafter(L, 0.0))
    sp = [W.SpeciesInit("s", -1.0, 1.0, 0.3, pos, 0.3 * rng.standard_normal((3000, 3)))]
    w = W.Workload("filt", n, d, W.courant_dt(d), bc, sp, sort_every=0, filter=filt)
    w.E0, w.B0 = W.random_fields(n, bc=bc, scale=0.05, seed=seed + 1)
    for a in range(3):  # tangential E is zero on PEC walls
        for c in range(3):
            if bc[a] == W.PEC and c != a:
                for side in (0, n[a]):
                    sl = [slice(None)] * 3
                    sl[2 - a] = side
                    w.E0[c][tuple(sl)] = 0.0
    g = Sim(w, precision=prec)
    o = oracle_from(w, w.E0, w.B0)
    if prec == "fp32":
        E, B, _ = g.fields()
        o.E[...] = E
        o.B[...] = B
        P, U, _ = g.particles_by_id(0)
        o.species[0].pos[...] = P
        o.species[0].u[...] = U
    g.step(1)
    o.step(1)
    compare_state(g, o, w, sp_tol=tol, f_tol=tol, label="filter %s %s %s %s" % (n, bc, filt, prec))
    g.close()


@pytest.mark.parametrize("filt", [(1, 0), (1, 1), (3, 0), (3, 1), (4, 1), (6, 0)])
@pytest.mark.parametrize("n,bc", [((33, 9, 5), (0, 0, 0)), ((2, 8, 4), (0, 0, 0)),
                                  ((35, 8, 7), (W.PEC, 0, W.ABSORBING))])
def test_filter_fp32_every_width(n, bc, filt):
    _run(n, bc, filt, "fp32", 2e-5, 21)


@pytest.mark.parametrize("filt", [(0, 1), (2, 0), (2, 1), (3, 1)])
@pytest.mark.parametrize("n", [(33, 9, 5), (3, 2, 64)])
def test_filter_fp64_every_width(n, filt):
    _run(n, (0, 0, 0), filt, "fp64", 1e-12, 23)
