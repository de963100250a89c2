"""The plain FP64 path from F64_TILED_MIN (98304) particles on, where the push
bins the particles by tiles of cells: against the oracle on grids thinner than
a tile, ragged ones, one with more tiles than the binning's LDS counters hold,
particles in random order, cell crossings and periodic wraps, two species and
per-particle weights.  Tolerances: those of the path's other parity tests
(1e-12 per step)."""
import numpy as np
import pytest

from gpu_common import compare_state, oracle_from
from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


def _workload(n, count, wpp, seed):
    rng = np.random.default_rng(seed)
    d = (1.0, 0.9, 1.1)
    L = np.asarray(n) * np.asarray(d)
    sp = []
    for q, m in ((-1.0, 1.0), (1.0, 4.0)):
        pos = np.minimum(rng.random((count, 3)) * L, np.nextafter(L, 0.0))
        u = 0.4 * rng.standard_normal((count, 3))
        w = 0.5 + rng.random(count) if wpp else None
        sp.append(W.SpeciesInit("s", q, m, 0.01, pos, u, wpp=None if w is None else 0.01 * w))
    w = W.Workload("f64", n, d, W.courant_dt(d), (0, 0, 0), sp, sort_every=0)
    w.E0, w.B0 = W.random_fields(n, scale=0.05, seed=seed + 1)
    return w


@pytest.mark.parametrize("n,count,wpp", [
    ((17, 9, 5), 98304, False),      # ragged last tiles on every axis
    ((8, 8, 4), 98304, True),        # one tile: every window point wraps onto it
    ((1, 2, 70), 98305, False),      # thinner than a window along x and y
    ((256, 128, 132), 100001, True),  # 16896 tiles: counters in global memory
])
def test_binned_push_matches_oracle(n, count, wpp):
    from paper_2609_16575_amd.sim import Sim
    w = _workload(n, count, wpp, 11)
    g, o = Sim(w, precision="fp64"), oracle_from(w, w.E0, w.B0)
    g.step(1)
    o.step(1)
    compare_state(g, o, w, sp_tol=1e-12, f_tol=1e-12, label="binned 1 %s" % (n,))
    g.step(2)  # the counters are left clear for the next step and species
    o.step(2)
    compare_state(g, o, w, sp_tol=3e-12, f_tol=3e-12, label="binned 3 %s" % (n,))
    g.sync()
    g.close()
