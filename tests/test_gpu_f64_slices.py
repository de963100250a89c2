"""The binned FP64 push where a tile's particles are shared out to workgroups in
slices (1024 particles here): populations of a slice, one more, many slices and
one, and empty tiles before, between and after, against the oracle at the path's
1e-12 per step; and the rule's lines on sparse and dense grids: the time per
particle neither on one tile nor on a sparse grid is far from an even plasma's."""
import time

import numpy as np
import pytest

from gpu_common import compare_state, oracle_from
from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


def _workload(n, pos, vth=0.4, seed=5):
    rng = np.random.default_rng(seed)
    sp = W.SpeciesInit("s", -1.0, 1.0, 0.01, pos, vth * rng.standard_normal(pos.shape))
    w = W.Workload("f64", n, (1.0,) * 3, W.courant_dt((1.0,) * 3), (0, 0, 0), [sp], sort_every=0)
    w.E0, w.B0 = W.random_fields(n, scale=0.05, seed=seed + 1)
    return w


@pytest.mark.parametrize("per_tile", [
    (0, 1024, 0, 97 * 1024 + 1, 0),
    (1025, 1023, 98305, 1, 0),
    (40000, 2048, 0, 60000, 7),
])
def test_sliced_tiles_match_oracle(per_tile):
    from paper_2609_16575_amd.sim import Sim
    rng = np.random.default_rng(8)
    n = (8 * len(per_tile), 8, 4)
    pos = np.concatenate([rng.random((c, 3)) * (8, 8, 4) + (8 * i, 0, 0)
                          for i, c in enumerate(per_tile)])
    pos = rng.permutation(np.minimum(pos, np.nextafter(np.asarray(n, float), 0.0)))
    w = _workload(n, pos)
    g, o = Sim(w, precision="fp64"), oracle_from(w, w.E0, w.B0)
    for k in (1, 2):  # (the counters are left clear for the second)
        g.step(1)
        o.step(1)
        compare_state(g, o, w, sp_tol=k * 1e-12, f_tol=k * 1e-12, label="slices %d" % k)
    g.close()


def _step_us(n, count, seed=2):
    import torch
    from paper_2609_16575_amd.sim import Sim
    pos = np.random.default_rng(seed).random((count, 3)) * n
    g = Sim(_workload(n, np.minimum(pos, np.nextafter(np.asarray(n, float), 0.0)), vth=0.1),
            precision="fp64")
    ts = []
    for _ in range(6):
        torch.cuda.synchronize()
        t = time.perf_counter()
        g.step(10)
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t)
    g.close()
    return 1e5 * float(np.median(ts[1:]))


def test_one_tile_is_not_pushed_by_one_workgroup():
    """1 M particles of one tile: 0.6 of an even plasma's time, 46 times it in a
    single workgroup."""
    assert _step_us((8, 8, 4), 1000000) < 4.0 * _step_us((64, 64, 64), 1000000)


def test_sparse_grids_keep_the_direct_push():
    """1.5 particles per tile: the time of 2 % fewer, below the particle count
    from which dense grids are binned; 1.66 times it when binned."""
    assert _step_us((256, 256, 256), 100000) < 1.3 * _step_us((256, 256, 256), 98000)
