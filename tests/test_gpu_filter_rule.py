"""The current filter where few passes run one by one, on grids that the patches
do not suit, against the oracle at the one-step bars; and the rule's lines: a
filter of four passes per axis costs no more than one of five, which never goes
by patches."""
import time

import numpy as np
import pytest

from paper_2609_16575_amd import workloads as W
from test_gpu_filter_tile import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc,filt,prec,tol", [
    ((2, 96, 400), (0, 0, 0), (1, 0), "fp32", 2e-5),   # in place of one launch: three
    ((2, 96, 400), (0, 0, 0), (1, 1), "fp32", 2e-5),
    ((3, 96, 400), (W.ABSORBING, 0, W.PEC), (3, 0), "fp32", 2e-5),
    ((2, 96, 400), (0, 0, 0), (3, 1), "fp32", 2e-5),
    ((2, 96, 400), (0, 0, 0), (1, 0), "fp64", 1e-12),
    ((2, 96, 400), (0, 0, 0), (1, 1), "fp64", 1e-12),
])
def test_few_passes_one_by_one(n, bc, filt, prec, tol):
    _run(n, bc, filt, prec, tol, 25)


@pytest.mark.parametrize("n", [(2, 512, 512), (512, 2, 512), (128, 128, 128)])
def test_four_passes_cost_no_more_than_five(n):
    """By patches 11, 3.3 and 1.6 times as much."""
    import torch
    from paper_2609_16575_amd.sim import Sim
    ms = []
    for passes in (4, 5):
        w = W.Workload("filt", n, (1.0,) * 3, W.courant_dt((1.0,) * 3), (0, 0, 0), [
            W.SpeciesInit("s", -1.0, 1.0, 0.3, np.full((8, 3), 0.5), np.zeros((8, 3)))],
            sort_every=0, filter=(passes, 0))
        g, ts = Sim(w, precision="fp32"), []
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            g.step(20)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        ms.append(1e3 * float(np.median(ts[1:])))
        g.close()
    assert ms[0] < 1.1 * ms[1], ms
