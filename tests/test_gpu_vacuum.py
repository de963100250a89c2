"""A call of several steps on a large grid without particles, where Faraday and
Ampere are one pass between two buffer pairs, against calls of one step (the
point kernels, which the oracle tests cover): every boundary type, sources, odd
and even counts, extents at and around a patch of 31 x 15 points and a chunk of
8 or 16 planes.  Both form every value from the same FP64 expression, rounded
once per step: at most an ulp of the largest value per step apart."""
import numpy as np
import pytest

from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu

P, A, C = W.PERIODIC, W.ABSORBING, W.PEC


@pytest.mark.parametrize("n,bc,source,steps,precision", [
    ((101, 103, 202), (P, P, P), None, 4, "fp32"),
    ((101, 103, 202), (P, P, P), None, 3, "fp64"),
    ((62, 45, 750), (A, A, A), "laser", 5, "fp32"),
    ((90, 45, 502), (C, C, A), "port", 5, "fp32"),
    ((30, 15, 4600), (C, P, A), "port", 4, "fp32"),
    ((1024, 130, 16), (P, A, P), "laser", 2, "fp32"),
])
def test_pairs_equal_single_steps(n, bc, source, steps, precision):
    from paper_2609_16575_amd.sim import Sim
    out = []
    for calls in ((steps,), (1,) * steps):
        w = W.Workload("vacuum", n, (0.7, 0.9, 1.1), W.courant_dt((0.7, 0.9, 1.1)), bc, [])
        if source == "laser":
            w.laser = W.LaserInit(a0=1.0, w0=9.0, tau=3.0, t0=1.0, omega0=2.0,
                                  yc=0.45 * n[1], zc=0.55 * n[2], i_s=2)
        if source == "port":
            w.port = W.PortInit(2, 0, 1, 0, 1.0, 0.9, 2.0)
        w.E0, w.B0 = W.random_fields(n, bc, scale=0.02, seed=11)
        g = Sim(w, precision=precision)
        for t in g.J:
            t.fill_(7.0)
        for k in calls:
            g.step(k)
        out.append(g.fields())
        assert float(g.J.abs().max()) == 0.0
        g.close()
    ulp = 2.0 ** (-23 if precision == "fp32" else -52)
    for a, b in zip(*out):
        assert np.abs(a - b).max() <= steps * ulp * np.abs(b).max()
