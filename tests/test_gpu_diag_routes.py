"""Charge density and diagnostics on each side of the rules that choose their
kernels by the particles per tile, against the general kernels on the same state
(bars of test_gpu_diag_tiles): narrow and wide workgroups for the charge on
cubic and thin tiles and at second order, and more tiles than partial slots; and
on a sparse grid particles grouped by tiles cost no more than ungrouped ones."""
import ctypes as C
import time

import numpy as np
import pytest

import test_gpu_diag_tiles
from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc,order,wpp,count", [
    ((17, 9, 5), (0, 0, 0), 1, True, 9000),      # 750 per tile: wide
    ((40, 2, 20), (W.ABSORBING, 0, W.ABSORBING), 1, True, 2000),  # 222: narrow
    ((17, 9, 7), (0, 0, 0), 2, False, 9000),     # 750, second order
    ((64, 64, 72), (0, 0, 0), 1, False, 30000),  # 26, charge and energies apart
    ((64, 64, 72), (0, 0, 0), 2, True, 60000),   # 52, together
    ((260, 128, 132), (0, 0, 0), 1, False, 1800000),  # 103 in 17424 tiles, 16384 slots
])
def test_routes_match_the_general_kernels(n, bc, order, wpp, count):
    test_gpu_diag_tiles.test_tile_diagnostics_match_the_general_kernels(n, bc, order, wpp, count)


def _us(f):
    import torch
    ts = []
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t)
    return 1e6 * float(np.median(ts[1:]))


@pytest.mark.parametrize("order", [1, 2])
def test_sparse_tiles_cost_no_more_than_ungrouped_particles(order):
    """1.5 particles per tile; 1.4 to 2.1 times as much by tiles."""
    import torch
    from paper_2609_16575_amd.sim import Sim
    n, rng = (256, 256, 256), np.random.default_rng(4)
    pos = np.minimum(rng.random((100000, 3)) * n, np.nextafter(256.0, 0.0))
    w = W.Workload("sparse", n, (1.0,) * 3, W.courant_dt((1.0,) * 3), (0, 0, 0), [
        W.SpeciesInit("s", -1.0, 1.0, 0.01, pos, 0.1 * rng.standard_normal(pos.shape))],
        sort_every=0)
    g = Sim(w, precision="fp32", shape_order=order)
    out = torch.empty(tuple(reversed(n)), dtype=torch.float64, device="cuda")
    calls = (g.diagnostics,
             lambda: g.L.empic_deposit_rho(g.h, -1, C.c_void_p(out.data_ptr())))
    loose = [_us(f) for f in calls]
    g.sort()
    grouped = [_us(f) for f in calls]
    for a, b in zip(grouped, loose):
        assert a < 1.25 * b, (grouped, loose)
    g.close()
