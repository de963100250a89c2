"""The diagnostics' choice of kernels goes by the slots that may be in use, also
where the particles came by a loaded state or by injection and not by a load: no
slower than on a handle that loaded as many (by the general kernels 5 to 7 times
as much)."""
import ctypes as C
import time

import numpy as np
import pytest

from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


def _us(g):
    import torch
    out = torch.empty(tuple(reversed(g.ext)), dtype=torch.float64, device="cuda")
    res = []
    for f in (g.diagnostics, lambda: g.L.empic_deposit_rho(g.h, -1, C.c_void_p(out.data_ptr()))):
        ts = []
        for _ in range(8):
            torch.cuda.synchronize()
            t = time.perf_counter()
            f()
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        res.append(1e6 * float(np.median(ts[1:])))
    return res


def _workload(n, bc, pos, seed=3):
    rng = np.random.default_rng(seed)
    sp = W.SpeciesInit("s", -1.0, 1.0, 0.01, pos, 0.05 * rng.standard_normal(pos.shape))
    return W.Workload("counts", n, (1.0,) * 3, W.courant_dt((1.0,) * 3), bc, [sp], sort_every=0)


def test_particles_of_a_loaded_state():
    from paper_2609_16575_amd.sim import Sim
    n = (96, 96, 96)
    pos = np.minimum(np.random.default_rng(2).random((4000000, 3)) * 96, np.nextafter(96.0, 0.0))
    w = _workload(n, (0, 0, 0), pos)
    a, b = Sim(w, precision="fp32"), Sim(w, precision="fp32")
    b.load_particles(0, np.zeros((0, 3)), np.zeros((0, 3)))
    a.sort()
    b.load_state(a.save_state())
    for x, y in zip(_us(a), _us(b)):
        assert y < 1.2 * x
    assert b.diagnostics()["n_particles"] == [4000000]
    a.close()
    b.close()


def test_injected_particles():
    from paper_2609_16575_amd.sim import Sim
    n, us = (64, 96, 96), []
    for injected in (True, False):
        cells = np.stack(np.meshgrid(*[np.arange(k) for k in n], indexing="ij"), -1).reshape(-1, 3)
        pos = np.repeat(cells + 0.5, 4, axis=0)
        w = _workload(n, (W.ABSORBING, 0, 0), pos[:8] if injected else pos)
        if injected:
            w.window = W.WindowInit(axis=0, cells=32, velocity=1.0, t_start=-1000.0,
                                    inject=[(0, (1, 2, 2), 0.01)])
        g = Sim(w, precision="fp32", capacity_slack=0.5)
        g.step(4)
        g.sort()
        us.append(_us(g))
        count = g.count(0)
        assert count > 0.9 * len(pos) or not injected, count
        g.close()
    for x, y in zip(us[1], us[0]):
        assert y < 1.25 * x, us
