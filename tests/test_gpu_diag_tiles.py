"""Diagnostics of tile-grouped particles (charge density and both kinetic
energies in one pass over the tiles) against the general kernels on the same
state: particles that left their tiles and windows since the last sort, ragged
and thin grids, walls, per-particle weights, second-order shapes, and more
tiles than partial slots.  The two differ in the order of FP64 sums and, for
the charge, by the tiles' fixed point (2^-48 of one particle's contribution):
1e-11 of the largest value."""
import numpy as np
import pytest

from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc,order,wpp,count", [
    ((17, 9, 5), (0, 0, 0), 1, True, 3000),
    ((40, 2, 20), (W.ABSORBING, 0, W.ABSORBING), 1, False, 6000),
    ((17, 9, 7), (0, 0, 0), 2, True, 3000),
    ((260, 128, 132), (0, 0, 0), 1, False, 40000),  # 17424 tiles, 16384 slots
])
def test_tile_diagnostics_match_the_general_kernels(n, bc, order, wpp, count):
    from paper_2609_16575_amd.sim import Sim
    rng = np.random.default_rng(5)
    L = np.asarray(n, dtype=float)
    pos = np.minimum(rng.random((count, 3)) * L, np.nextafter(L, 0.0))
    w1 = 0.01 * (0.5 + rng.random(count)) if wpp else None
    sp = W.SpeciesInit("s", -1.0, 1.0, 0.01, pos, 0.8 * rng.standard_normal((count, 3)), wpp=w1)
    w = W.Workload("diag", n, (1.0,) * 3, W.courant_dt((1.0,) * 3), bc, [sp], sort_every=0)
    w.E0, w.B0 = W.random_fields(n, bc=bc, scale=0.02, seed=6)
    a = Sim(w, precision="fp32", shape_order=order)
    a.step(10)
    da, ra = a.diagnostics(), a.rho()
    assert da["fallback_particles"] > 0  # some are outside their windows
    # the same state, freshly loaded: not grouped by tiles, the general kernels
    P, U, I = a.particles(0)
    E, B, _ = a.fields()
    w2 = W.Workload("diag", n, w.d, w.dt, bc, [W.SpeciesInit(
        "s", -1.0, 1.0, 0.01, P, U, wpp=None if w1 is None else w1[I])], sort_every=0)
    w2.E0, w2.B0 = E, B
    b = Sim(w2, precision="fp32", shape_order=order)
    db, rb = b.diagnostics(), b.rho()
    assert np.max(np.abs(ra - rb)) <= 1e-11 * np.max(np.abs(rb))
    for k in ("K_minus", "K_plus"):
        assert abs(da[k][0] - db[k][0]) <= 1e-11 * abs(db[k][0]), k
    for k in ("U_E", "U_B"):
        assert da[k] == db[k]
    assert da["n_particles"] == [len(I)] or bc != (0, 0, 0)
    a.close()
    b.close()
