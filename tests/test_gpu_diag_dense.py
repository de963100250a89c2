"""Charge density of tile-grouped particles where a node takes far more
contributions than a fixed-point window could: both shape orders, tiles of 2^21
and more particles of full weight, and light particles beside a heavy one."""
import numpy as np
import pytest

from paper_2609_16575_amd import workloads as W

pytestmark = pytest.mark.gpu


def _sim(n, pos, wpp, order):
    from paper_2609_16575_amd.sim import Sim
    sp = W.SpeciesInit("s", -1.0, 1.0, 1.0, pos, np.zeros_like(pos), wpp=wpp)
    w = W.Workload("dense", n, (1.0,) * 3, W.courant_dt((1.0,) * 3), (0, 0, 0), [sp], sort_every=0)
    return Sim(w, precision="fp32", shape_order=order)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("lattice", [(32, 32, 32), (64, 32, 32)])
def test_uniform_dense_plasma_has_density_one(order, lattice):
    """Weights 1/ppc on a regular lattice: -1 at every node, as the B-splines sum
    to one.  27 x 65536 FP64 additions of one sign: at most 2e-10 of the sum."""
    n = (4, 4, 4)
    ax = [(np.arange(n[a] * lattice[a]) + 0.5) / lattice[a] for a in range(3)]
    pos = np.stack(np.meshgrid(*ax, indexing="ij"), axis=-1).reshape(-1, 3)
    ppc = int(np.prod(lattice))
    g = _sim(n, pos, np.full(len(pos), 1.0 / ppc), order)
    g.sort()
    assert np.max(np.abs(g.rho() + 1.0)) <= 2e-10
    assert abs(g.diagnostics()["gauss_max"] - 1.0) <= 2e-10
    g.close()


def test_light_particles_keep_their_bits_at_second_order():
    """A particle of weight 1 in the middle of a tile, the others 1e-9: every node
    out of its reach agrees with the general FP64 kernel (the particles freshly
    loaded, not grouped by tiles) to 1e-12 of itself, a few hundred additions of
    one sign."""
    n, count = (8, 8, 8), 20000
    rng = np.random.default_rng(3)
    pos = np.minimum(rng.random((count, 3)) * n, np.nextafter(8.0, 0.0))
    pos[0] = (3.6, 3.6, 1.6)
    wpp = np.full(count, 1e-9)
    wpp[0] = 1.0
    g, f = _sim(n, pos, wpp, 2), _sim(n, pos, wpp, 2)
    g.sort()
    a, b = g.rho(), f.rho()
    far = np.ones((8, 8, 8), bool)
    far[0:5, 2:7, 2:7] = False
    assert np.max(np.abs(a - b)[far] / np.abs(b)[far]) <= 1e-12
    g.close()
    f.close()
