"""The order in which the push takes the tiles - on grids of 150 and more tiles
per layer in groups of four layers along z, the last one with fewer, else layer
by layer - reaches every tile once: 1 to 10 layers, unequal in x and y, with one
and several workgroups per tile, against the oracle, at both shape orders.  One step from a common state at 2e-5, as
elsewhere."""
import pytest

from gpu_common import compare_state, oracle_from
from test_gpu_split import _common_state, _workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count,order", [
    ((120, 80, 12), 6000, 1),
    ((81, 117, 17), 6000, 1),
    ((400, 17, 32), 6000, 2),
    ((1200, 2, 40), 6000, 1),
    ((24, 16, 12), 40000, 1),
    ((24, 16, 12), 9000, 1),
    ((8, 24, 20), 30001, 1),
    ((16, 8, 37), 30000, 2),
    # one electron ends 1e-8 of a cell below y = 1 in double precision and on it in
    # single: its twelve edges of J differ by up to 2.1e-4 (everything else holds)
    pytest.param((32, 4, 24), 30001, 1, marks=pytest.mark.xfail(
        reason="an electron within FP32 rounding of a cell face", strict=False)),
])
def test_push_reaches_every_tile(n, count, order):
    from paper_2609_16575_amd.sim import Sim
    w = _workload(n, (count,), 0.3, 47)
    g, o = Sim(w, precision="fp32", shape_order=order), oracle_from(w, w.E0, w.B0, order)
    _common_state(g, o, w)
    g.step(1)
    o.step(1)
    compare_state(g, o, w, sp_tol=2e-5, f_tol=2e-5, label="tile groups %s" % (n,))
    g.close()
