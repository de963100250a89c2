"""The push on grids thinner along y than a cubic tile (four cells of eight, so
that a window wraps onto itself), with one and with several workgroups per tile,
at both shape orders, against the oracle: one step from a common state at 2e-5,
as elsewhere.  That bar is for particles whose end point rounds to the same side
of every cell face in single and double precision: none of these ends within
2e-7 of one (asserted), a few units in the last place of an offset."""
import numpy as np
import pytest

from gpu_common import compare_state, oracle_from
from test_gpu_split import _common_state, _workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count,order,seed", [
    ((32, 4, 24), 30001, 1, 48),
    ((32, 4, 24), 5000, 1, 49),
    ((32, 4, 24), 30001, 2, 50),
    ((24, 5, 20), 9001, 1, 51),
])
def test_thin_grid_matches_oracle(n, count, order, seed):
    from paper_2609_16575_amd.sim import Sim
    w = _workload(n, (count,), 0.3, seed)
    g, o = Sim(w, precision="fp32", shape_order=order), oracle_from(w, w.E0, w.B0, order)
    _common_state(g, o, w)
    g.step(1)
    o.step(1)
    xi = o.species[0].pos / np.asarray(w.d)
    assert np.abs(xi - np.round(xi)).min() > 2e-7
    compare_state(g, o, w, sp_tol=2e-5, f_tol=2e-5, label="thin %s" % (n,))
    g.close()
