"""J after one call of several steps: only the last one stores it, so it has to
equal, bit for bit, what the same number of one-step calls leaves - with and
without particles, filtered, in double precision, and where a call of several
steps is refused in its midst."""
import ctypes as C

import numpy as np
import pytest

from paper_2609_16575_amd import _lib as LB
from paper_2609_16575_amd import workloads as W
from test_gpu_window import _sim as window_sim
from test_gpu_window import _window_slab

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,plasma,filt", [
    ("fp32", True, 0), ("fp32", True, 1), ("fp32", False, 0), ("fp64", True, 0),
    ("fp64", False, 0),
])
def test_j_of_one_call_equals_single_steps(precision, plasma, filt):
    from paper_2609_16575_amd.sim import Sim
    out = []
    for calls in ((5,), (1, 1, 1, 1, 1)):
        w = W.langmuir_thermal(n=(16, 8, 12), ppc=2, steps=1)
        if not plasma:
            w.species = []
        w.E0, w.B0 = W.random_fields(w.n, scale=0.02, seed=5)
        g = Sim(w, precision=precision)
        if filt:
            LB.check(g.h, g.L.empic_set_filter(g.h, filt, 1))
        for t in g.J:
            t.fill_(7.0)
        for k in calls:
            g.step(k)
        out.append([a.copy() for a in g.fields()])
        g.close()
    # (FP64 deposits with atomic adds, in no fixed order)
    tol = 1e-12 if precision == "fp64" and plasma else 0.0
    for a, b in zip(*out):
        assert np.abs(a - b).max() <= tol * max(1.0, np.abs(b).max())


def test_j_where_a_call_is_refused_in_its_midst():
    out = []
    for many in (True, False):
        w = _window_slab(t_start=0.0)
        g = window_sim(w)
        per = (C.c_int32 * 3)(64, 64, 64)
        LB.check(g.h, g.L.empic_set_injection(g.h, 0, per, float(w.species[0].w)))
        st = 0
        for _ in range(1 if many else 200):
            st = g.L.empic_step(g.h, 200 if many else 1)
            if st:
                break
        assert st == 5
        out.append([a.copy() for a in g.fields()])
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
