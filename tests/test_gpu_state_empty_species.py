"""empic_step_state with a species of capacity 0, which has no arrays in a state:
the same destination, bit for bit, as a handle without that species, at both
shape orders and with particles that left their windows since the sort."""
import ctypes as C

import numpy as np
import pytest

from paper_2609_16575_amd import _lib as LB
from test_gpu_split import _workload

pytestmark = pytest.mark.gpu


def _sim_class():
    from paper_2609_16575_amd.sim import Sim

    class EmptySim(Sim):
        """Registers species without particles at capacity 0."""

        def _add_species(self, s, cap):
            if len(s.pos):
                return super()._add_species(s, cap)
            b = [self._alloc_set(8, False) for _ in range(2)]
            sd = LB.SpeciesDesc(float(s.q), float(s.m), float(s.w), 0, 0)
            sid = C.c_int32()
            LB.check(self.h, self.L.empic_add_species(self.h, C.byref(sd), 0, C.byref(b[0]["pb"]),
                                                      C.byref(b[1]["pb"]), C.byref(sid)))
            self.caps[sid.value] = 0
            self.bufs.append(tuple(b))

        def _state_struct(self, st):
            S = super()._state_struct(st)
            for i, cap in enumerate(self.caps):
                if cap == 0:
                    S.cell[i] = S.id[i] = S.w[i] = S.tiles[i] = None
                    for a in range(3):
                        S.pos[i][a] = S.u[i][a] = None
            return S

    return EmptySim


@pytest.mark.parametrize("empty", [0, 1])
@pytest.mark.parametrize("n,count,order", [
    ((16, 16, 8), 3000, 1),
    ((17, 9, 12), 5000, 2),
    ((40, 2, 20), 3000, 1),
])
def test_empty_species_changes_nothing(n, count, order, empty):
    EmptySim = _sim_class()
    w = _workload(n, (count,), 0.6, 61)
    out = []
    for with_empty in (False, True):
        if with_empty:
            none, s = np.zeros((0, 3)), w.species[0]  # (the same weight: J's scale follows the largest)
            w.species.insert(empty, type(s)("none", 1.0, 1.0, s.w, none, none))
        g = EmptySim(w, precision="fp32", shape_order=order)
        g.sort()
        g.step(6)  # some particles leave their windows
        st = [g.save_state(), g.alloc_state()]
        for k in range(4):
            g.step_state(st[k % 2], st[(k + 1) % 2])
        g.sync()
        i = 1 - empty if with_empty else 0
        by_id = np.argsort(st[0]["id"][i].cpu().numpy()[:count])
        out.append([st[0][k].cpu().numpy() for k in ("E", "B")]
                   + [st[0][k][i].cpu().numpy()[..., by_id] for k in ("cell", "pos", "u")])
        assert g.diagnostics()["fallback_particles"] > 0
        g.close()
    for a, b in zip(*out):
        same = np.array_equal(a.view(np.uint32), b.view(np.uint32))
        assert same
