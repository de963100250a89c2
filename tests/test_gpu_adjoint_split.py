"""The adjoint's gather scatter where workgroups share a tile: a tile adds one
FP32 value per point and component, whatever the number of workgroups, so that
points which only one tile's particles reach come out the same, bit for bit, in
every run (an FP32 sum of several partial windows depends on their order)."""
import numpy as np
import pytest

from test_gpu_split import _workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count", [
    ((16, 16, 8), 40000),   # six workgroups per tile, one component each
    ((32, 32, 32), 150000),  # two, three components each
    ((32, 2, 16), 9000),    # the thin grids' tile
])
def test_tile_sums_do_not_depend_on_the_run(n, count):
    import torch
    from paper_2609_16575_amd.sim import Sim
    g = Sim(_workload(n, (count,), 0.3, 51), precision="fp32")
    g.sort()
    st = g.save_state()
    gen = torch.Generator(device="cuda").manual_seed(7)
    lam = g.alloc_adjoint()
    tens = [lam["E"], lam["B"], lam["pos"][0], lam["u"][0]]
    start = [torch.randn(t.shape, generator=gen, device="cuda") for t in tens]
    # interior of a tile: the curl of the transposed step reaches one point down
    side = (8, 8, 4) if n[1] > 3 else (16, 2, 8)
    inner = np.ones(tuple(reversed(n)), bool)
    for a in range(3):
        i = np.arange(n[a]) % side[a]
        ok = (i >= 2) & (i <= side[a] - 2) if side[a] > 2 else np.ones(n[a], bool)
        inner &= ok.reshape([-1 if b == 2 - a else 1 for b in range(3)])
    assert inner.any()
    first = None
    for _ in range(6):
        for t, s in zip(tens, start):
            t.copy_(s)
        g.step_vjp(st, lam)
        out = [lam["E"].cpu().numpy()[:, inner], lam["B"].cpu().numpy()[:, inner],
               lam["pos"][0][:, :count].cpu().numpy(), lam["u"][0][:, :count].cpu().numpy()]
        first = first or out
        for a, b in zip(out, first):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    g.close()
