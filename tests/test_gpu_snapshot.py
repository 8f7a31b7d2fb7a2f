"""Snapshots read and written in place against ones that are copied field by
field (not aligned for the FP64 positions): the same bytes, the same state."""
import numpy as np
import pytest

from gpu_util import device, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pos_fp64", [False, True])
@pytest.mark.parametrize("n", [1, 777, 10001])
def test_snapshot_in_place_and_copied(n, pos_fp64):
    import torch
    from paper_1412_0659_amd import Tree, binding as B
    device()
    s = ics.plummer(n, 91)
    t = Tree(n, pos_fp64=pos_fp64)
    t.set_state(to_dev(s.pos), to_dev(s.vel), to_dev(s.mass))
    t.step(1e-3, 0.5, 0.01)
    size = B.bh_state_bytes(t.ctx)
    a = torch.zeros(size, dtype=torch.uint8, device="cuda")
    store = torch.zeros(size + 4, dtype=torch.uint8, device="cuda")
    b = store[4:]
    B.bh_save_state(t.ctx, a)
    B.bh_save_state(t.ctx, b)
    assert torch.equal(a, b)
    t.step(1e-3, 0.5, 0.01)
    end = [x.cpu().numpy() for x in t.state()]
    for snap in (a, b):
        t.restore(snap, n)
        t.step(1e-3, 0.5, 0.01)
        for x, y in zip(t.state(), end):
            assert np.array_equal(x.cpu().numpy(), y)
    t.close()
