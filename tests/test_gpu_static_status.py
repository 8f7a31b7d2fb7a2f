"""The status word of tree_force_static at the sizes where another launch
clears it: a call on bad particles reports them, the next call on good ones
is clean and gives the forces of a context."""
import numpy as np
import pytest

from gpu_util import gpu_force, gpu_tree, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1024, 1025, 8192, 8193, 65536])
def test_status_is_of_the_call(n):
    import torch
    from paper_1412_0659_amd import binding as B
    s = ics.plummer(max(n, 2), 95)
    pos, mass = s.pos[:n], s.mass[:n]
    st = torch.zeros(1, dtype=torch.int32, device="cuda")

    def call(p, m):
        print(f"static n={n}", flush=True)
        acc = torch.empty((n, 3), dtype=torch.float32, device="cuda")
        pot = torch.empty((n,), dtype=torch.float32, device="cuda")
        B.tree_force_static(to_dev(p), to_dev(m), 0.6, 0.01, acc, pot, st)
        torch.cuda.synchronize()
        return acc.cpu().numpy(), pot.cpu().numpy(), int(st.cpu().item())

    t = gpu_tree(pos, mass)
    ra, rp = gpu_force(t, 0.6, 0.01)
    t.close()
    heavy = mass.copy()
    heavy[n - 1] = 0.0
    for bad in (heavy, -mass):
        assert call(pos, bad)[2] == 2  # mass <= 0
        acc, pot, ok = call(pos, mass)
        assert ok == 0 and np.array_equal(acc, ra) and np.array_equal(pot, rp)
