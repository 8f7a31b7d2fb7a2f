"""The direct sum's splits of targets and sources at their edges, and the
surface density with grids summed per block and straight in memory."""
import numpy as np
import pytest

from gpu_util import device, gpu_tree, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [0.01, 0.0])
@pytest.mark.parametrize("nt", [1, 63, 64, 65, 128, 129, 256, 257, 511, 513, 1100])
def test_direct_at_target_counts(oracle, nt, eps):
    import torch
    n = 1300 if nt != 513 else 70000
    s = ics.plummer(n, 95)
    idx = ics.subsample(n, nt, 96)
    t = gpu_tree(s.pos, s.mass)
    acc, pot = t.direct(torch.from_numpy(idx.astype(np.int64)).to(device()), eps)
    t.sync()
    acc, pot = acc.cpu().numpy(), pot.cpu().numpy()
    t.close()
    ra, rp = oracle.direct(s.pos, s.mass, float(np.float32(eps)), idx)
    ea = np.sqrt(((acc - ra) ** 2).sum(1) / (ra ** 2).sum(1))
    assert ea.max() <= 1e-12 and (np.abs(pot - rp) / np.abs(rp)).max() <= 1e-12


@pytest.mark.parametrize("n", [3, 511, 513, 5000, 300000])
@pytest.mark.parametrize("nr,nphi", [(1, 1), (2, 1), (16, 32), (64, 128), (64, 129)])
def test_density_grids(oracle, n, nr, nphi):
    import torch
    from paper_1412_0659_amd import Tree, binding as B
    grid = (0.2, 4.0, nr, nphi)
    s = ics.disk_halo(n - n // 3, n // 3, 97)
    t = Tree(n)
    sel = torch.from_numpy(s.is_disk.astype(np.uint8)).to(device())
    sig = torch.empty(nr, nphi, dtype=torch.float32, device="cuda")
    pos, mass = to_dev(s.pos), to_dev(s.mass)
    for mask, ref_mask in ((sel, s.is_disk), (None, None)):
        for _ in range(2):
            B.bh_cic_density(t.ctx, pos, mass, mask, grid, sig)
            t.sync()
            ref = oracle.cic_density(s.pos, s.mass, ref_mask, grid)
            assert np.abs(sig.cpu().numpy() - ref).max() <= 1e-5 * max(np.abs(ref).max(), 1e-30)
    t.close()
