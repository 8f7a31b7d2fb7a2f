"""Surface density on either side of the lines between the two deposits (adds
straight to memory, or on the blocks' own grids in LDS), and across the own
grids' largest size, against the oracle."""
import numpy as np
import pytest

from gpu_util import device, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nphi,ns", [(8, 8, (1, 63, 64, 5000)), (16, 16, (255, 256)),
                                        (1, 257, (257, 4111, 4112)), (32, 64, (32767, 32768)),
                                        (64, 128, (8192, 131071, 131072)), (1, 8193, (131088,))])
def test_both_deposits(oracle, nr, nphi, ns):
    """A weight is linear in a cell coordinate of up to max(nr, nphi), FP32 after
    some six roundings, and a cell's particles hold up to four times the mass
    that it gets (their sums are FP64): 4 x 6 x 2^-24 max(nr, nphi) of the
    largest density."""
    import torch
    from paper_1412_0659_amd import Tree, binding as B
    device()
    grid = (0.2, 4.0, nr, nphi)
    for n in ns:
        s = ics.disk_halo_scaled(max(n, 10), 99)
        pos, mass = s.pos[:n].copy(), s.mass[:n].copy()
        t = Tree(n)
        for sel in (None, np.arange(n) % 5 != 0):
            print(f"density n={n} {nr}x{nphi} selected {sel is not None}", flush=True)
            den = torch.empty(nr, nphi, dtype=torch.float32, device="cuda")
            dsel = None if sel is None else torch.from_numpy(sel).cuda()
            B.bh_cic_density(t.ctx, to_dev(pos), to_dev(mass), dsel, grid, den)
            t.sync()
            ref = oracle.cic_density(pos, mass, sel, grid)
            got = den.cpu().numpy().astype(np.float64)
            assert np.abs(got - ref).max() <= 24 * 2.0**-24 * max(nr, nphi) * ref.max()
        t.close()
