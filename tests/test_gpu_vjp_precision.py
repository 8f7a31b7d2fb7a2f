"""The particle and the cell part of a target's gradient meet in FP64: a pair
close together, whose two sides cancel in each particle's gradient under a
uniform cotangent, leaves the cells' part as exact as it is without the pair."""
import numpy as np
import pytest

from gpu_util import device, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sep", [0.02, 0.005])
@pytest.mark.parametrize("far", [60, 2500])
def test_close_pair_keeps_the_cells_part(oracle, far, sep):
    """One group of two particles sep apart, everything else accepted as
    cells: the pair's terms, m / sep^3 in FP32, are equal bits on both sides
    (masses and cotangents are equal) and cancel in the FP64 sums.  What is
    left is FP32 arithmetic on the cells' terms: 1e-5 of their size."""
    import torch
    from paper_1412_0659_amd import Tree
    device()
    theta, eps = 0.6, 0.0
    rng = np.random.default_rng(98)
    ball = rng.normal(size=(far, 3))
    ball = 0.5 * ball / np.linalg.norm(ball, axis=1)[:, None] + [8.0, 5.0, 3.0]
    pos = np.concatenate([[[-0.5 * sep, 0.1, 0.2], [0.5 * sep, 0.1, 0.2]], ball]).astype(np.float32)
    n = far + 2
    mass = np.full(n, 2.0**-12, np.float32)
    u = np.tile(np.array([0.7, -0.4, 0.2], np.float32), (n, 1))
    t = Tree(n, nleaf=2, ncrit=2, adjoint=True)
    t.build(to_dev(pos), to_dev(mass))
    gp, gm = (torch.zeros(*sh, dtype=torch.float32, device="cuda") for sh in ((n, 3), (n,)))
    t.force_vjp(theta, eps, to_dev(u), 1.0, gp, gm)
    t.sync()
    gp = gp.cpu().numpy().astype(np.float64)
    t.close()
    ot = oracle.build_tree(pos, mass, 2, 2)
    g = int(np.flatnonzero(ot.perm[ot.gbeg] < 2)[0])
    d = oracle.record_decisions(ot, theta)
    assert ot.gcnt[g] == 2 and d.lf_off[g + 1] - d.lf_off[g] == 1  # its own leaf alone
    assert d.pc_off[g + 1] > d.pc_off[g]
    # the pair alone gives nothing (in exact arithmetic): the rest is the cells' part
    gx_ref, _ = oracle.frozen_force_vjp(d, pos, mass, eps, u)
    # size of the cells' terms, of both sides: (m / r^3) sum |u|, r = 8 to 11
    size = 2 * far * 2.0**-12 / 9.5**3
    err = np.abs(gp[:2] - gx_ref[:2]).max() / size
    print(f"far {far} sep {sep}: pair term {2.0**-12 / sep**3:.3g}, cells {size:.3g}, "
          f"error {err:.2e}", flush=True)
    assert err <= 1e-5
