"""The adjoint walk's branches against the oracle: groups of more targets than
the accumulator tiles hold (paired sets of up to 64, nleaf 64), more sources
than one list, and a target side whose sums are not finite."""
import numpy as np
import pytest

from gpu_util import device, paired_groups, rel_err, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


def _vjp(n, s, u, theta, eps, **kw):
    import torch
    from paper_1412_0659_amd import Tree
    device()
    t = Tree(n, adjoint=True, **kw)
    t.build(to_dev(s.pos), to_dev(s.mass))
    gp, gm = (torch.zeros(*sh, dtype=torch.float32, device="cuda") for sh in ((n, 3), (n,)))
    t.force_vjp(theta, eps, to_dev(u), 1.0, gp, gm)
    t.sync()
    t.close()
    return gp.cpu().numpy().astype(np.float64), gm.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("nleaf,ncrit,pairs", [(64, 64, 0), (16, 64, 64), (1, 5, 0), (16, 33, 0)])
def test_vjp_group_sizes(oracle, nleaf, ncrit, pairs):
    n, theta, eps = 6000, 0.5, 0.01
    s = ics.disk_halo_scaled(n, 75)
    u = np.random.default_rng(76).normal(size=(n, 3)).astype(np.float32)
    gp, gm = _vjp(n, s, u, theta, eps, nleaf=nleaf, ncrit=ncrit, pair_groups=pairs)
    ot = oracle.build_tree(s.pos, s.mass, nleaf, ncrit)
    if pairs:
        ot = paired_groups(oracle, ot, pairs)
    gx_ref, gm_ref = oracle.frozen_force_vjp(oracle.record_decisions(ot, theta), s.pos, s.mass,
                                             eps, u)
    ex, em = rel_err(gp, gx_ref), rel_err(gm, gm_ref)
    assert np.median(ex) <= 1e-5 and np.percentile(ex, 99) <= 1e-4
    assert np.median(em) <= 1e-5 and np.percentile(em, 99) <= 1e-4


def test_vjp_non_finite_pairs_stay_with_their_targets(oracle):
    """Two particles 1e-13 apart without softening: r^-5 overflows for that
    pair alone.  Every other particle of their group keeps its gradient."""
    n, theta = 40, 0.5
    rng = np.random.default_rng(77)
    pos = rng.normal(size=(n, 3)).astype(np.float32)
    pos[7] = 0.0
    pos[8] = (1e-13, 0.0, 0.0)
    s = ics.Snapshot(pos, np.zeros_like(pos), np.full(n, 1.0 / n, np.float32), np.zeros(n, bool))
    u = rng.normal(size=(n, 3)).astype(np.float32)
    gp, gm = _vjp(n, s, u, theta, 0.0)
    far = np.ones(n, bool)
    far[7:9] = False
    assert np.isfinite(gp[far]).all() and np.isfinite(gm[far]).all()
    d = pos[None, :, :].astype(np.float64) - pos[:, None, :]
    r2 = (d * d).sum(2)
    np.fill_diagonal(r2, 1.0)
    m = s.mass.astype(np.float64)
    ud = (u[:, None, :] * d).sum(2)
    w = m[None, :, None] * (u[:, None, :] / r2[:, :, None] ** 1.5
                            - 3 * (ud / r2 ** 2.5)[:, :, None] * d)
    w[np.arange(n), np.arange(n)] = 0.0
    ref = w.sum(0) - w.sum(1)
    assert rel_err(gp[far], ref[far]).max() <= 1e-4
