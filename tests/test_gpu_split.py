"""Walks whose groups are shared by 8, 4 or 2 waves (small sets), at the
sizes where the number of waves changes: interaction counts bit-exact and
forces within the walk's tolerance (1e-5 median, 1e-4 99th percentile) of the
oracle; a tree too small to be dealt out by ranges; run to run identical."""
import numpy as np
import pytest

from gpu_util import gpu_force, gpu_tree, rel_err, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 70, 700, 4096, 4097, 40960, 40961, 147457])
def test_split_walk_matches_oracle(oracle, n):
    theta, eps = 0.55, 0.01
    s = ics.plummer(n, 71) if n != 40960 else ics.disk_halo_scaled(n, 72)
    print(f"split walk n={n}", flush=True)
    t = gpu_tree(s.pos, s.mass)
    acc, pot = gpu_force(t, theta, eps)
    npp, npc = t.export("group_npp").astype(np.int64), t.export("group_npc").astype(np.int64)
    acc2, pot2 = gpu_force(t, theta, eps)
    assert np.array_equal(acc, acc2) and np.array_equal(pot, pot2)
    st = t.stats()
    t.close()
    ot = oracle.build_tree(s.pos, s.mass)
    oacc, opot, onpp, onpc = oracle.walk(ot, theta, eps)
    assert np.array_equal(npp, onpp) and np.array_equal(npc, onpc)
    assert st["n_pp"] == int((onpp * ot.gcnt).sum()) and st["n_pc"] == int((onpc * ot.gcnt).sum())
    ea, ep = rel_err(acc, oacc), rel_err(pot, opot)
    assert np.median(ea) <= 1e-5 and np.percentile(ea, 99) <= 1e-4
    assert np.median(ep) <= 1e-5 and np.percentile(ep, 99) <= 1e-4


@pytest.mark.parametrize("n", [300, 8193, 24577])
def test_split_vjp_matches_oracle(oracle, n):
    import torch
    from paper_1412_0659_amd import Tree
    theta, eps = 0.6, 0.01
    s = ics.plummer(n, 73)
    u = np.random.default_rng(74).normal(size=(n, 3)).astype(np.float32)
    print(f"split vjp n={n}", flush=True)
    t = Tree(n, adjoint=True)
    t.build(to_dev(s.pos), to_dev(s.mass))
    gp, gm = (torch.zeros(*sh, dtype=torch.float32, device="cuda") for sh in ((n, 3), (n,)))
    t.force_vjp(theta, eps, to_dev(u), 1.0, gp, gm)
    t.sync()
    gp, gm = gp.cpu().numpy().astype(np.float64), gm.cpu().numpy().astype(np.float64)
    t.close()
    d = oracle.record_decisions(oracle.build_tree(s.pos, s.mass), theta)
    gx_ref, gm_ref = oracle.frozen_force_vjp(d, s.pos, s.mass, eps, u)
    ex, em = rel_err(gp, gx_ref), rel_err(gm, gm_ref)
    assert np.median(ex) <= 1e-5 and np.percentile(ex, 99) <= 1e-4
    assert np.median(em) <= 1e-5 and np.percentile(em, 99) <= 1e-4
