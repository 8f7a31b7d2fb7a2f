"""Walks whose groups are shared by a number of waves that depends on the
group's size: the sizes where that rule changes, groups of 1 to 64 targets,
groups of one size only.  Interaction counts bit-exact, forces within the
walk's tolerance (1e-5 median, 1e-4 99th percentile) of the oracle, run to run
identical; adjoint likewise."""
import numpy as np
import pytest

from gpu_util import gpu_force, gpu_tree, rel_err, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


def _same(a, b):
    e = rel_err(a, b)
    assert np.median(e) <= 1e-5 and np.percentile(e, 99) <= 1e-4


@pytest.mark.parametrize("n,ncrit", [(8192, 64), (8193, 64), (20480, 64), (20481, 64), (262144, 64),
                                     (262145, 64), (9000, 16), (9000, 1), (30000, 33)])
def test_walk(oracle, n, ncrit):
    theta, eps = 0.7, 0.01
    s = ics.plummer(n, 81)
    print(f"walk n={n} ncrit={ncrit}", flush=True)
    t = gpu_tree(s.pos, s.mass, ncrit=ncrit)
    acc, pot = gpu_force(t, theta, eps)
    npp, npc = t.export("group_npp").astype(np.int64), t.export("group_npc").astype(np.int64)
    cnt = t.export("group_count")
    acc2, pot2 = gpu_force(t, theta, eps)
    assert np.array_equal(acc, acc2) and np.array_equal(pot, pot2)
    st = t.stats()
    t.close()
    if ncrit == 64 and n > 20000:
        assert cnt.min() == 1 and cnt.max() >= 63
    ot = oracle.build_tree(s.pos, s.mass, ncrit=ncrit)
    oacc, opot, onpp, onpc = oracle.walk(ot, theta, eps)
    assert np.array_equal(npp, onpp) and np.array_equal(npc, onpc)
    assert st["n_pp"] == int((onpp * ot.gcnt).sum()) and st["n_pc"] == int((onpc * ot.gcnt).sum())
    _same(acc, oacc)
    _same(pot, opot)


@pytest.mark.parametrize("kind", ["plummer", "coincident", "pairs"])
@pytest.mark.parametrize("n", [1, 2, 16, 17, 18, 65, 400])
def test_first_pass_of_few_levels(oracle, n, kind):
    """Trees of one, two and more levels, chains of single cells down to the
    last level: the pass that takes the levels 0 to 2 together."""
    s = ics.plummer(max(n, 2), 87)
    pos, mass = s.pos[:n].copy(), s.mass[:n].copy()
    if kind == "coincident":
        pos[:] = pos[0]
    elif kind == "pairs":
        pos[1::2] = pos[0]
    for nleaf, theta in ((16, 0.5), (1, 1.0)):
        print(f"{kind} n={n} nleaf={nleaf}", flush=True)
        t = gpu_tree(pos, mass, nleaf)
        acc, pot = gpu_force(t, theta, 0.05)
        npp, npc = t.export("group_npp").astype(np.int64), t.export("group_npc").astype(np.int64)
        t.close()
        oacc, opot, onpp, onpc = oracle.walk(oracle.build_tree(pos, mass, nleaf), theta, 0.05)
        assert np.array_equal(npp, onpp) and np.array_equal(npc, onpc)
        scale = max(np.abs(oacc).max(), 1e-30)
        assert np.abs(acc - oacc).max() <= 1e-5 * scale + 1e-6
        if n > 1:
            assert np.percentile(rel_err(pot, opot), 99) <= 1e-4


@pytest.mark.parametrize("n", [2048, 2049, 32768, 32769])
def test_vjp(oracle, n):
    import torch
    from paper_1412_0659_amd import Tree
    theta, eps = 0.8, 0.01
    s = ics.plummer(n, 83)
    u = np.random.default_rng(84).normal(size=(n, 3)).astype(np.float32)
    print(f"vjp n={n}", flush=True)
    t = Tree(n, adjoint=True)
    t.build(to_dev(s.pos), to_dev(s.mass))
    gp, gm = (torch.zeros(*sh, dtype=torch.float32, device="cuda") for sh in ((n, 3), (n,)))
    t.force_vjp(theta, eps, to_dev(u), 1.0, gp, gm)
    t.sync()
    gp, gm = gp.cpu().numpy().astype(np.float64), gm.cpu().numpy().astype(np.float64)
    t.close()
    d = oracle.record_decisions(oracle.build_tree(s.pos, s.mass), theta)
    gx_ref, gm_ref = oracle.frozen_force_vjp(d, s.pos, s.mass, eps, u)
    _same(gp, gx_ref)
    _same(gm, gm_ref)


@pytest.mark.parametrize("n", [360448, 360449, 1048576, 1048577])
def test_sizes_agree_with_their_neighbours(n):
    """Particle n - 1 is far away and of no weight: the sets of n and n - 1
    particles on either side of a line have the same forces on the others,
    and the same gradients, to FP32 rounding."""
    import torch
    from paper_1412_0659_amd import Tree
    theta, eps, m = 0.9, 0.01, n - 2
    s = ics.plummer(m, 85)
    far = np.array([[40.0, 40.0, 40.0], [-40.0, -40.0, -40.0], [40.0, -40.0, 40.0]], np.float32)
    u = np.random.default_rng(86).normal(size=(m + 3, 3)).astype(np.float32)
    u[m:] = 0.0
    out = []
    for k in (2, 3):
        pos = np.concatenate([s.pos, far[:k]]).astype(np.float32)
        mass = np.concatenate([s.mass, np.full(k, 1e-30)]).astype(np.float32)
        print(f"n={m + k}", flush=True)
        t = Tree(m + k, adjoint=True)
        t.build(to_dev(pos), to_dev(mass))
        acc, pot = t.force(theta, eps)
        gp, gm = (torch.zeros(*sh, dtype=torch.float32, device="cuda")
                  for sh in ((m + k, 3), (m + k,)))
        t.force_vjp(theta, eps, to_dev(u[:m + k]), 1.0, gp, gm)
        t.sync()
        out.append([x[:m].cpu().numpy().astype(np.float64) for x in (acc, pot, gp, gm)])
        t.close()
    for a, b in zip(*out):
        _same(a, b)
