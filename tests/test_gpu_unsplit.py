"""Walks of sets of more than 2^20 particles, one wave per group: what the
smaller sets' tests check of the shared walks, here of the kernel that
finishes its targets itself.  Counts bit-exact and forces within the walk's
tolerance (1e-5 median, 1e-4 99th percentile) of the oracle at seeded groups."""
import numpy as np
import pytest

from gpu_util import gpu_force, paired_groups, rel_err, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu

N = (1 << 20) + 1


@pytest.fixture(scope="module")
def snap():
    return ics.plummer(N, 101)


@pytest.fixture(scope="module")
def tree(oracle, snap):
    return oracle.build_tree(snap.pos, snap.mass)


def _check(oracle, ot, t, acc, pot, theta, eps, seed):
    rng = np.random.default_rng(seed)
    sel = np.sort(rng.choice(ot.ngroups, size=1500, replace=False))
    oacc, opot, onpp, onpc = oracle.walk(ot, theta, eps, groups=sel)
    npp, npc = t.export("group_npp").astype(np.int64), t.export("group_npc").astype(np.int64)
    assert np.array_equal(npp[sel], onpp[sel]) and np.array_equal(npc[sel], onpc[sel])
    st = t.stats()
    assert st["n_pp"] == int((npp * ot.gcnt).sum()) and st["n_pc"] == int((npc * ot.gcnt).sum())
    tgt = np.concatenate([ot.perm[ot.gbeg[g]:ot.gbeg[g] + ot.gcnt[g]] for g in sel])
    for a, b in ((acc, oacc), (pot, opot)):
        e = rel_err(a[tgt], b[tgt])
        assert np.median(e) <= 1e-5 and np.percentile(e, 99) <= 1e-4


@pytest.mark.parametrize("eps,pairs", [(0.0, 0), (0.01, 64)])
def test_no_softening_and_paired_sets(oracle, snap, tree, eps, pairs):
    from paper_1412_0659_amd import Tree
    print(f"unsplit eps={eps} pairs={pairs}", flush=True)
    t = Tree(N, pair_groups=pairs)
    t.build(to_dev(snap.pos), to_dev(snap.mass))
    acc, pot = gpu_force(t, 0.7, eps)
    _check(oracle, paired_groups(oracle, tree, pairs) if pairs else tree, t, acc, pot, 0.7, eps, 102)
    t.close()


def test_spill_and_refill(oracle, monkeypatch):
    """One particle per leaf and the walk stack's LDS window cut to 192
    ranges: a uniform ball at a small angle spills from it."""
    from paper_1412_0659_amd import Tree
    monkeypatch.setenv("BH_WALK_SMALL_STACK", "1")
    rng = np.random.default_rng(103)
    pos = rng.uniform(-1, 1, (N, 3)).astype(np.float32)
    mass = np.full(N, 1.0 / N, np.float32)
    print("unsplit spill", flush=True)
    t = Tree(N, nleaf=1)
    t.build(to_dev(pos), to_dev(mass))
    acc, pot = gpu_force(t, 0.3, 1e-3)
    _check(oracle, oracle.build_tree(pos, mass, 1, 64), t, acc, pot, 0.3, 1e-3, 104)
    t.close()


@pytest.mark.parametrize("pos_fp64", [False, True])
def test_step(snap, pos_fp64):
    """A step, its last kick made by the walk, against the same step taken
    apart: force, kick and drift on the host in FP64 rounded to FP32 once (as
    the library's fused multiply-adds round), force of the drifted set, kick."""
    import torch
    from paper_1412_0659_amd import Tree
    theta, eps, dt = 0.7, 0.01, 1e-3
    h = np.float32(0.5 * np.float32(dt))
    f32 = np.float32
    pos, mass = to_dev(snap.pos), to_dev(snap.mass)
    print(f"unsplit step pos_fp64={pos_fp64}", flush=True)
    t = Tree(N, pos_fp64=pos_fp64)
    t.set_state(pos, to_dev(snap.vel), mass)
    t.step(dt, theta, eps)
    p, v = (x.cpu().numpy() for x in t.state())
    st = t.stats()
    assert st["n_pp"] > 0 and st["n_pc"] > 0
    t.close()
    w = Tree(N)
    w.build(pos, mass)
    a0, _ = gpu_force(w, theta, eps)
    v1 = (a0 * h.astype(np.float64) + snap.vel).astype(f32)
    x1 = (v1.astype(np.float64) * f32(dt).astype(np.float64) + snap.pos).astype(f32)
    assert np.array_equal(p, x1)
    w.build(to_dev(x1), mass)
    a1, _ = gpu_force(w, theta, eps)
    assert w.stats()["n_pp"] == st["n_pp"] and w.stats()["n_pc"] == st["n_pc"]
    w.close()
    v2 = (a1 * h.astype(np.float64) + v1).astype(f32)
    # equal but for the order of particles of equal keys (FP32 sums of their group)
    assert np.abs(v - v2).max() <= 1e-5 * np.abs(a1).max() * h + 2.0**-23 * np.abs(v2).max()
    assert (v == v2).all(1).mean() > 0.99
