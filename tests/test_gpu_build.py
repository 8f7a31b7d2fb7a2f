"""The octree build at the edges of its tiles of 1024 particles: cells that
start, end and lie across tiles, leaves and groups of every size the build
takes, coincident particles over several tiles; bit-exact with the oracle."""
import numpy as np
import pytest

from gpu_util import assert_tree_equal, gpu_tree
from workloads import ics

pytestmark = pytest.mark.gpu


def _points(kind, n):
    rng = np.random.default_rng(n)
    if kind == "plummer":
        return ics.plummer(n, 81).pos
    pos = rng.normal(size=(n, 3)).astype(np.float32)
    pos[n // 5:n // 5 + (2 * n) // 3] = pos[n // 5]  # coincident, over tile edges
    return pos


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2048, 2049, 5000])
@pytest.mark.parametrize("kind", ["plummer", "coincident"])
@pytest.mark.parametrize("nleaf,ncrit,curve", [(16, 64, "morton"), (1, 1, "ph"), (64, 7, "morton"),
                                               (3, 64, "ph")])
def test_build_at_tile_edges(oracle, n, kind, nleaf, ncrit, curve):
    pos = _points(kind, n)
    mass = np.full(n, 1.0 / n, np.float32)
    print(f"build {kind} n={n} nleaf={nleaf} ncrit={ncrit} {curve}", flush=True)
    t = gpu_tree(pos, mass, nleaf, ncrit, curve=curve)
    ot = oracle.build_tree(pos, mass, nleaf, ncrit, curve=curve)
    assert_tree_equal(t, ot)
    for arr in ("mom_M", "mom_com", "mom_Q"):
        assert np.array_equal(t.export(arr), ot.mom[arr[4:]])
    t.close()


def test_moments_of_more_spans_than_one_block_round():
    """More than 128 spans of 131072 particles (the top of the moment pass in
    rounds): every parent's count and moments follow from its children's, in
    child order, bit for bit, and the leaves' masses from their particles."""
    import torch
    from gpu_util import device
    from paper_1412_0659_amd import Tree
    n = 16_900_000
    g = torch.Generator(device=device())
    g.manual_seed(5)
    pos = torch.randn(n, 3, generator=g, device="cuda")
    mass = torch.rand(n, generator=g, device="cuda") + 0.5
    t = Tree(n)
    t.build(pos, mass)
    t.sync()
    nch = t.export("cell_nchild").astype(np.int64)
    cnt = t.export("cell_count").astype(np.int64)
    beg = t.export("cell_begin").astype(np.int64)
    ch0 = t.export("cell_child0").astype(np.int64)
    M, com, Q = t.export("mom_M"), t.export("mom_com"), t.export("mom_Q")
    perm = t.export("perm")
    t.close()
    assert cnt[0] == n and beg[0] == 0
    par = np.nonzero(nch)[0]
    sums = {"cnt": np.zeros(len(par), np.int64), "M": np.zeros(len(par)),
            "Q": np.zeros((len(par), 6))}
    pairs = ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))
    for k in range(8):
        has = nch[par] > k
        c = ch0[par[has]] + k
        sums["cnt"][has] += cnt[c]
        sums["M"][has] += M[c]
        d = com[c] - com[par[has]]
        for q, (i, j) in enumerate(pairs):
            sums["Q"][has, q] += Q[c, q] + (M[c] * d[:, i]) * d[:, j]
    assert np.array_equal(sums["cnt"], cnt[par])
    assert np.array_equal(sums["M"], M[par])
    assert np.array_equal(sums["Q"], Q[par])
    leaf = np.nonzero(nch == 0)[0]
    ms = np.concatenate([[0.0], np.cumsum(mass.cpu().numpy().astype(np.float64)[perm])])
    ref = ms[beg[leaf] + cnt[leaf]] - ms[beg[leaf]]
    assert np.allclose(M[leaf], ref, rtol=1e-7)  # (differences of 1e7-long running sums)
