"""Paired target sets that walk a local essential tree: their boxes reach over
two terminal cells, so they open cells that each terminal cell's box accepts
and that the tree keeps as leaves without particles.  Interaction counts
bit-exact and forces within the walk's tolerance (1e-5 median, 1e-4 99th
percentile) of the oracle's walk of the tree cut down the same way."""
import numpy as np
import pytest

from gpu_util import paired_groups, rel_err, to_dev
from test_gpu_let import LT, _disk, _oracle_domains

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,theta,max_cells", [(3, 0.7, 1024), (2, 0.9, 1024), (3, 0.7, 64)])
def test_paired_sets_walk_the_let(oracle, p, theta, max_cells):
    from paper_1412_0659_amd import Tree
    pos, mass = _disk(12000)
    eps = 0.01
    _, _, box, doms = _oracle_domains(oracle, pos, mass, p, "morton", theta, eps)
    trees, otrees = [], []
    for ix in doms:
        t = Tree(len(ix), pair_groups=64)
        t.set_box(*box)
        t.build(to_dev(pos[ix]), to_dev(mass[ix]))
        t.boundary(max_cells)
        trees.append(t)
        otrees.append(oracle.build_tree(pos[ix], mass[ix], box=box))
    bnd = [LT.boundary(ot, max_cells) for ot in otrees]
    empty = 0  # sets that open an empty leaf
    for a in range(p):
        own = paired_groups(oracle, otrees[a], 64)
        oacc, opot, onpp, onpc = oracle.walk(own, theta, eps)
        _, bc, bh = LT.boundary_boxes(otrees[a], bnd[a][2], box)
        for b in range(p):
            if b == a:
                continue
            vis, opn, ins = LT.let_mark(otrees[b], theta, bc, bh, bnd[b][2])
            cut = LT.prune(otrees[b], vis if ins else bnd[b][1],
                           opn if ins else bnd[b][1] & ~bnd[b][2])
            r = LT.walk_remote(own, otrees[b], theta, eps, cells=cut)
            whole = LT.walk_remote(own, otrees[b], theta, eps)
            empty += int(((whole[2] != r[2]) | (whole[3] != r[3])).sum())
            oacc, opot, onpp, onpc = oacc + r[0], opot + r[1], onpp + r[2], onpc + r[3]
        print(f"domain {a} of {p} theta={theta} cells={max_cells}", flush=True)
        trees[a].let_build([t for t in trees if t is not trees[a]], theta)
        acc, pot = trees[a].force_let(theta, eps)
        trees[a].sync()
        assert np.array_equal(trees[a].export("group_npp").astype(np.int64), onpp)
        assert np.array_equal(trees[a].export("group_npc").astype(np.int64), onpc)
        for got, ref in ((acc, oacc), (pot, opot)):
            e = rel_err(got.cpu().numpy(), ref)
            assert np.median(e) <= 1e-5 and np.percentile(e, 99) <= 1e-4
    assert empty > 0
    for t in trees:
        t.close()
