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
