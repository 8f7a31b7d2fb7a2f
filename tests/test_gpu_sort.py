"""The sort at the edges of its block tiles and merges, and on both sides of
the size where the radix passes take over: keys and the stable permutation
bit-exact, with many equal keys and in ascending and descending key order."""
import numpy as np
import pytest

from gpu_util import gpu_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385,
                               18432, 40000, 65537, 3 << 20, (3 << 20) + 1])
@pytest.mark.parametrize("kind", ["random", "equal", "descending"])
def test_sort_is_stable(oracle, n, kind):
    rng = np.random.default_rng(n)
    pos = rng.uniform(size=(n, 3)).astype(np.float32)
    if kind == "equal":  # eight distinct keys
        pos = np.round(pos).astype(np.float32)
    if kind == "descending":
        pos = np.sort(pos, axis=0)[::-1].copy()
    t = gpu_tree(pos, np.full(n, 1.0 / n, np.float32))
    keys, perm, box = t.export("keys"), t.export("perm").astype(np.int64), t.export("box")
    t.close()
    lo, side, scale = oracle.bbox(pos)
    assert np.array_equal(box[:3], lo) and box[3] == side and box[4] == scale
    ref = oracle.morton_keys(pos, lo, scale)
    order = np.argsort(ref, kind="stable")
    assert np.array_equal(perm, order) and np.array_equal(keys, ref[order])
