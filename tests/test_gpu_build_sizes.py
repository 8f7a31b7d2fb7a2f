"""The octree build and the moment pass at the sizes where the threads of a
tile change (262144, 524288 and 4194304 particles): cells that follow from the
sorted keys, moments that follow from the children's, bit for bit."""
import numpy as np
import pytest

from gpu_util import assert_tree_equal, gpu_tree
from workloads import ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,curve", [(262144, "morton"), (262145, "ph"), (524288, "ph"),
                                     (524289, "morton")])
def test_build_where_the_threads_change(oracle, n, curve):
    s = ics.disk_halo_scaled(n, 91)
    print(f"build n={n} {curve}", flush=True)
    t = gpu_tree(s.pos, s.mass, curve=curve)
    ot = oracle.build_tree(s.pos, s.mass, curve=curve)
    assert_tree_equal(t, ot)
    for arr in ("mom_M", "mom_com", "mom_Q"):
        assert np.array_equal(t.export(arr), ot.mom[arr[4:]])
    t.close()


@pytest.mark.parametrize("n", [4194304, 4194305])
def test_parents_of_large_sets(n):
    import torch
    from gpu_util import device
    from paper_1412_0659_amd import Tree
    g = torch.Generator(device=device())
    g.manual_seed(7)
    pos = torch.randn(n, 3, generator=g, device="cuda")
    mass = torch.rand(n, generator=g, device="cuda") + 0.5
    print(f"build n={n}", flush=True)
    t = Tree(n)
    t.build(pos, mass)
    t.sync()
    nch, cnt, beg, ch0 = (t.export("cell_" + k).astype(np.int64)
                          for k in ("nchild", "count", "begin", "child0"))
    M, com, Q = t.export("mom_M"), t.export("mom_com"), t.export("mom_Q")
    t.close()
    assert cnt[0] == n and beg[0] == 0 and np.all(cnt[nch == 0] <= 16)
    par = np.flatnonzero(nch)
    m, c = np.zeros(len(par)), np.zeros(len(par), np.int64)
    for k in range(8):  # children in order
        on = nch[par] > k
        j = ch0[par[on]] + k
        assert np.array_equal(beg[j], beg[par[on]] + c[on])
        m[on] += M[j]
        c[on] += cnt[j]
    assert np.array_equal(c, cnt[par]) and np.array_equal(m, M[par])
    q = np.zeros((len(par), 6))
    for k in range(8):
        on = nch[par] > k
        j = ch0[par[on]] + k
        d = com[j] - com[par[on]]
        md = M[j][:, None] * d
        q[on] += Q[j] + np.stack([md[:, 0] * d[:, 0], md[:, 1] * d[:, 1], md[:, 2] * d[:, 2],
                                  md[:, 0] * d[:, 1], md[:, 0] * d[:, 2], md[:, 1] * d[:, 2]], 1)
    assert np.array_equal(q, Q[par])
