"""The adjoint walk's target side where a flush's sums are not all finite,
for groups of at most 32 targets (their lists are taken again from the start)
and of more (chunk by chunk), in the particle and in the cell list, each of
several chunks per wave: the other targets of the group keep their gradients."""
import numpy as np
import pytest

from gpu_util import rel_err
from test_gpu_vjp_forms import _vjp
from workloads import ics

pytestmark = pytest.mark.gpu


def _snap(pos):
    n = len(pos)
    return ics.Snapshot(pos, np.zeros_like(pos), np.full(n, 1.0 / n, np.float32), np.zeros(n, bool))


@pytest.mark.parametrize("ncrit", [24, 64])
def test_particle_list(oracle, ncrit):
    """Two particles 1e-13 apart without softening: r^-5 overflows for that
    pair alone."""
    n, theta = 1300, 1e-3
    rng = np.random.default_rng(78)
    pos = rng.normal(size=(n, 3)).astype(np.float32)
    pos[7] = 0.0
    pos[8] = (1e-13, 0.0, 0.0)
    s = _snap(pos)
    u = rng.normal(size=(n, 3)).astype(np.float32)
    ot = oracle.build_tree(pos, s.mass, 16, ncrit)
    g = np.searchsorted(ot.gbeg, np.flatnonzero(ot.perm == 7)[0], "right") - 1
    d = oracle.record_decisions(ot, theta)
    assert (3 < ot.gcnt[g] <= 32) if ncrit == 24 else ot.gcnt[g] > 32
    assert d.pc_off[g + 1] == d.pc_off[g]  # all 1300 particles are listed, 160 per wave
    print(f"particle list, group of {ot.gcnt[g]}", flush=True)
    gp, gm = _vjp(n, s, u, theta, 0.0, ncrit=ncrit)
    far = np.ones(n, bool)
    far[7:9] = False
    assert np.isfinite(gp[far]).all() and np.isfinite(gm[far]).all()
    assert not np.isfinite(gp[7:9]).all()
    x = pos.astype(np.float64)
    ref = np.zeros((n, 3))
    gmr = np.zeros(n)
    m = 1.0 / n
    for i in range(n):  # target i
        dd = x - x[i]
        r2 = (dd * dd).sum(1)
        r2[i] = 1.0
        ud = dd @ u[i].astype(np.float64)
        w = m * (u[i] / r2[:, None] ** 1.5 - 3 * (ud / r2**2.5)[:, None] * dd)
        w[i] = 0.0
        ref += w
        ref[i] -= w.sum(0)
        gmr += ud / r2**1.5
    e, em = rel_err(gp[far], ref[far]), rel_err(gm[far], gmr[far])
    assert np.median(e) <= 1e-5 and np.percentile(e, 99) <= 1e-4
    assert np.median(em) <= 1e-5 and np.percentile(em, 99) <= 1e-4


@pytest.mark.parametrize("k,ncrit", [(20, 24), (44, 56)])
def test_cell_list(oracle, k, ncrit):
    """A target 2.8e-6 from a cell of two coincident particles without
    softening: r^-7 overflows for that pair of target and cell alone."""
    theta = 0.25
    rng = np.random.default_rng(79)
    gap = 1.4e-6
    near = np.concatenate([[[0.5 - gap, 0.3, 0.3]], np.tile([0.5 + gap, 0.3, 0.3], (2, 1)),
                           rng.uniform([0.4, 0.26, 0.26], [0.499, 0.36, 0.36], (k - 1, 3)),
                           [[0.0, 0.0, 0.0], [1.0, 1.0, 1.0]]])
    b = rng.uniform(0, 1, (6000, 3))
    b = b[~((b > [0.3, 0.2, 0.2]) & (b < 0.5)).all(1)]
    pos = np.concatenate([near, b]).astype(np.float32)
    n = len(pos)
    s = _snap(pos)
    u = rng.normal(size=(n, 3)).astype(np.float32)
    ot = oracle.build_tree(pos, s.mass, 1, ncrit)
    slot = np.empty(n, np.int64)
    slot[ot.perm] = np.arange(n)
    g = np.searchsorted(ot.gbeg, slot[0], "right") - 1
    d = oracle.record_decisions(ot, theta)
    pc = d.pc[d.pc_off[g]:d.pc_off[g + 1]]
    c = ot.cells
    pair = [i for i in pc if c["begin"][i] <= slot[1] < c["begin"][i] + c["count"][i]]
    assert len(pair) == 1 and c["count"][pair[0]] == 2
    assert (3 < ot.gcnt[g] <= 32) if k == 20 else ot.gcnt[g] > 32
    assert len(pc) >= 16 * 96  # (up to 16 waves share the list)
    print(f"cell list, group of {ot.gcnt[g]}, {len(pc)} cells", flush=True)
    gp, gm = _vjp(n, s, u, theta, 0.0, nleaf=1, ncrit=ncrit)
    far = np.ones(n, bool)
    far[:3] = False
    assert np.isfinite(gp[far]).all() and np.isfinite(gm[far]).all()
    assert not np.isfinite(gp[0]).all()
    gx_ref, gm_ref = oracle.frozen_force_vjp(d, pos, s.mass, 0.0, u)
    mine = np.zeros(n, bool)
    mine[ot.perm[ot.gbeg[g]:ot.gbeg[g] + ot.gcnt[g]]] = True
    for got, ref in ((gp, gx_ref), (gm, gm_ref)):
        e = rel_err(got[far], ref[far])
        assert np.median(e) <= 1e-5 and np.percentile(e, 99) <= 1e-4
        # the group's own targets, each against at least their median gradient
        a, r = got[far & mine].reshape(-1, ref[0].size), ref[far & mine].reshape(-1, ref[0].size)
        size = np.linalg.norm(r, axis=1)
        e = np.linalg.norm(a - r, axis=1) / np.maximum(size, np.median(size))
        assert e.max() <= 1e-4
