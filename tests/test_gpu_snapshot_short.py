"""Snapshots that the given allocation does not hold are refused with the HIP
error that their copies get; the context goes on working.  Snapshots inside a
captured graph are read and written by its replays."""
import ctypes

import numpy as np
import pytest

from gpu_util import device, to_dev
from workloads import ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pos_fp64", [False, True])
def test_short_allocation_is_refused(pos_fp64):
    import torch
    from paper_1412_0659_amd import Tree, binding as B
    device()
    n = 20001
    s = ics.plummer(n, 92)
    t = Tree(n, pos_fp64=pos_fp64, adjoint=True)
    t.set_state(to_dev(s.pos), to_dev(s.vel), to_dev(s.mass))
    full = t.save()
    t.sync()
    hip = ctypes.CDLL("libamdhip64.so.7")
    p, base, size = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(4096)) == 0
    assert hip.hipMemGetAddressRange(ctypes.byref(base), ctypes.byref(size), p) == 0
    # one field alone is larger than what is there
    assert base.value == p.value and size.value < 4 * n
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    lib = B.load()
    g = torch.zeros(n, 3, device="cuda")
    v = B._ptr(g)
    for name, args in (("bh_save_state", (p, stream)), ("bh_load_state", (p, n, stream)),
                       ("leapfrog_vjp_segment", (p, n, 2, 0, 1e-3, 0.5, 0.01, v, v, v, v, None,
                                                 stream))):
        print(name, flush=True)
        assert getattr(lib, name)(t.ctx, *args) == B.BH_EHIP
        assert hip.hipGetLastError() == 1  # (taken back: the next call would report it)
    t.restore(full, n)
    pos, vel = t.state()
    assert np.array_equal(pos.cpu().numpy(), s.pos) and np.array_equal(vel.cpu().numpy(), s.vel)
    t.close()
    assert hip.hipFree(p) == 0


def test_snapshots_in_a_graph():
    import torch
    from paper_1412_0659_amd import Tree, binding as B
    device()
    n = 3000
    s = ics.plummer(n, 93)
    t = Tree(n)
    t.set_state(to_dev(s.pos), to_dev(s.vel), to_dev(s.mass))
    start = t.save()
    t.step(1e-3, 0.5, 0.01)
    end = t.save()
    out = torch.zeros_like(end)
    t.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.bh_load_state(t.ctx, start, n)
        B.leapfrog_step(t.ctx, 1e-3, 0.5, 0.01)
        B.bh_save_state(t.ctx, out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        # the same particles in the same order: equal bytes
        assert torch.equal(out, end)
        t.step(1e-3, 0.5, 0.01)
        t.sync()
    t.close()
