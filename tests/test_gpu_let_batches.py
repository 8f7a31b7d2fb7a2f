"""Local essential trees of as many and more sources than one batch of their
construction holds (16): forces of all domains within the walk's tolerance of
the oracle's own and remote walks."""
import numpy as np
import pytest

from gpu_util import rel_err, to_dev
from test_gpu_let import LT, _disk, _oracle_domains

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [2, 17, 18, 34])
def test_domains_in_batches(oracle, p):
    import torch
    from paper_1412_0659_amd import Domains
    pos, mass = _disk(9000)
    theta, eps = 0.6, 0.01
    d = Domains(to_dev(pos), to_dev(mass), p, theta, eps, max_boundary=64)
    for _ in range(2):  # a second construction in the buffers of the first
        info = d.build_lets()
        acc, pot = d.forces()
        torch.cuda.synchronize()
    _, cuts, box, doms = _oracle_domains(oracle, pos, mass, p, "morton", theta, eps)
    assert np.array_equal(d.cuts, cuts) and len(info) == p
    oacc, opot, _ = LT.domain_forces(pos, mass, doms, box, theta, eps, "morton")
    ea, ep = rel_err(acc.cpu().numpy(), oacc), rel_err(pot.cpu().numpy(), opot)
    assert np.median(ea) <= 1e-5 and np.percentile(ea, 99) <= 1e-4
    assert np.median(ep) <= 1e-5 and np.percentile(ep, 99) <= 1e-4
    d.close()
