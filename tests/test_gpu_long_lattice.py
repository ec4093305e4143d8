"""A very long 3D lattice: enqueueing a step costs the host what its launches
cost (three, a few microseconds each), not a search over its planes."""
import time

import numpy as np
import pytest

from paper_1906_03065_amd import lbib
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_host_time_of_a_step():
    import torch

    nz = 60000
    p = W.base_params(2, 1, nz, lattice=1, kappa_c=0.0, mobility=0.1)
    one = np.ones((nz, 1, 2))
    s = lbib.from_workload(dict(params=p, fields=W.fields_from_C(one, 0.0 * one, 0.0 * one), membranes=[]))
    s.step(4)
    best = 1.0
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        s.step(4)
        best = min(best, (time.perf_counter() - t) / 4)
    torch.cuda.synchronize()
    assert best < 80e-6, best
    assert s.check() == 0
