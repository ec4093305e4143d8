"""The launch shape is a tuning knob: segments, tiles and step order leave every
bit of the results alone."""
import numpy as np
import pytest

from helpers import run_gpu
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


def _state(g, caps):
    return [g.fields()] + [g.membrane(i) for i in range(caps)]


def _same(a, b, what):
    for p, q in zip(a, b):
        for k in p:
            assert np.array_equal(p[k], q[k]), (what, k, float(np.abs(p[k] - q[k]).max()))


@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("caps", [0, 1])
@pytest.mark.parametrize("calls", [(1,), (4,)])
def test_segments_3d(storage, caps, calls):
    """The step with every relaxation time 1, from and to populations and inside
    a call: segments of one plane, of a few and of all."""
    if caps:
        w = W.capsule3d(n=24, R=6.0, subdiv=2, two=False, bridge=False, r_cut=4.0)
    else:
        w = W.drop3d(nx=37, ny=22, nz=25, wall_z=0)
        for q in ("tau", "tau_phi", "tau_psi"):
            w["params"][q] = 1.0
    ref = None
    for seg in (0, 1, 3, 7, 100):
        g = run_gpu(w, storage)
        if seg:
            g.set_launch(seg=seg)
        for n in calls:
            g.step(n)
        s = _state(g, caps)
        if ref is None:
            ref = s
        _same(s, ref, seg)
