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


@pytest.mark.parametrize("storage", ["fp16", "bf16"])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("overlap", [0, 1])
def test_lanes_and_ring_2d_16bit(storage, form, overlap):
    """The 16-bit formats' march: lanes per workgroup, ring depth and segments."""
    w = W.capsule_at_interface(nx=301, ny=97, R=14.0, n_markers=100, wall_y=1)
    w["params"]["force_form"] = form
    ref = None
    for bx, ring, seg in ((0, 0, 0), (64, 3, 0), (64, 4, 5), (128, 3, 11), (128, 4, 0), (192, 3, 0), (192, 4, 9),
                          (256, 4, 0), (256, 4, 97)):
        g = run_gpu(w, storage)
        g.set_overlap(overlap)
        if bx:
            g.set_launch(block_x=bx, ring=ring, seg=seg)
        g.step(6)
        s = _state(g, 1)
        if ref is None:
            ref = s
        _same(s, ref, (bx, ring, seg))


@pytest.mark.parametrize("storage,tau", [("fp32", 0.85), ("fp64", 0.85), ("fp16", 1.0), ("bf16", 0.85)])
def test_tiles_3d_relaxing(storage, tau):
    """The relaxing step and the 16-bit formats: tiles of 16 x 16, 32 x 8 and
    64 x 4 nodes, and segments, with a capsule."""
    w = W.capsule3d(n=24, R=6.0, subdiv=2, two=False, bridge=False, r_cut=4.0, tau=tau)
    ref = None
    for tx, seg in ((0, 0), (16, 0), (32, 3), (64, 0), (64, 5), (16, 24)):
        g = run_gpu(w, storage)
        if tx:
            g.set_launch(block_x=tx, seg=seg)
        g.step(6)
        s = _state(g, 1)
        if ref is None:
            ref = s
        _same(s, ref, (tx, seg))
