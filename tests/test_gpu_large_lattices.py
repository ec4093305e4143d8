"""2D lattices whose populations exceed the last-level cache run the lattice
kernel in paced workgroups of several waves.  A periodic field repeated over
such a lattice evolves as the one period does on a small lattice, bit for bit:
strips and segments with remainders, walls, both force forms, relaxation times
of 1 and others, a batch of a large and a small member."""
import numpy as np
import pytest

from paper_1906_03065_amd import lbib
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


def _fluid(nx, ny, wall_y, tau, form):
    g = np.random.default_rng(5)
    p = W.base_params(nx, ny, wall_y=wall_y, kappa=(0.02, 0.03, 0.015), kappa_c=0.0, mobility=0.1, tau=tau)
    p.update(force_form=form, fext=[1e-6, -2e-6])
    c3, c1 = 0.3 * g.random((ny, nx)), 0.3 * g.random((ny, nx))
    f = W.fields_from_C(c1, 1.0 - c1 - c3, c3)
    f["u"] = [1e-3 * g.standard_normal((ny, nx)) for _ in range(2)]
    return dict(params=p, fields=f, membranes=[])


def _repeat(w, rx, ry):
    p = dict(w["params"], nx=rx * w["params"]["nx"], ny=ry * w["params"]["ny"])
    t = lambda a: np.tile(a, (ry, rx))
    f = w["fields"]
    return dict(params=p, membranes=[], fields=dict(rho=t(f["rho"]), phi=t(f["phi"]), psi=t(f["psi"]),
                                                    u=[t(a) for a in f["u"]]))


def _same(large, small, rx, ry):
    a, b = large.fields(), small.fields()
    for q in a:
        assert np.array_equal(a[q], np.tile(b[q], (ry, rx))), q


@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("tau", [1.0, 0.8])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("nx,ny,rx,ry,wall_y", [(275, 273, 4, 4, 0), (275, 273, 16, 1, 1)])
def test_repeated_field(nx, ny, rx, ry, wall_y, form, tau, storage):
    w = _fluid(nx, ny, wall_y, tau, form)
    a, b = lbib.from_workload(_repeat(w, rx, ry), storage=storage), lbib.from_workload(w, storage=storage)
    for n in (1, 1, 2):
        a.step(n)
        b.step(n)
    _same(a, b, rx, ry)
    a.set_launch(seg=11)
    for s in (a, b):
        s.step(1)
    _same(a, b, rx, ry)


@pytest.mark.parametrize("taus", [(1.0, 1.0), (0.8, 0.8), (1.0, 0.8)])
def test_batch_with_a_large_member(taus):
    ws = [_fluid(275, 273, 0, t, 1) for t in taus]
    b = lbib.Batch.from_workloads([_repeat(ws[0], 4, 4), ws[1]])
    s = [lbib.from_workload(w) for w in ws]
    for n in (1, 2, 4):
        b.step(n)
        for m in s:
            m.step(n)
    b.synchronize()
    _same(b[0], s[0], 4, 4)
    _same(b[1], s[1], 1, 1)


@pytest.mark.parametrize("tau", [1.0, 0.8])
def test_step_order(tau):
    """The overlapped step order: waves of a paced workgroup that leave for the
    second pass."""
    w = W.c2(n=1152, n_caps=4)
    w["params"]["tau"] = tau
    a, b = (lbib.from_workload(w) for _ in range(2))
    a.set_overlap(1)
    for n in (1, 1, 3):
        a.step(n)
        b.step(n)
    _same(a, b, 1, 1)
    for i in range(len(w["membranes"])):
        p, q = a.membrane(i), b.membrane(i)
        for k in p:
            assert np.array_equal(p[k], q[k]), (i, k)
    assert a.check() == b.check() == 0


def test_one_strip():
    """As large, but a single strip wide: waves on their own."""
    w = _fluid(57, 173, 0, 0.8, 1)
    a, b = lbib.from_workload(_repeat(w, 1, 121)), lbib.from_workload(w)
    for n in (1, 2):
        a.step(n)
        b.step(n)
    _same(a, b, 1, 121)
