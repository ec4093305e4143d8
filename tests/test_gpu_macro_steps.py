"""Steps inside a call of several pass on a node's macroscopic numbers instead
of its populations when every relaxation time is 1.  The populations are the
same numbers either way, so any division of the same steps into calls leaves
the same bits: one call of n steps against n calls of one, which keep to
populations throughout, on lattices whose strips and segments have tails, that
are thinner than a strip's or a segment's halo, with walls and periodic."""
import numpy as np
import pytest

from paper_1906_03065_amd import lbib
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


def _fluid(nx, ny, wall, form, mw=(1.0, 1.0, 1.0)):
    g = np.random.default_rng(nx * 1000 + ny)
    p = W.base_params(nx, ny, wall_y=wall, kappa=(0.02, 0.03, 0.015), kappa_c=0.0, mobility=0.1, force_form=form)
    p["mw"] = list(mw)
    p["fext"] = [1e-6, -2e-6]
    c3, c1 = 0.3 * g.random((ny, nx)), 0.3 * g.random((ny, nx))
    f = W.fields_from_C(c1, 1.0 - c1 - c3, c3, mw=mw)
    f["u"] = [1e-3 * g.standard_normal((ny, nx)) for _ in range(2)]
    return dict(params=p, fields=f, membranes=[])


def _state(s, caps):
    f = s.fields()
    out = [f[k] for k in ("rho", "c1", "c2", "c3", "ux", "uy")]
    for i in range(caps):
        m = s.membrane(i)
        out += [m["X"], m["U"], m["F"]]
    return out


def _same(a, b):
    for u, v in zip(a, b):
        assert np.array_equal(u, v), float(np.abs(u - v).max())


@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,wall,form", [(64, 48, 1, 1), (59, 37, 0, 0), (117, 3, 1, 1), (58, 4, 1, 0), (61, 2, 1, 1),
                                             (5, 7, 0, 1), (1, 9, 1, 1), (175, 1, 0, 1)])
def test_calls_divide_alike(nx, ny, wall, form, storage):
    w = _fluid(nx, ny, wall, form)
    a, b = (lbib.from_workload(w, storage=storage) for _ in range(2))
    a.step(7)
    for _ in range(7):
        b.step(1)
    _same(_state(a, 0), _state(b, 0))
    a.step(2)
    b.step(1)
    b.step(1)
    _same(_state(a, 0), _state(b, 0))


@pytest.mark.parametrize("mw", [(1.0, 1.0, 1.0), (2.5, 1.0, 1.5)])
@pytest.mark.parametrize("wall,storage", [(1, "fp32"), (0, "fp64")])
def test_calls_divide_alike_with_a_capsule(wall, storage, mw):
    w = W.capsule_at_interface(nx=123, ny=90, R=15.0, n_markers=118, wall_y=wall, centre=(61.3, 44.2), seed=3, mw=mw)
    w["params"]["force_form"] = 1
    runs = []
    for calls in ((12,), (1,) * 12, (5, 1, 2, 4)):
        s = lbib.from_workload(w, storage=storage)
        for seg, n in zip((0, 5, 9, 40) * 3, calls):
            s.set_launch(seg=seg)
            s.step(n)
        assert s.check() == 0
        runs.append(_state(s, 1))
    _same(runs[0], runs[1])
    _same(runs[0], runs[2])


def test_batch_calls_divide_alike():
    """Members that relax keep the whole batch on populations."""
    ws = [W.capsule_at_interface(nx=96, ny=88, R=14.0, n_markers=110, seed=31),
          W.capsule_at_interface(nx=200, ny=72, R=12.5, n_markers=98, seed=32)]
    relaxing = W.capsule_at_interface(nx=130, ny=64, R=11.0, n_markers=88, tau=0.8, seed=33)
    for graph in (1, 0):
        singles = [lbib.from_workload(w) for w in ws]
        for s in singles:
            for _ in range(9):
                s.step(1)
        for more in ([], [relaxing]):
            b = lbib.Batch.from_workloads(ws + more)
            b.graph(graph)
            b.step(6)
            b.step(1)
            b.step(2)
            b.synchronize()
            for s, m in zip(singles, b.members):
                _same(_state(s, 1), _state(m, 1))
