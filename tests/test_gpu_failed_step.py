"""A step call that reports a HIP error between two of its steps (here one that
an invalid device number left behind on the host) leaves the state of the steps
that ran, as populations: it reads, checks, saves and steps on like the state
of a call that ended there."""
import ctypes

import numpy as np
import pytest

from paper_1906_03065_amd import lbib
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


def _fails(s, n):
    assert lbib.lib().hipSetDevice(ctypes.c_int(9999)) != 0
    with pytest.raises(lbib.LbibError) as e:
        s.step(n)
    assert e.value.code == lbib.EHIP


def _same(a, b, caps=1):
    fa, fb = a.fields(), b.fields()
    for q in fa:
        assert np.array_equal(fa[q], fb[q]), (q, float(np.abs(fa[q] - fb[q]).max()))
    for i in range(caps):
        ma, mb = a.membrane(i), b.membrane(i)
        for q in ma:
            assert np.array_equal(ma[q], mb[q]), q
    assert a.steps_done == b.steps_done
    assert a.energy() == b.energy()
    assert a.check() == b.check() == 0


@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("mw", [(1.0, 1.0, 1.0), (2.5, 1.0, 1.5)])
@pytest.mark.parametrize("dim,overlap", [(2, 0), (2, 1), (3, 0)])
def test_failed_call_leaves_populations(dim, overlap, storage, mw):
    if dim == 2:
        w = W.capsule_at_interface(nx=70, ny=61, R=12.0, n_markers=60, wall_y=1)
    else:
        w = W.drop3d(nx=37, ny=22, nz=25)
    caps = len(w["membranes"])
    phi, psi = w["fields"]["phi"], w["fields"]["psi"]
    w["params"]["mw"] = list(mw)
    w["fields"] = W.fields_from_C((1.0 - psi + phi) / 2, (1.0 - psi - phi) / 2, psi, mw=mw)
    a, b = (lbib.from_workload(w, storage=storage) for _ in range(2))
    if overlap:
        a.set_overlap(1)
    for s in (a, b):
        s.step(3)
    _fails(a, 5)
    assert 3 < a.steps_done < 8
    b.step(a.steps_done - 3)
    _same(a, b, caps)
    blob = a.save()
    a.step(4)
    b.step(4)
    _same(a, b, caps)
    a.load(blob)
    a.step(4)
    _same(a, b, caps)


@pytest.mark.parametrize("graph", [1, 0])
def test_failed_batch_call(graph):
    ws = [W.capsule_at_interface(nx=n, ny=60, R=12.0, n_markers=60) for n in (64, 75)]
    a, b = (lbib.Batch.from_workloads(ws) for _ in range(2))
    a.graph(graph)
    for s in (a, b):
        s.step(4)
    _fails(a, 5)
    b.step(a[0].steps_done - 4)
    for k in range(2):
        _same(a[k], b[k])
    a.step(3)
    b.step(3)
    for k in range(2):
        _same(a[k], b[k])
