"""Batches in which some members relax and others do not (one lattice launch for
both): every member bitwise equal to its single run, in calls of any length."""
import numpy as np
import pytest

from paper_1906_03065_amd import lbib
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("graph", [1, 0])
@pytest.mark.parametrize("taus", [(1.0, 0.8, 1.0, 1.3), (0.9, 1.0, 0.9, 0.9)])
def test_mixed_members(taus, graph, form):
    ws = [W.capsule_at_interface(nx=n, ny=60 + 7 * i, R=12.0, n_markers=70, tau=t, seed=i, wall_y=i % 2)
          for i, (n, t) in enumerate(zip((64, 131, 75, 260), taus))]
    for w in ws:
        w["params"]["force_form"] = form
    b = lbib.Batch.from_workloads(ws)
    b.graph(graph)
    s = [lbib.from_workload(w) for w in ws]
    for n in (1, 2, 5):
        b.step(n)
        for m in s:
            m.step(n)
    b.synchronize()
    assert b.graph() == graph
    for k, m in enumerate(s):
        assert b[k].check() == m.check()  # (the band of some is as wide as their period)
        fa, fb = b[k].fields(), m.fields()
        for q in fa:
            assert np.array_equal(fa[q], fb[q]), (k, q)
        ma, mb = b[k].membrane(0), m.membrane(0)
        for q in ma:
            assert np.array_equal(ma[q], mb[q]), (k, q)
