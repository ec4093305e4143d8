"""A 3D run with a non-finite marker, on meshes of one cluster of triangles and
of several, away from and at the antipode of the box, whether nodes keep their
closest triangle between steps (and renew it) or search every step: the
triangles that are left decide, and a repeated run gives the same bits."""
import numpy as np
import pytest

from helpers import run_gpu
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R,r_cut", [(28, 6.0, 4.0), (32, 6.0, 8.9)])
@pytest.mark.parametrize("subdiv", [0, 2])
@pytest.mark.parametrize("cache", [1, 0])
def test_nonfinite_marker(n, R, r_cut, subdiv, cache):
    w = W.capsule3d(n=n, R=R, subdiv=subdiv, two=False, bridge=False, r_cut=r_cut)
    a, b = run_gpu(w, "fp32"), run_gpu(w, "fp32")
    for s in (a, b):
        s.set_coupling_cache(cache)
        s.step(2)
        s.poke(2, 3 * 5 + 1, float("nan"))
    for k in (1, 2, 5):
        a.step(k)
        b.step(k)
        fa, fb = a.fields(), b.fields()
        ma, mb = a.membrane(0), b.membrane(0)
        for q in fa:
            assert np.isfinite(fa[q]).all() and np.array_equal(fa[q], fb[q]), (k, q)
        for q in ma:
            assert np.array_equal(ma[q], mb[q], equal_nan=True), (k, q)
        assert np.argwhere(~np.isfinite(ma["X"])).tolist() == [[5, 1]]
