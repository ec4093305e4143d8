"""Membrane energies of very many markers over a few nodes: the sums' workspace
goes by the nodes.  A uniformly stretched ring against its closed form: 1e-10
relative, since a segment's length is a difference of coordinates 1e5 times
larger, each rounded to 2^-53."""
import numpy as np
import pytest

from paper_1906_03065_amd import lbib
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n", [(4, 1, 140000), (2, 2, 66000), (64, 64, 9000)])
def test_strain_energy_of_many_markers(nx, ny, n):
    ks, lam = 0.05, 1.25
    X = W.circle_markers(nx / 2.0, ny / 2.0, 0.4, n)
    p = W.base_params(nx, ny, wall_y=0, kappa_c=0.0, mobility=0.1, r_cut=1.0)
    one = np.ones((ny, nx))
    length = np.hypot(*(np.roll(X, -1, axis=0) - X).T)
    w = dict(params=p, fields=W.fields_from_C(one, 0.0 * one, 0.0 * one),
             membranes=[dict(X=X, tris=None, kappa_s=ks, kappa_b=0.0, rest=length / lam)])
    s = lbib.from_workload(w, storage="fp32")
    want = 0.5 * ks * (lam - 1.0) ** 2 * length.sum() / lam
    for _ in range(3):
        e = s.energy()
        assert abs(e["E_s"] - want) < 1e-10 * want
        assert abs(e["mass"][0] - nx * ny) < 1e-12 * nx * ny
