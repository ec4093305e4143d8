"""D3Q19 with every relaxation time 1: the steps inside a call pass on a node's
macroscopic numbers instead of its populations.  The populations are the same
numbers either way, so any division of the same steps into calls leaves the same
bits: lattices with tails of strips, tiles and segments in every direction,
thinner than a strip's or a tile's halo, wide enough for the wide tile, with
walls in y, in z, in both and in none."""
import numpy as np
import pytest

from paper_1906_03065_amd import lbib
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


def _fluid(nx, ny, nz, wall_y, wall_z, mw=(1.0, 1.0, 1.0)):
    g = np.random.default_rng(nx * 10000 + ny * 100 + nz)
    p = W.base_params(nx, ny, wall_y=wall_y, kappa=(0.02, 0.03, 0.015), kappa_c=0.0, mobility=0.1)
    p.update(lattice=1, nz=nz, wall_z=wall_z, force_form=0, mw=list(mw), fext=[1e-6, -2e-6, 1.5e-6])
    sh = (nz, ny, nx)
    c3, c1 = 0.3 * g.random(sh), 0.3 * g.random(sh)
    f = W.fields_from_C(c1, 1.0 - c1 - c3, c3, mw=mw)
    f["u"] = [1e-3 * g.standard_normal(sh) for _ in range(3)]
    return dict(params=p, fields=f, membranes=[])


def _same(a, b, caps=0):
    fa, fb = a.fields(), b.fields()
    for q in fa:
        assert np.array_equal(fa[q], fb[q]), (q, float(np.abs(fa[q] - fb[q]).max()))
    for i in range(caps):
        ma, mb = a.membrane(i), b.membrane(i)
        for q in ma:
            assert np.array_equal(ma[q], mb[q]), (q, float(np.abs(ma[q] - mb[q]).max()))


@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz,wall_y,wall_z", [(64, 9, 11, 0, 0), (33, 13, 6, 1, 1), (125, 5, 4, 0, 1),
                                                    (7, 6, 5, 1, 0), (1, 3, 9, 0, 0), (5, 2, 2, 1, 1), (3, 1, 1, 0, 0),
                                                    (130, 110, 107, 1, 1)])
def test_calls_divide_alike(nx, ny, nz, wall_y, wall_z, storage):
    w = _fluid(nx, ny, nz, wall_y, wall_z)
    a, b = (lbib.from_workload(w, storage=storage) for _ in range(2))
    a.step(5)
    for _ in range(5):
        b.step(1)
    _same(a, b)
    a.step(2)
    b.step(1)
    b.step(1)
    _same(a, b)


@pytest.mark.parametrize("mw", [(1.0, 1.0, 1.0), (2.5, 1.0, 1.5)])
@pytest.mark.parametrize("wall_z,storage", [(1, "fp32"), (0, "fp64")])
def test_calls_divide_alike_with_capsules(wall_z, storage, mw):
    w = W.capsule3d(n=36, R=7.0, subdiv=2, wall_z=wall_z, two=False, bridge=False, shift=(9.0, 3.0, 1.0))
    phi, psi = w["fields"]["phi"], w["fields"]["psi"]
    w["params"]["mw"] = list(mw)
    w["fields"] = W.fields_from_C((1.0 - psi + phi) / 2, (1.0 - psi - phi) / 2, psi, mw=mw)
    a, b = (lbib.from_workload(w, storage=storage) for _ in range(2))
    a.step(9)
    for _ in range(3):
        b.step(1)
        b.step(2)
    _same(a, b, 1)
