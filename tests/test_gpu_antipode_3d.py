"""Tiles that straddle the antipode of a mesh's box and lie within its band:
their nodes belong to different periodic images, searched wave by wave and
image by image.  Bands that nearly fill the period, a box whose last tile is
partial, the antipode at and between the edges of a 4^3 sub-tile, along one
axis and along all three, and a mesh with more triangles than a wave's list
holds: FP64 against the oracle, which compares every node with every triangle."""
import numpy as np
import pytest

from helpers import compare, marker_err, run_gpu, run_oracle
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R,subdiv,r_cut,wall_z,shift", [
    (32, 6.0, 2, 8.9, 0, (0.0, 0.0, 0.0)), (32, 6.0, 3, 8.9, 1, (1.9, 3.6, 0.0)),
    (34, 6.5, 4, 9.2, 0, (5.0, -4.2, 2.6))])
def test_antipode_tiles_vs_oracle(orc, n, R, subdiv, r_cut, wall_z, shift):
    """The same closest triangles give the same profile and forces to rounding:
    1e-9 as in the other FP64 parity tests."""
    w = W.capsule3d(n=n, R=R, subdiv=subdiv, two=False, bridge=False, r_cut=r_cut, wall_z=wall_z, shift=shift)
    o = run_oracle(orc, w)
    g = run_gpu(w, "fp64")
    for k in (1, 3):
        o.step(k - o.steps_done)
        g.step(k - g.steps_done)
        for q, v in compare(g, o, D=3).items():
            assert v < 1e-9, (k, q, v)
        assert marker_err(g, o, 1) < 1e-10
    assert g.check() == 0


@pytest.mark.parametrize("subdiv,r_cut,steps", [(2, 4.0, 60), (4, 4.0, 25), (4, 9.2, 12)])
def test_renewed_entries_bitwise(subdiv, r_cut, steps):
    """Meshes coarse and fine against the lattice, the fine ones with entries that
    last a few steps at most: the state is bitwise the one without kept entries."""
    w = W.capsule3d(n=34, R=6.5, subdiv=subdiv, two=False, bridge=False, r_cut=r_cut, tau=0.85,
                    shift=(5.0, -4.2, 2.6))
    w["params"]["fext"] = [4e-6, 2e-6, 1e-6]
    a, b = run_gpu(w, "fp32"), run_gpu(w, "fp32")
    b.set_coupling_cache(0)
    for n in (1, steps - 1):
        a.step(n)
        b.step(n)
        fa, fb = a.fields(), b.fields()
        ma, mb = a.membrane(0), b.membrane(0)
        for q in fa:
            assert np.array_equal(fa[q], fb[q]), (n, q)
        for q in ma:
            assert np.array_equal(ma[q], mb[q]), (n, q)
    assert a.check() == 0


def _globe(nlon, nlat):
    """Unit sphere of meridians and parallels, outward: nlon triangles around
    each pole, which get thin as nlon grows."""
    V = [(0.0, 0.0, -1.0)]
    for i in range(1, nlat):
        t = np.pi * i / nlat
        V += [(np.sin(t) * np.cos(p), np.sin(t) * np.sin(p), -np.cos(t)) for p in 2 * np.pi * np.arange(nlon) / nlon]
    V.append((0.0, 0.0, 1.0))
    at = lambda i, j: 1 + (i - 1) * nlon + j % nlon
    T = []
    for j in range(nlon):
        T.append((0, at(1, j + 1), at(1, j)))
        for i in range(1, nlat - 1):
            T += [(at(i, j), at(i, j + 1), at(i + 1, j + 1)), (at(i, j), at(i + 1, j + 1), at(i + 1, j))]
        T.append((at(nlat - 1, j), at(nlat - 1, j + 1), len(V) - 1))
    return np.array(V), np.array(T, dtype=np.int32)


@pytest.mark.parametrize("nlon,nlat", [(14, 9), (16, 9), (160, 8)])
def test_many_and_thin_triangles_around_a_vertex(orc, nlon, nlat):
    """Vertices whose triangles overflow a row of the one-ring table (above 15
    neighbours), and triangles too thin for an FP32 normal: FP64 against the
    oracle over steps that hold, renew and search entries, 1e-9 as above."""
    w = W.capsule3d(n=34, R=6.5, subdiv=1, two=False, bridge=False, r_cut=4.0, shift=(0.3, -0.2, 0.1))
    c = w["membranes"][0]["X"].mean(axis=0)
    V, T = _globe(nlon, nlat)
    w["membranes"][0].update(X=6.5 * V + c, tris=T)
    o = run_oracle(orc, w)
    g = run_gpu(w, "fp64")
    for k in (1, 6):
        o.step(k - o.steps_done)
        g.step(k - g.steps_done)
        for q, v in compare(g, o, D=3).items():
            assert v < 1e-9, (k, q, v)
        assert marker_err(g, o, 1) < 1e-10
    assert g.check() == 0
