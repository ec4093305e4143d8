"""Checkpoints of lattices whose planes do not end on an aligned address: a
state loaded into another handle is the saved one to the last node, in every
storage, and files without the planes' end still load."""
import numpy as np
import pytest

from helpers import run_gpu
from paper_1906_03065_amd import lbib
from paper_1906_03065_amd import workloads as W

pytestmark = pytest.mark.gpu


def _fluid(dim, nx, ny, nz=1):
    g = np.random.default_rng(nx)
    p = W.base_params(nx, ny, nz, lattice=dim - 2, kappa=(0.02, 0.03, 0.015), kappa_c=0.0, mobility=0.1)
    sh = (nz, ny, nx)[3 - dim:]
    c3, c1 = 0.3 * g.random(sh), 0.3 * g.random(sh)
    return dict(params=p, fields=W.fields_from_C(c1, 1.0 - c1 - c3, c3), membranes=[])


def _same(a, b):
    fa, fb = a.fields(), b.fields()
    for q in fa:
        assert np.array_equal(fa[q], fb[q]), (q, float(np.abs(fa[q] - fb[q]).max()))


@pytest.mark.parametrize("storage", ["fp32", "fp64", "fp16", "bf16"])
@pytest.mark.parametrize("dim,size", [(2, (64, 64)), (2, (70, 61)), (2, (7, 9)), (2, (53, 1)), (3, (24, 22, 20)),
                                      (3, (13, 11, 9))])
def test_checkpoint_restores_every_node(dim, size, storage):
    w = _fluid(dim, *size)
    a = run_gpu(w, storage)
    a.step(2)
    blob = a.save()
    c = run_gpu(w, storage)
    c.step(5)  # other numbers everywhere
    c.load(blob)
    _same(a, c)
    for s in (a, c):
        s.step(3)
    _same(a, c)
    with pytest.raises(lbib.LbibError):
        c.load(blob[:-8])
    if blob[:8] == b"BLIBCKP2":  # as files were before: the first tag, without the planes' end
        n = 8 * 12 + int(np.frombuffer(blob, np.int64, 12)[10])
        c.load(b"BLIBCKP1" + blob[8:n])
        assert c.steps_done == 2
