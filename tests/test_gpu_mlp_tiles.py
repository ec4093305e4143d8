"""The network's kernels at the edges of their row tiles (sixteen rows, 256
partial gradients): forward pass and gradient against the FP64 reference,
and a parameter array that is aligned to four bytes only."""
import numpy as np
import pytest

from oracle import mlp_ref as M
from paper_1906_03065_amd import lbib, mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [15, 16, 17, 4096, 4097, 8209])
def test_row_tiles_vs_fp64(B):
    """FP32 sums of at most 128 products (forward) and of the rows of one
    workgroup (gradient), each rounding 6e-8: 128 x 6e-8 < 1e-5 of the
    largest output, and the gradient's terms through three layers < 1e-4 of
    the largest entry."""
    g = np.random.default_rng(B)
    X, T = g.normal(size=(B, 6)).astype(np.float32), g.normal(size=(B, 32)).astype(np.float32)
    p = mlp.init_params(5)
    net = lbib.Mlp(B)
    net.set_params(p)
    y = net.forward(X).cpu().numpy()
    yo, _ = M.forward(p.astype(np.float64), X.astype(np.float64))
    assert np.abs(y - yo).max() <= 1e-5 * np.abs(yo).max()
    loss, gr = net.gradient(X, T)
    lo, go = M.loss_grad(p.astype(np.float64), X.astype(np.float64), T.astype(np.float64))
    assert np.abs(gr - go).max() <= 1e-4 * np.abs(go).max()
    assert abs(loss / lo - 1) <= 1e-5


def test_noalloc_parameters_aligned_to_a_float():
    import torch

    g = np.random.default_rng(3)
    p = mlp.init_params(7)
    net = lbib.Mlp(40)
    net.set_params(p)
    x = torch.as_tensor(g.normal(size=(40, 6)).astype(np.float32)).to(net.device)
    ref = net.forward(x)
    held = torch.empty(len(p) + 3, dtype=torch.float32, device=net.device)
    for off in (1, 2, 3):
        q = held[off:off + len(p)]
        q.copy_(torch.as_tensor(p))
        y = torch.empty_like(ref)
        lbib.mlp_forward_noalloc(q, x, y)
        assert torch.equal(y, ref)
