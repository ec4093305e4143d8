"""Forward passes whose outputs lie over their inputs, in full, in part, and
beside them: bitwise those of separate arrays, with and without a workspace.
With very many rows some workgroups start when others have written theirs."""
import numpy as np
import pytest

from paper_1906_03065_amd import lbib, mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,noalloc", [(1, 0), (16, 1), (17, 0), (17, 1), (300, 0), (300, 1), (4096, 0), (4096, 1),
                                       (60000, 0)])
def test_outputs_over_inputs(B, noalloc):
    import torch

    g = np.random.default_rng(B)
    net = lbib.Mlp(B)
    p = mlp.init_params(3)
    net.set_params(p)
    prm = torch.as_tensor(p).to(net.device)
    x = torch.as_tensor(g.normal(size=(B, 6)).astype(np.float32)).to(net.device)
    want = net.forward(x)
    # inputs at the start of the outputs, at their end, across either end, and just outside
    for at in (0, 26 * B, 13 * B, -3, 32 * B - 5, -6 * B, 32 * B):
        buf = torch.full((48 * B,), float("nan"), device=net.device)
        y0 = 8 * B
        xin = buf[y0 + at:y0 + at + 6 * B].view(B, 6)
        xin.copy_(x)
        y = buf[y0:y0 + 32 * B].view(B, 32)
        if noalloc:
            lbib.mlp_forward_noalloc(prm, xin, y)
        else:
            rc = lbib.lib().lbib_mlp_forward(net.h, xin.data_ptr(), B, y.data_ptr())
            assert rc == 0
        torch.cuda.synchronize()
        assert torch.equal(y, want), at
