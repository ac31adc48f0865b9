"""The fused MLP passes at the edges of their tiles: rows that fill no tile,
one tile exactly and one row more, the row counts around the switch between
the 16-row and the 64-row forward, batches that end inside a 32-row block or
a 512-row chunk of the weight gradients, and rows at 4-byte alignment.

The bound is the one the other MLP tests derive (mlp_case.TOL)."""
import numpy as np
import pytest

from mlp_case import BLOCKS, TOL, case, rel_l2
from oracle import mlp_ref as M
from paper_2509_26279_amd import sas

pytestmark = pytest.mark.gpu


def _net(p, mu, sd, max_batch):
    net = sas.MLP(max_batch=max_batch, seed=1)
    net.set_params(p)
    net.set_norm(mu, sd)
    return net


@pytest.mark.parametrize("n", [15, 16, 17, 16383, 16384, 16385, 16447])
@pytest.mark.parametrize("shift", [0, 1])
def test_forward_tiles(gpu, n, shift):
    import torch
    p, x, y, mu, sd = case(n, n)
    net = _net(p, mu, sd, 64)
    flat = torch.zeros(n * 32 + 4, dtype=torch.float32, device="cuda")
    xt = flat[shift:shift + n * 32].view(n, 32)   # shift 1: rows 4 bytes off a 16-byte line
    xt.copy_(torch.as_tensor(x))
    z = net.forward(xt).cpu().numpy()
    ref, _ = M.forward(p, x, mu, sd)
    assert z.shape == (n,)
    assert rel_l2(z, ref) < TOL
    net.close()


@pytest.mark.parametrize("B", [1, 16, 31, 33, 511, 513, 1025])
def test_gradient_tiles(gpu, B):
    import torch
    p, x, y, mu, sd = case(7000 + B, B)
    y[0] = 1.0                                    # a positive row also at B = 1
    net = _net(p, mu, sd, 1100)                   # the batch leaves part of the buffers unused
    xt, yt = torch.as_tensor(x).cuda(), torch.as_tensor(y).cuda()
    net.grad(torch.full((1100, 32), 3.0, device="cuda"), torch.ones(1100, device="cuda"))
    loss, g = net.grad(xt, yt, 3.0)               # what the full batch left is not read
    rl, rg = M.loss_and_grad(p, x, y, mu, sd, pos_weight=3.0)
    assert float(loss.cpu()) == pytest.approx(rl, rel=TOL)
    g = g.cpu().numpy().astype(np.float64)
    for name, a, b in BLOCKS:
        assert rel_l2(g[a:b], rg[a:b]) < TOL, name
    net.close()
