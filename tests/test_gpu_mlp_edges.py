"""Training batches that end inside a 32-row block, where the rows past the
batch must not be seen even if a weight is infinite, and passes over more rows
than one launch of workgroups takes at a time."""
import numpy as np
import pytest

from mlp_case import BLOCKS, TOL, case, rel_l2
from oracle import mlp_ref as M
from paper_2509_26279_amd import sas

pytestmark = pytest.mark.gpu

W1, B1, W2, B2 = 0, 4096, 4224, 20608


def _net(p, mu, sd, max_batch=64):
    net = sas.MLP(max_batch=max_batch, seed=1)
    net.set_params(p)
    net.set_norm(mu, sd)
    return net


@pytest.mark.parametrize("B", [1, 31, 32, 33, 48])
def test_rows_past_the_batch_meet_an_infinite_weight(gpu, B):
    import torch
    p, x, y, mu, sd = case(100 + B, B)
    y[0] = 1.0
    x[:] = np.abs(x) + 5.0
    mu[:], sd[:] = 0.0, 1.0
    p[W1:B1].reshape(32, 128)[:, 5] = -1.0  # unit 5 is off in every row, and on (its
    p[B1 + 5] = 0.5                         # bias) where the inputs are zero
    w2 = p[W2:B2].reshape(128, 128)
    w2[:, 7] = 0.0                          # unit 7 of the second layer is off
    p[B2 + 7] = -1.0
    xt, yt = torch.as_tensor(x).cuda(), torch.as_tensor(y).cuda()
    got = []
    for v in (0.0, np.inf):                 # a weight between units that are off
        w2[5, 7] = v
        net = _net(p, mu, sd)
        loss, g = net.grad(xt, yt, 3.0)
        got.append((loss.cpu().numpy().copy(), g.cpu().numpy()))
        net.close()
    assert np.isfinite(got[0][1]).all()
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("n", [49152, 49153, 49217, 120000])
def test_forward_second_trip(gpu, n):
    import torch
    p, x, y, mu, sd = case(n, n)
    net = _net(p, mu, sd)
    z = net.forward(torch.as_tensor(x).cuda()).cpu().numpy()
    net.close()
    assert rel_l2(z, M.forward(p, x, mu, sd)[0]) < TOL
    tail = slice(49152 - 64, min(n, 49152 + 64))  # around the first row of a second trip
    assert rel_l2(z[tail], M.forward(p, x[tail], mu, sd)[0]) < TOL


@pytest.mark.parametrize("B", [32768, 32769, 33000])
def test_gradient_second_trip(gpu, B):
    import torch
    p, x, y, mu, sd = case(B, B)
    net = _net(p, mu, sd, max_batch=33000)
    loss, g = net.grad(torch.as_tensor(x).cuda(), torch.as_tensor(y).cuda(), 3.0)
    rl, rg = M.loss_and_grad(p, x, y, mu, sd, pos_weight=3.0)
    assert float(loss.cpu()) == pytest.approx(rl, rel=TOL)
    g = g.cpu().numpy().astype(np.float64)
    for name, a, b in BLOCKS:
        assert rel_l2(g[a:b], rg[a:b]) < TOL, name
    net.close()


@pytest.mark.parametrize("n,max_batch", [(1, 64), (1000, 64), (20000, 4096), (20000, 20000)])
@pytest.mark.parametrize("at", [0, 1])
def test_logits_over_their_rows(gpu, n, max_batch, at):
    import torch
    p, x, y, mu, sd = case(n, n)
    net = _net(p, mu, sd, max_batch)
    xt = torch.as_tensor(x).cuda()
    ref = net.forward(xt).cpu().numpy()
    over = xt.flatten().clone()
    assert sas.load().sas_mlp_forward(net._m, over.data_ptr(), n, over.data_ptr() + 4 * at,
                                      None) == sas.SAS_OK
    torch.cuda.synchronize()
    assert np.array_equal(over[at:at + n].cpu().numpy(), ref)
    net.close()
