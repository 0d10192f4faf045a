"""Bias gradients and the Adam step of the kernel network at sizes around their tiles (32 columns, 32 x 8
rows of the column sums; 32 x 32 tiles of the parameter update and its transposed bf16 copy)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pg = pytest.importorskip("paper_2206_15117_amd.polgrid")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,width,hidden,n_out,batch", [(1, 1, 1, 1, 1), (5, 33, 1, 70, 37), (24, 32, 2, 31, 255),
                                                           (7, 64, 3, 129, 256), (24, 40, 1, 1000, 300), (3, 8, 16, 5, 65)])
def test_bias_gradient_and_update(n_in, width, hidden, n_out, batch):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    net = pg.MLP(n_in, width, hidden, n_out, batch, seed=3)
    x = torch.randn((batch, n_in), device="cuda", generator=g)
    t = torch.randn((batch, n_out), device="cuda", generator=g)
    before = [(net.copy(pg.MLP_W, i).clone(), net.copy(pg.MLP_B, i).clone()) for i in range(hidden + 1)]
    net.train_step(x, t, 1e-2)
    # the output bias gradient is the column sum of dL/dy: float32 additions in a tree of depth
    # batch / 32 + 5, so at most that many rounding units of the sum of magnitudes
    gy = net.copy(pg.MLP_GY, hidden, batch).double()
    gb = net.copy(pg.MLP_GB, hidden).double()
    bound = (batch / 32 + 6) * 2.0 ** -24 * gy.abs().sum(0) + 1e-30
    assert bool(((gb - gy.sum(0)).abs() <= bound).all())
    for i, (w0, b0) in enumerate(before):
        for what, gwhat, p0 in ((pg.MLP_W, pg.MLP_GW, w0), (pg.MLP_B, pg.MLP_GB, b0)):
            grad = net.copy(gwhat, i).double()
            # the first step from zero moments: p - lr g / (|g| + eps), in float32 to a few units
            want = p0.double() - 1e-2 * grad / (grad.abs() + 1e-8)
            got = net.copy(what, i).double()
            assert float((got - want).abs().max()) <= 1e-2 * 1e-5 + 2.0 ** -23 * float(p0.abs().max())
        w = net.copy(pg.MLP_W, i)
        assert torch.equal(net.copy(pg.MLP_W_BF16, i), w.to(torch.bfloat16))
    # the forward product reads the transposed copies: a network loaded with these weights agrees bit for bit
    other = pg.MLP(n_in, width, hidden, n_out, batch, seed=9)
    for i in range(hidden + 1):
        other.load(i, net.copy(pg.MLP_W, i), net.copy(pg.MLP_B, i))
    assert torch.equal(net.forward(x), other.forward(x))
    assert np.isfinite(net.forward(x).cpu().numpy()).all()
