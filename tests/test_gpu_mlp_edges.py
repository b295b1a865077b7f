"""The network kernels where their tiling can go wrong: around 16 contacts (a
tile), 64 (a block of four waves) and the row count at which the grid is full
and waves walk several tiles.

Gradient: the mean over 2 m rows is the mean of the two halves' gradients, and
the adjoints' scale 2 / (n nout) differs by exactly a power of two between the
two, so every bf16 operand is the same and only the float32 sums differ.  A sum
is at most 40 additions deep (a tile's products, the waves' tiles, the rows of
partial sums), its terms add up to at most sqrt(n) times a typical sum (random
signs): 40 * 2^-24 * sqrt(2 m) of the largest entry.

Inference: a contact's outputs do not depend on the rows around it, bit for
bit (every contact has its own column of the products).
"""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


def _rows(n, seed):
    rng = np.random.default_rng(seed)
    f = np.zeros((n, 8), np.float32)
    f[:, 0] = rng.normal(-1e-3, 1.5e-3, n)
    f[:, 1:4] = rng.normal(0, 0.1, (n, 3))
    f[:, 4] = rng.uniform(0.01, 0.5, n)
    f[:, 5] = rng.uniform(0.3, 1.0, n)
    f[:, 6] = 0.002
    f[:, 7] = np.nan  # ignored
    return f, rng.normal(0, 1, (n, 16)).astype(np.float32)


def _net(seed):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_12185_amd import cfsim
    f, _ = _rows(4096, seed)
    p = mlp.init_params(np.nan_to_num(f), seed=seed)
    p[mlp.OFF_B1:mlp.OFF_W2] = np.linspace(-0.5, 0.5, mlp.NH)
    return torch, cfsim.ImpedanceNet(p.astype(np.float32))


@pytest.mark.parametrize("m", [1, 8, 15, 17, 33, 63, 65, 8191, 8193, 40001])
@pytest.mark.parametrize("nout", [1, 10])
def test_gradient_of_halves(m, nout):
    print(f"case: gradient halves m {m} nout {nout}", flush=True)
    torch, net = _net(3)
    f, t = _rows(2 * m, m)
    t[:, nout:] = np.nan  # outputs past nout take no target
    F, T = torch.from_numpy(f).cuda(), torch.from_numpy(t).cuda()
    g, loss = net.gradient(F, T, nout)
    parts = [net.gradient(F[k * m:(k + 1) * m].contiguous(), T[k * m:(k + 1) * m].contiguous(), nout)
             for k in range(2)]
    ref = 0.5 * (parts[0][0].double() + parts[1][0].double())
    tol = 40 * 2.0 ** -24 * (2 * m) ** 0.5
    assert torch.isfinite(g).all()
    assert float((g.double() - ref).abs().max()) <= tol * float(ref.abs().max())
    lref = 0.5 * float(parts[0][1].item() + parts[1][1].item())
    assert abs(float(loss.item()) - lref) <= 40 * 2.0 ** -24 * lref


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 65535, 65537, 131089])
def test_forward_rows_are_independent(n):
    print(f"case: forward rows n {n}", flush=True)
    torch, net = _net(4)
    f, _ = _rows(n, n)
    F = torch.from_numpy(f).cuda()
    y = torch.full((n, 16), float("nan"), device="cuda")
    net.forward(F, out=y)
    pick = sorted({0, n // 3, n - 1})
    alone = torch.cat([net.forward(F[k:k + 1].contiguous()) for k in pick])
    assert torch.isfinite(y).all()
    assert torch.equal(y[pick], alone)
    ref, _ = mlp.forward(net.params.cpu().numpy().astype(np.float64), np.nan_to_num(f[pick]).astype(np.float64))
    # bf16 rounding of inputs, weights and activations: a few times 2^-9
    assert np.abs(alone.cpu().numpy() - ref).max() <= 0.03 * np.abs(ref).max() + 1e-3
