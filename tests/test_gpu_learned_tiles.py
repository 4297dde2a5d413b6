"""Network kernels at the edges of their tiling (16 samples per matrix tile,
64 per wavefront of the inference and per workgroup and pass of the gradient,
at most 256 workgroups), against the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2604_02125_amd import crk  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    crk.lib()


def _net(seed):
    rng = np.random.default_rng(seed)
    th = np.concatenate([rng.normal(0, 0.35, 1024), rng.normal(0, 0.1, 64), rng.normal(0, 0.18, 4096),
                         rng.normal(0, 0.1, 64), rng.normal(0, 0.12, 64), rng.normal(0, 0.1, 1)]).astype(np.float32)
    net = crk.MLP(theta=th)
    return net, net.theta_bf16.view(torch.bfloat16).double().cpu().numpy()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 129, 16385, 32769])
def test_tile_edges(orc, n):
    net, th = _net(n)
    rng = np.random.default_rng(100 + n)
    x = rng.uniform(0.0, 1.0, (n, 16)).astype(np.float32)
    y = (rng.uniform(size=n) < 0.4).astype(np.float32)
    xg, yg = torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda")
    z, a = net.forward(xg, alpha_max=0.008)
    zo, ao = orc.mlp_forward(16, 64, th, x.astype(np.float64), 0.008)
    # a sum of up to 64 FP32 products rounds to 64 2^-24 = 4e-6 of its terms at most, over three layers
    assert np.max(np.abs(z.cpu().numpy() - zo)) <= 1.2e-5 * max(1.0, np.max(np.abs(zo)))
    assert np.max(np.abs(a.cpu().numpy() - ao)) <= 0.008 * 1.2e-5 * max(1.0, np.max(np.abs(zo)))
    loss, g, _ = net.loss_grad(xg, yg)
    lo, go = orc.mlp_loss_grad(16, 64, th, x.astype(np.float64), y.astype(np.float64))
    # the same rounding per back-propagated value; sums over samples whose
    # terms cancel to about 1/sqrt(n) and no more
    tol = 2.4e-5 * max(1.0, np.sqrt(n) / 4)
    assert abs(loss.item() - lo) <= 1e-5 * max(1.0, abs(lo))
    assert np.linalg.norm(g.cpu().numpy() - go) <= tol * np.linalg.norm(go)


def test_infinite_inputs():
    """An infinite feature acts as in FP32 arithmetic (its sample only)."""
    net, th = _net(3)
    x = torch.rand(40, 16, generator=torch.Generator().manual_seed(1))
    x[5, 2], x[21, 7] = float("inf"), -float("inf")
    x[33, 1] = float("nan")
    t = torch.tensor(th, dtype=torch.float32)
    W1, b1, W2, b2 = t[:1024].view(64, 16), t[1024:1088], t[1088:5184].view(64, 64), t[5184:5248]
    def relu(v):                    # NaN counts as zero, as in the kernels
        return torch.where(v > 0, v, torch.zeros_like(v))
    h1 = relu((W1 * x[:, None, :]).sum(-1) + b1)
    ref = (t[5248:5312] * relu((W2 * h1[:, None, :]).sum(-1) + b2)).sum(-1) + t[5312]
    z, _ = net.forward(x.cuda())
    z = z.cpu()
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(z), fin) and torch.equal(torch.isnan(z), torch.isnan(ref))
    assert torch.equal(z[~fin & ~ref.isnan()], ref[~fin & ~ref.isnan()])
    assert (z[fin] - ref[fin]).abs().max() <= 2.4e-5 * max(1.0, ref[fin].abs().max())
