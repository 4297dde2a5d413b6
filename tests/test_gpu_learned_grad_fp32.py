"""The network gradient is FP32 arithmetic: an infinite feature leaves
infinities where FP32 products and sums have them, and no NaN beside them;
the rounding error stays that of FP32 sums."""
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


def _bf16(net):
    return (net.theta_bf16.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)


@pytest.mark.parametrize("sample,feature", [(0, 0), (21, 2), (39, 15)])
def test_infinite_feature(sample, feature):
    """Positive weights, so that no infinities of both signs meet: FP32
    arithmetic leaves +inf in the sums that the feature enters, finite values
    elsewhere, and no NaN."""
    rng = np.random.default_rng(feature)
    net = crk.MLP(theta=rng.uniform(0.01, 0.05, 5313).astype(np.float32))
    x, y = rng.uniform(0.1, 1.0, (40, 16)).astype(np.float32), np.zeros(40, np.float32)
    x[sample, feature] = np.inf
    t = torch.tensor(_bf16(net))
    W1, b1, W2, b2, W3, b3 = t[:1024].view(64, 16), t[1024:1088], t[1088:5184].view(64, 64), t[5184:5248], t[5248:5312], t[5312]
    X = torch.tensor(x)
    h1 = torch.relu((W1 * X[:, None, :]).sum(-1) + b1)
    h2 = torch.relu((W2 * h1[:, None, :]).sum(-1) + b2)
    dz = (torch.sigmoid((W3 * h2).sum(-1) + b3) - torch.tensor(y)) / 40
    d2 = dz[:, None] * W3
    d1 = (W2.t() * d2[:, None, :]).sum(-1)
    ref = torch.cat([(d1[:, :, None] * X[:, None, :]).sum(0).flatten(), d1.sum(0),
                     (d2[:, :, None] * h1[:, None, :]).sum(0).flatten(), d2.sum(0), (dz[:, None] * h2).sum(0), dz.sum()[None]])
    assert ref.isinf().sum() == 64 + 4096 + 64 and not ref.isnan().any()
    _, g, _ = net.loss_grad(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"))
    g = g.cpu()
    assert not g.isnan().any()
    assert torch.equal(g.isinf(), ref.isinf())
    fin = ~ref.isinf()
    # sums of 64 and of 40 rounded products of one sign, twice: (64 + 64 + 40) 2^-24
    assert ((g - ref).abs()[fin] <= 2e-5 * ref.abs()[fin]).all()


@pytest.mark.parametrize("n", [200, 8192])
def test_rounding_error_is_fp32(orc, n):
    """Every hidden unit active and every weight and input positive, so that
    no sum cancels: each entry of the gradient is a sum over the samples of
    products of values that themselves went through at most three sums of
    positive FP32 products (16, 64 and 64 terms, chains of fused
    multiply-adds), so its relative error stays below their lengths times
    2^-24; entry by entry, not in a norm."""
    rng = np.random.default_rng(n)
    net = crk.MLP(theta=rng.uniform(0.005, 0.03, 5313).astype(np.float32))
    x, y = rng.uniform(0.1, 1.0, (n, 16)).astype(np.float32), np.zeros(n, np.float32)
    _, go = orc.mlp_loss_grad(16, 64, _bf16(net).astype(np.float64), x.astype(np.float64), y.astype(np.float64))
    _, g, _ = net.loss_grad(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"))
    # 64 samples in one chain, then at most 16 partials and a tree of four
    assert np.max(np.abs(g.cpu().numpy() - go) / np.abs(go)) <= (16 + 64 + 64 + 64 + 20) * 2.0 ** -24
