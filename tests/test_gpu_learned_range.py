"""The learned indicator's fallback looks at every one of an element's 16
features: four lanes hold four each, so a range that excludes an element by
one feature alone is tried in each of the four groups, at both ends, in
``crk_indicator`` and in the pipelined step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2604_02125_amd import crk, inputs  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    crk.lib()


@pytest.mark.parametrize("end", ["lo", "hi"])
@pytest.mark.parametrize("feature", [0, 3, 4, 5, 10, 15])
def test_every_feature_can_exclude_an_element(orc, feature, end):
    n = 24
    s = crk.Solver(dim=2, nx=n, ny=n, x0=-1.0, x1=1.0, y0=-1.0, y1=1.0, degree=3, volume_flux=crk.VOL_KG,
                   limiter=crk.LIM_BLEND)
    xi, _ = orc.gll(3)
    u = inputs.perturb(inputs.kelvin_helmholtz(n, n, xi, v2_modes=inputs.khi_modes(3)), 5, 1e-2)
    ug, dt = torch.tensor(u, device="cuda"), s.new_dt()
    modal = s.indicator(ug)[0].cpu().numpy()
    f = crk.features(s, ug).cpu().numpy()
    net = crk.MLP(seed=7)
    u16 = net.theta_bf16.cpu().numpy().view(np.uint16).astype(np.uint32) << 16
    _, a = orc.mlp_forward(16, 64, u16.view(np.float32).astype(np.float64), f.astype(np.float64), 0.008)
    a = np.where(a < 1e-3, 0.0, a)
    lo, hi = np.full(16, -1.0, np.float32), np.full(16, 2.0, np.float32)
    cut = np.float32(np.median(f[:, feature]))
    (lo if end == "lo" else hi)[feature] = cut
    out = f[:, feature] < cut if end == "lo" else f[:, feature] > cut
    assert 0 < out.sum() < s.nelem                    # some elements fall back by this feature alone
    assert np.max(np.abs(a[out] - modal[out])) > 1e-4  # and would show if they did not
    net.lo, net.hi = torch.tensor(lo, device="cuda"), torch.tensor(hi, device="cuda")
    net.bind(s)
    got = s.indicator(ug)[0].cpu().numpy()
    assert np.array_equal(got[out], modal[out])
    assert np.max(np.abs(got[~out] - a[~out])) <= 1e-7
    # the pipelined step with these coefficients against the one that is given them
    p = orc.Problem(dim=2, nx=n, ny=n, x0=-1.0, x1=1.0, y0=-1.0, y1=1.0, N=3, vol_flux=orc.VOL_KG,
                    limiter=orc.LIM_BLEND_GIVEN)
    alpha = orc.smooth_alpha(p, np.where(out, modal, a))
    ref, _ = orc.crk_step(p, u, orc.compute_dt(p, u), alpha)
    v = s.new_state()
    s.prepare(ug, dt)
    s.advance(ug, v, dt)
    v = v.cpu().numpy()
    assert max(np.max(np.abs(v[k] - ref[k])) / np.max(np.abs(ref[k])) for k in range(4)) <= 1e-8
