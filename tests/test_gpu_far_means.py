"""Means between far states in the kernels that step them: the paper's 1D
density wave (density 0.02 to 1.98) on meshes so coarse that most pairs differ
by more than a factor of two, in the single launch of ``run``; and states with
a NaN or a value that is not positive among far ones, whose means must be NaN
as the logarithms are."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2604_02125_amd import crk, inputs  # noqa: E402
from test_gpu_far_states import far_state  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    crk.lib()


@pytest.mark.parametrize("lim", [0, 1])
@pytest.mark.parametrize("N", [1, 2, 3, 4])
@pytest.mark.parametrize("nx", [2, 5, 16, 51])
def test_coarse_density_wave(orc, nx, N, lim):
    p = orc.Problem(dim=1, nx=nx, N=N, vol_flux=orc.VOL_RANOCHA, limiter=orc.LIM_BLEND_MODAL if lim else orc.LIM_NONE)
    s = crk.Solver(dim=1, nx=nx, degree=N, volume_flux=crk.VOL_RANOCHA, limiter=lim, alpha_max=p.alpha_max,
                   alpha_min=p.alpha_min)
    xi, _ = orc.gll(N)
    ref = inputs.density_wave_1d(nx, xi)
    buf, dt = [torch.tensor(ref, device="cuda"), s.new_state()], s.new_dt()
    s.prepare(buf[0], dt)
    got = s.run(buf[0], buf[1], dt, 6).cpu().numpy()
    for _ in range(6):
        ref, _ = orc.crk_step(p, ref, orc.compute_dt(p, ref))
    for v in range(3):
        assert np.max(np.abs(got[v] - ref[v])) <= 1e-12 * np.max(np.abs(ref[v]))


@pytest.mark.parametrize("what", ["nan_energy", "nan_density", "negative_pressure", "zero_pressure"])
@pytest.mark.parametrize("eq,N", [("euler", 1), ("euler", 2), ("euler", 3), ("mhd", 2), ("mhd", 3)])
def test_inadmissible_node(orc, eq, N, what):
    """One step of given size: the element of the bad node and its neighbours
    are not finite where the oracle's are not, every other element agrees."""
    kw = dict(dim=2, nx=7, ny=6, N=N, vol_flux=3 if eq == "mhd" else 2)
    if eq == "mhd":
        kw.update(eq=orc.MHD, gamma=5.0 / 3.0)
    p = orc.Problem(**kw)
    s = crk.Solver(dim=2, nx=7, ny=6, degree=N, equation=p.eq, gamma=p.gamma, volume_flux=p.vol_flux)
    u = far_state(orc, p, seed=N)
    if eq == "mhd":
        p.ch = orc.compute_ch(p, u)
    dt = 0.1 * orc.compute_dt(p, u)
    e, k, en = 17, 1, 4 if eq == "mhd" else 3
    if what == "nan_density":
        u[0, e, k] = np.nan
    elif what == "nan_energy":
        u[en, e, k] = np.nan
    else:
        rest = 0.5 * (u[1:en, e, k] ** 2).sum() / u[0, e, k] + 0.5 * (u[en + 1:, e, k] ** 2).sum()
        u[en, e, k] = rest if what == "zero_pressure" else rest - 0.5
    with np.errstate(all="ignore"):
        ref, _ = orc.crk_step(p, u, dt)
    out = s.new_state()
    s.step(torch.tensor(u, device="cuda"), out, torch.tensor([dt, p.ch if eq == "mhd" else 0.0], dtype=torch.float64, device="cuda"),
           compute_dt=False)
    got = out.cpu().numpy()
    assert not np.isfinite(got[en, e]).all() and not np.isfinite(ref[en, e]).all()
    x, y = e % 7, e // 7
    touched = {e, y * 7 + (x + 1) % 7, y * 7 + (x - 1) % 7, (y + 1) % 6 * 7 + x, (y - 1) % 6 * 7 + x}
    rest = [i for i in range(42) if i not in touched]
    for v in range(u.shape[0]):
        assert np.isfinite(got[v, rest]).all()
        assert np.max(np.abs(got[v, rest] - ref[v, rest])) <= 1e-12 * max(np.max(np.abs(ref[v, rest])), 1e-300)
