"""Standard RKFR steps of GLM-MHD in FP64 on both sides of the mesh size up to
which a stage loads its operands ahead (1024 wavefronts: 4096 elements of
degree 3 in tiles of four, 7168 of degree 2 in pairs of wavefronts of 14),
against the oracle with the 1e-12 of the other RKFR tests."""
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


@pytest.mark.parametrize("nx,ny,N,vol", [(64, 64, 3, 3), (17, 241, 3, 3), (64, 64, 3, 0), (17, 241, 3, 0),
                                         (64, 112, 2, 0), (67, 107, 2, 0), (1, 3, 2, 0), (3, 1, 3, 3)])
def test_mhd_rkfr_around_the_ahead_limit(orc, nx, ny, N, vol):
    p = orc.Problem(dim=2, nx=nx, ny=ny, N=N, eq=orc.MHD, gamma=5.0 / 3.0, vol_flux=vol)
    s = crk.Solver(dim=2, nx=nx, ny=ny, degree=N, equation=crk.CRK_GLM_MHD, gamma=5.0 / 3.0, volume_flux=vol)
    xi, _ = orc.gll(N)
    u = inputs.perturb(inputs.orszag_tang(nx, ny, xi), 7, 1e-3)
    p.ch = orc.compute_ch(p, u)
    dt = orc.compute_dt(p, u)
    ref = orc.rkfr_step(p, u, dt)
    out = s.new_state()
    s.rkfr_step(torch.tensor(u, device="cuda"), out, torch.tensor([dt, p.ch], dtype=torch.float64, device="cuda"),
                compute_dt=False)
    got = out.cpu().numpy()
    big = np.max(np.abs(ref))
    for v in range(ref.shape[0]):
        assert np.max(np.abs(got[v] - ref[v])) <= 1e-12 * max(np.max(np.abs(ref[v])), 1e-3 * big), v
