"""GLM-MHD local stages with two lanes per node and the central volume flux,
which hold the most registers (six dense stages spill at degrees 3 and 4):
default and dense six-stage tableaus, degrees 2 to 4, against the oracle with
the 1e-12 of the other parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2604_02125_amd import crk, inputs  # noqa: E402

DENSE6_A = [[0] * 6, [0.2, 0, 0, 0, 0, 0], [0.1, 0.15, 0, 0, 0, 0], [0.3, -0.1, 0.4, 0, 0, 0],
            [0.05, 0.1, 0.2, 0.25, 0, 0], [0.1, 0.2, -0.05, 0.3, 0.15, 0]]
DENSE6_B = [0.1, 0.15, 0.2, 0.25, 0.2, 0.1]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    crk.lib()


@pytest.mark.parametrize("dense", [False, True], ids=["default", "dense6"])
@pytest.mark.parametrize("N", [2, 3, 4])
@pytest.mark.parametrize("nx,ny", [(13, 11), (1, 7)])
def test_central_two_lane_step(orc, nx, ny, N, dense):
    tab = dict(A=DENSE6_A, b=DENSE6_B) if dense else {}
    p = orc.Problem(dim=2, nx=nx, ny=ny, N=N, eq=orc.MHD, gamma=5.0 / 3.0, vol_flux=0, **tab)
    s = crk.Solver(dim=2, nx=nx, ny=ny, degree=N, equation=crk.CRK_GLM_MHD, gamma=5.0 / 3.0, volume_flux=crk.VOL_CENTRAL, **tab)
    xi, _ = orc.gll(N)
    ref = inputs.random_smooth_mhd(nx, ny, xi, seed=9)
    buf, dt = [torch.tensor(ref, device="cuda"), s.new_state()], s.new_dt()
    s.prepare(buf[0], dt)
    for n in range(2):
        p.ch = orc.compute_ch(p, ref)
        ref, _ = orc.crk_step(p, ref, orc.compute_dt(p, ref))
        s.advance(buf[n % 2], buf[(n + 1) % 2], dt)
    got = buf[0].cpu().numpy()
    for v in range(9):
        assert np.max(np.abs(got[v] - ref[v])) <= 1e-12 * np.max(np.abs(ref[v])), v
