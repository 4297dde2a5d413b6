"""Pipelined steps on meshes whose rows are shorter than a tile (a tile spans
several rows), just as long and just longer, with and without walls, against
the oracle; tile counts that leave the last workgroup of four tiles partly
empty are among them.  Two steps, the 1e-12 of the other parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2604_02125_amd import crk, inputs  # noqa: E402

W, P = 1, 0


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    crk.lib()


# elements per tile: 16 (N = 1), 14 (N = 2), 4 (N = 3), 5 (N = 4)
@pytest.mark.parametrize("bc", [(P, P), (W, P), (P, W), (W, W)], ids=["periodic", "xwall", "ywall", "box"])
@pytest.mark.parametrize("N,nx,ny", [(1, 1, 37), (1, 2, 9), (1, 5, 13), (1, 15, 9), (1, 16, 7), (1, 17, 5), (2, 3, 11),
                                     (3, 1, 9), (3, 2, 11), (3, 3, 7), (3, 4, 5), (3, 5, 5), (4, 2, 9), (4, 6, 3)])
def test_rows_around_the_tile_length(orc, N, nx, ny, bc):
    p = orc.Problem(dim=2, nx=nx, ny=ny, N=N, vol_flux=1, bc=bc, limiter=orc.LIM_BLEND_MODAL)
    s = crk.Solver(dim=2, nx=nx, ny=ny, degree=N, volume_flux=1, limiter=crk.LIM_BLEND, alpha_max=p.alpha_max,
                   alpha_min=p.alpha_min, boundary=bc)
    xi, _ = orc.gll(N)
    u = inputs.perturb(inputs.random_smooth_euler(nx, ny, xi, seed=3, amp=0.25), 4, 0.02)
    ref = u.copy()
    for _ in range(2):
        ref, _ = orc.crk_step(p, ref, orc.compute_dt(p, ref))
    buf, dt = [torch.tensor(u, device="cuda"), s.new_state()], s.new_dt()
    s.prepare(buf[0], dt)
    for n in range(2):
        s.advance(buf[n % 2], buf[(n + 1) % 2], dt)
    got = buf[0].cpu().numpy()
    big = np.max(np.abs(ref))
    for v in range(4):
        assert np.max(np.abs(got[v] - ref[v])) <= 1e-12 * max(np.max(np.abs(ref[v])), 1e-3 * big)
