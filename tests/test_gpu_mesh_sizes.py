"""The pipelined step on both sides of the mesh sizes at which the launches
change: the local phase of a limited flow in one launch or two (16 wavefronts
per SIMD with Kennedy-Gruber in FP64; one launch for the other fluxes and for
degrees 1 and 4), and the GLM-MHD local phase with two lanes or one per node
(four wavefronts per SIMD in FP64 at degree 3), against the FP64 oracle with
the tolerances of the other parity tests."""
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


def _rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    return max(np.max(np.abs(a[v] - b[v])) / max(np.max(np.abs(b[v])), 1e-300) for v in range(b.shape[0]))


def _run(s, u, steps):
    buf = [torch.tensor(u, dtype=s.dtype, device="cuda"), s.new_state()]
    dt = s.new_dt()
    s.prepare(buf[0], dt)
    for n in range(steps):
        s.advance(buf[n % 2], buf[(n + 1) % 2], dt)
    return buf[steps % 2].cpu().numpy().astype(np.float64)


# elements per tile: 4 (N = 3, one wavefront), 14 (N = 2) and 5 (N = 4), two wavefronts; N = 1 has no flags
@pytest.mark.parametrize("nx,ny,N,vol", [(256, 256, 3, 1), (241, 272, 3, 1), (97, 85, 3, 2), (512, 224, 2, 1),
                                         (443, 259, 2, 1), (73, 71, 4, 1), (41, 43, 1, 1), (3, 2, 3, 1)])
def test_limiter_in_one_and_two_launches(orc, nx, ny, N, vol):
    p = orc.Problem(dim=2, nx=nx, ny=ny, x0=-1.0, x1=1.0, y0=-1.0, y1=1.0, N=N, vol_flux=vol,
                    limiter=orc.LIM_BLEND_MODAL)
    s = crk.Solver(dim=2, nx=nx, ny=ny, x0=-1.0, x1=1.0, y0=-1.0, y1=1.0, degree=N, volume_flux=vol,
                   limiter=crk.LIM_BLEND, alpha_max=p.alpha_max, alpha_min=p.alpha_min)
    xi, _ = orc.gll(N)
    u = inputs.kelvin_helmholtz(nx, ny, xi)
    r = inputs.perturb(u, 17, 0.05)                  # rough lower half: blending and clear tiles
    u[:, : (ny // 2) * nx, :] = r[:, : (ny // 2) * nx, :]
    ref = u.copy()
    for _ in range(3):
        ref, _ = orc.crk_step(p, ref, orc.compute_dt(p, ref))
    assert _rel(_run(s, u, 3), ref) <= 1e-12
    if nx * ny < 10000:
        # the phases issued separately give the same bits
        buf, dt = [torch.tensor(u, device="cuda"), s.new_state()], s.new_dt()
        s.prepare(buf[0], dt)
        for n in range(3):
            for ph in (crk.PHASE_LOCAL_PLAIN, crk.PHASE_LOCAL_BLEND, crk.PHASE_INTERFACE):
                s.advance(buf[n % 2], buf[(n + 1) % 2], dt, phases=ph)
        assert np.array_equal(buf[1].cpu().numpy(), _run(s, u, 3))


@pytest.mark.parametrize("nx,ny,N,prec", [
    (128, 128, 3, crk.FP64), (5, 3277, 3, crk.FP64), (23, 17, 3, crk.FP32), (1, 1, 4, crk.FP64), (1, 6, 3, crk.FP64), (7, 1, 2, crk.FP64), (5, 3, 2, crk.FP32), (13, 11, 1, crk.FP64)])
def test_mhd_around_the_lane_split_threshold(orc, nx, ny, N, prec):
    p = orc.Problem(dim=2, nx=nx, ny=ny, N=N, eq=orc.MHD, gamma=5.0 / 3.0, vol_flux=3)
    s = crk.Solver(dim=2, nx=nx, ny=ny, degree=N, equation=crk.CRK_GLM_MHD, gamma=5.0 / 3.0, volume_flux=crk.VOL_DERIGS,
                   precision=prec)
    xi, _ = orc.gll(N)
    u = inputs.random_smooth_mhd(nx, ny, xi, seed=5)
    if prec == crk.FP32:
        u = u.astype(np.float32).astype(np.float64)
    ref = u.copy()
    for _ in range(2):
        p.ch = orc.compute_ch(p, ref)
        ref, _ = orc.crk_step(p, ref, orc.compute_dt(p, ref))
    assert _rel(_run(s, u, 2), ref) <= (1e-12 if prec == crk.FP64 else 2e-5)
