"""The local phase of a limited flow in one launch or in two (one per kind of
tile): the same bits.  Two launches serve meshes of more than 16 wavefronts per
SIMD in FP64, 64 in FP32, with Kennedy-Gruber at degrees 2 and 3, whatever the
indicator.  A mesh on the one-launch side, doubled in y with its state twice,
is on the two-launch side (1024 SIMDs; tiles of one wavefront hold 4 elements of
degree 3, of two 14 of degree 2): the same tiles, elements and time step."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2604_02125_amd import crk, inputs  # noqa: E402

WEIGHTS = os.path.join(crk.HERE, "mlp_indicator.npz")
#        nx, ny, degree, precision
MESHES = [(256, 256, 3, crk.FP64), (224, 512, 2, crk.FP64), (512, 512, 3, crk.FP32), (448, 1024, 2, crk.FP32)]
IDS = ["n3_fp64", "n2_fp64", "n3_fp32", "n2_fp32"]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    crk.lib()


def _solver(nx, ny, copies, N, prec, net):
    s = crk.Solver(dim=2, nx=nx, ny=copies * ny, x0=-1.0, x1=1.0, y0=-1.0, y1=-1.0 + 2.0 * copies, degree=N,
                   volume_flux=crk.VOL_KG, limiter=crk.LIM_BLEND, precision=prec)
    if net is not None:
        net.bind(s)
    return s


def _state(nx, ny, N):
    """Kelvin-Helmholtz (periodic in y), its lower half rough: both kinds of tile."""
    xi, _, _ = crk.reference_element(N)
    u = inputs.kelvin_helmholtz(nx, ny, xi)
    u[:, : (ny // 2) * nx] = inputs.perturb(u, 17, 0.1)[:, : (ny // 2) * nx]
    return torch.tensor(u, device="cuda")


def _run(s, u, phases, steps=3):
    buf, dt = [u.clone(), s.new_state()], s.new_dt()
    s.prepare(buf[0], dt)
    for n in range(steps):
        for ph in phases:
            s.advance(buf[n % 2], buf[(n + 1) % 2], dt, phases=ph)
    return buf[steps % 2], dt


BOTH = (crk.PHASE_LOCAL | crk.PHASE_INTERFACE,)
APART = (crk.PHASE_LOCAL_PLAIN, crk.PHASE_LOCAL_BLEND, crk.PHASE_INTERFACE)


def _nets(N):
    return [None] + ([crk.MLP.load(WEIGHTS)] if N == 3 and os.path.exists(WEIGHTS) else [])


@pytest.mark.parametrize("nx,ny,N,prec", MESHES, ids=IDS)
def test_one_launch_equals_two(nx, ny, N, prec):
    u1 = _state(nx, ny, N)
    for net in _nets(N):
        a, b = _solver(nx, ny, 1, N, prec, net), _solver(nx, ny, 2, N, prec, net)
        u1 = u1.to(a.dtype)
        u2 = torch.cat([u1, u1], dim=1)
        blended = (a.indicator(u1)[1] > 0).double().mean().item()
        assert 0.05 < blended < 0.95
        one, d1 = _run(a, u1, BOTH)
        two, d2 = _run(b, u2, BOTH)
        assert torch.equal(d1, d2)
        assert torch.equal(two[:, : nx * ny], one) and torch.equal(two[:, nx * ny:], one)
        # the phases issued separately, on both sides
        assert torch.equal(_run(a, u1, APART)[0], one)
        assert torch.equal(_run(b, u2, APART)[0], two)


@pytest.mark.parametrize("nx,ny,N,prec", MESHES, ids=IDS)
def test_large_meshes_take_two_launches(nx, ny, N, prec):
    """Above the limit the launch without the blending code leaves flagged tiles
    to the other, with the modal and with the learned indicator; below it
    one launch does all."""
    for net in _nets(N):
        for copies in (1, 2):
            s = _solver(nx, ny, copies, N, prec, net)
            u = torch.cat([_state(nx, ny, N).to(s.dtype)] * copies, dim=1)
            out, dt = torch.full(s.shape, -7.0, dtype=s.dtype, device="cuda"), s.new_dt()
            s.prepare(u, dt)
            s.advance(u, out, dt, phases=crk.PHASE_LOCAL_PLAIN)
            left = (out == -7.0).all(dim=0).all(dim=1)              # elements that the launch did not write
            blends = s.indicator(u)[1] > 0
            if copies == 1:
                assert not left.any()
            else:
                assert left[blends].all() and not left.all()
