"""The numerical flux of a face is one number: both elements that share it use
the same bits, so the totals telescope.

Degree 1 on unit elements (coefficients 2 D / dx = -2, 2 and 1 / (w dx) = 2) and
states that are constant in each element and differ by 1e-6 between elements:
the volume term cancels within an element, the surface term is 2 (F - f(u)),
which is small, so its rounding is some 2^-53 of 1e-6 while two values of F
would differ by 2^-53 of F.  The sum of the residual over all nodes is then the
sum of the roundings of each node's few additions of small terms (bound:
eight units of the largest residual per node and direction) unless an F is
double-valued.  In two dimensions the flow is along one axis: the residual adds
the directions one after the other, and the last bit in which the volume
term's two forms of f(u) differ, equal and opposite at the two nodes of a
line, would not survive the addition of another direction's flux."""
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


CASES = [("euler", 1, vol, 0) for vol in (0, 1, 2)] + [("euler", 2, vol, axis) for vol in (0, 1, 2) for axis in (0, 1)] + [
    ("mhd", 2, vol, axis) for vol in (0, 3) for axis in (0, 1)]


@pytest.mark.parametrize("seed", [1, 2])
@pytest.mark.parametrize("eq,dim,vol,axis", CASES)
def test_totals_telescope(eq, dim, vol, axis, seed):
    nx, ny = (96, 1) if dim == 1 else (16, 12)
    mhd = eq == "mhd"
    s = crk.Solver(dim=dim, nx=nx, ny=ny, x0=0.0, x1=float(nx), y0=0.0, y1=float(ny), degree=1, volume_flux=vol,
                   equation=crk.CRK_GLM_MHD if mhd else crk.CRK_EULER, gamma=5.0 / 3.0 if mhd else 1.4)
    M, E, NP = s.shape
    rng = np.random.default_rng(seed)
    # every conserved variable and every flux of order one, away from powers of two
    base = np.array([1.3, 0.9, 0.7, 5.1]) if dim == 2 else np.array([1.3, 0.9, 5.1])
    if mhd:
        base = np.array([1.3, 0.9, 0.7, 0.6, 5.1, 0.7, 0.6, 0.55, 0.3])
    if dim == 2:
        base[2 - axis] = 0.0                       # momentum along `axis` only
    u = base[:, None] * (1.0 + 1e-6 * rng.uniform(-1.0, 1.0, (M, E)))
    ug = torch.tensor(np.repeat(u[:, :, None], NP, axis=2), device="cuda")
    dt = torch.tensor([0.1, 2.5], dtype=torch.float64, device="cuda") if mhd else None
    r = s.fr_rhs(ug, crk.SURF_RUSANOV, dt).cpu().numpy()
    # sums in 80 bits: exact enough here
    for v in range(1 if mhd else M):
        total = abs(float(r[v].astype(np.longdouble).sum()))
        assert total <= 8 * dim * E * NP * 2.0 ** -53 * np.max(np.abs(r)), v


@pytest.mark.parametrize("degree", [2, 3, 4])
@pytest.mark.parametrize("eq,dim,vol,axis", CASES)
def test_totals_telescope_at_higher_degree(eq, dim, vol, degree, axis):
    """There the volume term of a constant state leaves a rounding of its own:
    it is measured in the middle of three equal elements, where the surface
    term vanishes, and taken off."""
    mhd = eq == "mhd"
    M = 9 if mhd else dim + 2
    base = np.array([1.3, 0.9, 0.7, 5.1]) if dim == 2 else np.array([1.3, 0.9, 5.1])
    if mhd:
        base = np.array([1.3, 0.9, 0.7, 0.6, 5.1, 0.7, 0.6, 0.55, 0.3])
    if dim == 2:
        base[2 - axis] = 0.0
    n = 48                                             # elements along the axis
    u = base[:, None] * (1.0 + 1e-6 * np.random.default_rng(degree).uniform(-1.0, 1.0, (M, n)))

    def residual(states):                              # [M, k] along the axis, constant across it -> [M, k, nodes]
        k = states.shape[1]
        nx, ny = (k, 1) if dim == 1 else ((k, 3) if axis == 0 else (3, k))
        s = crk.Solver(dim=dim, nx=nx, ny=ny, x0=0.0, x1=float(nx), y0=0.0, y1=float(ny), degree=degree, volume_flux=vol,
                       equation=crk.CRK_GLM_MHD if mhd else crk.CRK_EULER, gamma=5.0 / 3.0 if mhd else 1.4)
        if dim == 2:
            states = np.repeat(states[:, None, :], 3, 1) if axis == 0 else np.repeat(states[:, :, None], 3, 2)
        ug = torch.tensor(np.repeat(states.reshape(M, -1, 1), s.shape[2], axis=2), device="cuda")
        dt = torch.tensor([0.1, 2.5], dtype=torch.float64, device="cuda") if mhd else None
        r = s.fr_rhs(ug, crk.SURF_RUSANOV, dt).cpu().numpy()
        if dim == 1:
            return r
        return r.reshape(M, ny, nx, -1)[:, 1] if axis == 0 else r.reshape(M, ny, nx, -1)[:, :, 1]

    surface = residual(u).astype(np.longdouble) - residual(np.repeat(u, 3, axis=1))[:, 1::3]
    bound = 8 * dim * n * surface.shape[2] * 2.0 ** -53 * np.max(np.abs(surface))
    for v in range(1 if mhd else M):
        assert abs(float(surface[v].sum())) <= bound, v
