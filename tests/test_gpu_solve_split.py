"""The standalone solve where its launches change: the smallest grids, both sides of the line
between one workgroup per strip and one per strip and operator (65536 threads of the strips), and
the longest lines, against the plain spectral solve; Dirichlet rows and columns of both parities."""
import numpy as np
import pytest

from oracle import ccmsav_ref as R
from parity_util import rel_linf
from workloads import general_params

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_10057_amd import ccmsav as C  # noqa: E402


@pytest.mark.parametrize("bc", ["neumann", "dirichlet"])
@pytest.mark.parametrize("nx,ny", [(16, 16), (16, 64), (1024, 512), (2048, 512), (256, 2048),
                                   (256, 4096), (8192, 32), (32, 8192)])
def test_solves_on_both_sides_of_the_split(nx, ny, bc):
    print(f"[case] {nx} x {ny} {bc}", flush=True)
    params = general_params(nx, ny, 2)
    p = R.Params.from_dict(params)
    rng = np.random.default_rng(nx + ny)
    rhs = rng.standard_normal((ny, nx))
    lam = (R.neumann_lap_eigs if bc == "neumann" else R.dirichlet_lap_eigs)(nx, ny, p.h)
    solve = R.spectral_solve if bc == "neumann" else R.spectral_solve_dirichlet
    C1, C2, C3 = R.chi_coefficients(p, 1.5 / p.dt)
    want = (solve(rhs, C1 - C2 * lam + C3 * lam ** 2), solve(rhs, 1.5 / p.dt - p.lam * lam))
    dev = torch.from_numpy(rhs).cuda()
    chi, zeta = torch.empty_like(dev), torch.empty_like(dev)
    phi = torch.full_like(dev, 0.3)
    with C.Context(params, phi, phi + 0.8) as ctx:
        ctx.elliptic_solve(dev, chi, zeta, bc=bc)
        for got, ref in zip((chi, zeta), want):
            assert rel_linf(got.cpu().numpy(), ref) <= 1e-12
        # one output only, written over the right-hand side
        ctx.elliptic_solve(dev, None, dev, bc=bc)
        assert rel_linf(dev.cpu().numpy(), want[1]) <= 1e-12
