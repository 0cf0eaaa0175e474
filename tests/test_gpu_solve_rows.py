"""The standalone solve's FP32 row transform is as accurate in each row as that row allows: beside rows
a million times larger, a row's coefficients (in the context's workspace behind the state and stencil
fields) agree with the extended-precision DCT of the same row, rounded to FP32, within six times
u log2(nx) of the row's root mean square (twice what an FFT of nx points reaches on average)."""
import numpy as np
import pytest
from scipy import fft

from workloads import general_params

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_10057_amd import ccmsav as C  # noqa: E402


@pytest.mark.parametrize("bc", ["neumann", "dirichlet"])
@pytest.mark.parametrize("nx,ny", [(16, 16), (64, 32), (512, 16), (1024, 16), (4096, 16), (8192, 16)])
def test_small_rows_keep_their_digits(nx, ny, bc):
    print(f"[case] {nx} x {ny} {bc}", flush=True)
    p = general_params(nx, ny, 2)
    rows = np.random.default_rng(nx).standard_normal((ny, nx))
    rows *= np.where(np.arange(ny) % 2, 1e-6, 1.0)[:, None]
    rows = rows.astype(np.float32).astype(float)
    dev = torch.from_numpy(rows).cuda()
    chi, zeta = torch.empty_like(dev), torch.empty_like(dev)
    ws = torch.zeros(C.workspace_bytes(p, C.MIXED), dtype=torch.uint8, device="cuda")
    phi = torch.full_like(dev, 0.3)
    with C.Context(p, phi, phi + 0.8, "mixed", workspace=ws) as ctx:
        ctx.elliptic_solve(dev, chi, zeta, bc=bc)
        torch.cuda.synchronize()
        ws = ws.cpu().numpy()
    up = lambda x: (x + 255) // 256 * 256
    mid, stride = up(48 * nx * ny) + up(32 * nx * ny), 2 * ny + 264
    got = ws[mid:mid + (nx // 2) * stride * 4].view(np.float32).reshape(nx // 2, stride)
    got = got[:, :2 * ny].reshape(nx // 2, ny, 2).transpose(1, 0, 2).reshape(ny, nx)
    sign = 1.0 if bc == "neumann" else 1.0 - 2.0 * (np.add.outer(np.arange(ny), np.arange(nx)) % 2)
    want = fft.dct((rows * sign).astype(np.longdouble), axis=1, norm="ortho")
    bar = 6 * 2.0 ** -24 * np.log2(nx) * np.sqrt((want ** 2).mean(1, keepdims=True))
    worst = float((abs(got - want) / bar).max())
    assert worst <= 1.0, worst
