"""The Gram pass transforms two fields of a column as one complex line: its inner products from the
row-transformed fields that it reads, against the same products in extended precision, for pairs of
very different sizes (Q~ beside K~ with osmotic weights of 1e5, 1e-6 and zero: thousands of times
larger, smaller, and no second field at all), on columns of every length.

Both are taken from the context's workspace (regions of the layout in order: six state fields, the
stencil fields, the row-transformed fields, the solved ones, the two arrays of partial sums). The bar
is that of transforms whose errors are relative to the field itself: unit roundoff u, elements off by
u log2(N) times their column's root mean square (twice what an FFT of N points reaches on average),
independently of each other, so that a sum of weighted products has the standard deviation
sqrt(sum w^2 (dx^2 y^2 + dy^2 x^2)); four of these, and 8 u of the sum of the products' sizes for
constants that are the same in all elements."""
import numpy as np
import pytest
from scipy import fft

from test_gpu_stencil_units import rectangle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_10057_amd import ccmsav as C  # noqa: E402

F, S, H, Q, K, G, L, P = range(8)
CHI = [(F, S), (F, H), (F, Q), (F, K), (S, S), (S, H), (S, Q), (S, K), (H, H), (H, Q), (H, K),
       (Q, Q), (Q, K), (K, K)]
ZETA = [(P, G), (P, L)]


def regions(nx, ny, size):
    """Offsets of mid, part2, lamx and lamy in the workspace (16-row units of 60 columns)."""
    up = lambda x: (x + 255) // 256 * 256
    field = (nx // 2) * (2 * ny + 1056 // size) * size
    mid = up(48 * nx * ny) + up(8 * nx * ny * size)
    part1 = mid + up(8 * field) + up(2 * field)
    part2 = part1 + up((nx + 59) // 60 * (ny // 16) * 128)
    lamx = part2 + up(nx * 128) + up(ny * 80)
    return mid, part2, lamx, lamx + up(nx * 8)


def row_transformed(ws, mid, nx, ny, size):
    """The eight fields [slot][y][kx] from their strips."""
    stride = 2 * ny + 1056 // size
    if size == 8:
        raw = ws[mid:mid + 8 * (nx // 2) * stride * 8].view(np.float64).reshape(8, nx // 2, stride)
        return raw[:, :, :2 * ny].reshape(8, nx // 2, ny, 2).transpose(0, 2, 1, 3).reshape(8, ny, nx)
    stride = 4 * ny + 1056 // size
    raw = ws[mid:mid + 4 * (nx // 2) * stride * 4].view(np.float32).reshape(4, nx // 2, stride)
    raw = raw[:, :, :4 * ny].reshape(4, nx // 2, ny, 2, 2).transpose(0, 4, 2, 1, 3)
    raw = raw.reshape(8, ny, nx)                    # pairs (F, P), (S, H), (Q, K), (G, L)
    return raw[[0, 2, 3, 4, 5, 6, 7, 1]]


@pytest.mark.parametrize("gamma", [1e5, 1e-6, 0.0])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("nx,ny", [(64, 16), (64, 64), (64, 128), (64, 512), (64, 1024),
                                   (16, 2048), (16, 4096), (16, 8192)])
def test_inner_products_are_as_accurate_as_each_field(nx, ny, precision, gamma):
    print(f"[case] {nx} x {ny} {precision} gamma {gamma}", flush=True)
    p, phi0, psi0 = rectangle(nx, ny)
    p = dict(p, gamma_in=gamma, gamma_out=gamma, beta_in=1.0, beta_out=1.0)
    ws = torch.zeros(C.workspace_bytes(p, C.PRECISIONS[precision]), dtype=torch.uint8,
                     device="cuda")
    with C.Context(p, phi0, psi0, precision, workspace=ws) as ctx:
        ctx.step(3)
        ctx.sync()
        ws = ws.cpu().numpy()
    size = 4 if precision == "mixed" else 8
    mid, part2, lamx, lamy = regions(nx, ny, size)
    got = ws[part2:part2 + nx * 128].view(np.float64).reshape(nx, 16).astype(np.longdouble).sum(0)
    lam = (ws[lamy:lamy + 8 * ny].view(np.float64).astype(np.longdouble)[:, None]
           + ws[lamx:lamx + 8 * nx].view(np.float64)[None, :])
    hat = fft.dct(row_transformed(ws, mid, nx, ny, size).astype(np.longdouble), axis=1, norm="ortho")
    alpha, r2 = 1.5 / p["dt"], np.sqrt(2.0)
    c1 = alpha + p["M_phi"] * p["gamma_surf"] * 3 * r2 * p["beta"] / (4 * p["eps"])
    c2 = p["M_phi"] * (p["gamma_surf"] * 3 * r2 * p["eps"] / 4 + p["theta"])
    c3 = p["M_phi"] * p["gamma_bend"] * 3 * r2 * p["eps"] / 8
    chi, zeta = 1.0 / (c1 + lam * (c2 + c3 * lam)), 1.0 / (alpha + p["lam"] * lam)
    u = 2.0 ** (-24 if size == 4 else -53)
    dev = u * np.log2(ny) * np.sqrt((hat ** 2).mean(1, keepdims=True))
    assert np.isfinite(got.astype(float)).all()
    for i, (x, y) in enumerate(CHI + ZETA):
        w = chi if i < len(CHI) else zeta
        a, b, da, db = hat[x], hat[y], dev[x], dev[y]
        bar = (4.0 * np.sqrt((w ** 2 * (da ** 2 * b ** 2 + db ** 2 * a ** 2)).sum())
               + 8.0 * u * (w * abs(a * b)).sum())
        err = abs(got[i] - (w * a * b).sum())
        assert err <= bar, ("FSHQKGLP"[x] + "FSHQKGLP"[y], float(err / bar), float(err))
