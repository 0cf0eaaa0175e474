"""The row DCT's bands of rows on strips of every line length that takes several rounds of field
pairs: the FP32 kernel loads the next round's rows while the current one is transformed (not the
full band at 8192 points), the FP64 kernel round by round. Both bands give the same bits, as every
value goes through the same operations in the same order."""
import numpy as np
import pytest

from test_gpu_stencil_units import C, rectangle

pytestmark = pytest.mark.gpu


def states(p, phi0, psi0, precision, band):
    with C.Context(p, phi0, psi0, precision) as ctx:
        ctx.set_launch_variants(row_dct=band)
        ctx.step(3)
        return (*ctx.fields(), *ctx.savs())


@pytest.mark.parametrize("nx", [256, 512, 1024, 2048, 4096, 8192])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_both_bands_give_the_same_bits(nx, precision):
    print(f"[case] {nx} x 16 {precision}", flush=True)
    p, phi0, psi0 = rectangle(nx, 16)
    a, b = (states(p, phi0, psi0, precision, band) for band in (0, 1))
    for u, v in zip(a, b):
        assert np.isfinite(u).all() and np.array_equal(u, v)
