"""The 5x5 kernel reduces as many rows of partial sums as the grid has columns (Gram pass) and stencil
units, however few cells that are: wide and tall rectangles split them over workgroups as large squares
do. Its time, the least of several runs, is within half as much again of that at 1024^2, where it is a
matter of launch and latency; by one workgroup, the rows of 4096 and 8192 columns take two to four
times as long. The steps' results are checked against the oracle where the split has its edges."""
import numpy as np
import pytest

from oracle import ccmsav_ref as R
from parity_util import rel_linf
from test_gpu_stencil_units import C, rectangle

pytestmark = pytest.mark.gpu


def solve_ms(nx, ny):
    p, phi, psi = rectangle(nx, ny)
    with C.Context(p, phi, psi, "mixed") as ctx:
        ctx.step(3)
        return min(ctx.profile_steps(20)["solve5"] for _ in range(5))


def test_time_follows_the_rows_of_partials():
    square = solve_ms(1024, 1024)
    for nx, ny in ((4096, 16), (8192, 64), (64, 8192)):
        ms = solve_ms(nx, ny)
        print(f"[case] {nx} x {ny}: {1e3 * ms:.1f} us, 1024^2: {1e3 * square:.1f} us", flush=True)
        assert ms <= 1.5 * square, (nx, ny, ms, square)


@pytest.mark.parametrize("nx,ny", [(512, 512), (512, 1024), (1024, 16), (1024, 256), (2048, 16),
                                   (64, 1024)])
def test_steps_match_the_oracle(nx, ny):
    print(f"[case] {nx} x {ny}", flush=True)
    p, phi0, psi0 = rectangle(nx, ny)
    st = R.initial_state(phi0, psi0, p)
    with C.Context(p, phi0, psi0) as ctx:
        for _ in range(3):
            R.step(st)
            ctx.step(1)
        phi, psi = ctx.fields()
        savs = ctx.savs()[0]
    assert max(rel_linf(phi, st.phi), rel_linf(psi, st.psi)) <= 1e-12
    assert rel_linf(np.array(savs), np.array(st.sav)) <= 1e-12
