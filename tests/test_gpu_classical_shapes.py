"""The classical scheme's conjugate gradient kernels at the sizes where their work is cut differently:
grids narrower than a wave's 64 columns, one and several segments of 64 columns, the row kernels'
longest lines (thin rectangles of 4096 and 8192 columns, and of as many rows), and a grid of more
units of 64 columns by four rows than the product kernel has waves (2048^2: 16384 units, 8192 waves).

Bars, from runs of the oracle alone: rectangles against its PCG trajectory (same tolerance 1e-12) at
1e-11 (its one-ulp envelope is below 4e-15; a solve that stopped an iteration later would move the
result by its distance from the direct solve, up to 9.9e-12), against its direct solve at
max(1e-11, 3 x the distance of its own PCG run), iterations within one; 2048^2 after one step against
its PCG at 1e-12 (50 x its distance from a run with tolerance 1e-14, 1.9e-14)."""
from types import SimpleNamespace

import pytest

from parity_util import rel_linf
from test_gpu_classical import gpu_run, note, oracle_run
from test_gpu_stencil_units import rectangle
from workloads import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(16, 16), (16, 128), (32, 256), (64, 16), (128, 32), (2048, 32),
                                   (4096, 16), (16, 4096), (8192, 16), (16, 8192)])
def test_rectangles_match_the_oracle(nx, ny):
    note(f"classical {nx} x {ny}, 3 steps")
    p, phi0, psi0 = rectangle(nx, ny)
    m = SimpleNamespace(params=p, phi0=phi0, psi0=psi0)
    ref, direct, got = oracle_run(m, 3), oracle_run(m, 3, solver="direct"), gpu_run(m, 3)
    for k in range(4):
        errs = [rel_linf(got[k][i], ref[k][i]) for i in range(3)]
        errs_d = [rel_linf(got[k][i], direct[k][i]) for i in range(3)]
        tol_d = max(1e-11, 3.0 * max(rel_linf(ref[k][i], direct[k][i]) for i in range(3)))
        assert max(errs) <= 1e-11, (k, errs)
        assert max(errs_d) <= tol_d, (k, errs_d, tol_d)
        if k:
            assert all(abs(a - b) <= 1 for a, b in zip(got[k][3], ref[k][3])), (k, got[k][3])


def test_more_units_than_waves():
    m = make_workload("vesicle1024", 2048)[0]
    note("classical 2048^2, 1 step")
    ref, got = oracle_run(m, 1), gpu_run(m, 1)
    errs = [rel_linf(got[1][i], ref[1][i]) for i in range(3)]
    note(f"  {max(errs):.2e}, iterations {got[1][3]}")
    assert max(errs) <= 1e-12, errs
    assert all(abs(a - b) <= 1 for a, b in zip(got[1][3], ref[1][3])), got[1][3]
