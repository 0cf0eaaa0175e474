"""The stencil pass's split into units (60 columns by a band of rows, one wave each or four).

- Against the oracle where the split has its edges: grids of one partial segment, of a segment and
  a few columns, units that do not fill their last workgroup, bands that do not divide the grid's
  rows, and rectangles on either side of the line between the two rules (8192 rows x segments).
- A member gives the same bits whether a unit is walked by four waves (a context that leaves the
  device room) or by one (an ensemble that does not), with and without a captured graph.
"""
import numpy as np
import pytest

from oracle import ccmsav_ref as R
from workloads import general_params, vesicle_member

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_10057_amd import ccmsav as C  # noqa: E402


def rectangle(nx, ny):
    """An ellipse three fifths of each side wide, in the middle of the grid."""
    p = general_params(nx, ny, 1)
    x = (np.arange(nx) + 0.5 - 0.5 * nx) / (0.3 * nx)
    y = (np.arange(ny) + 0.5 - 0.5 * ny) / (0.3 * ny)
    rho = np.hypot(x[None, :], y[:, None])
    phi = np.tanh((1.0 - rho) * 0.3 * min(nx, ny) * p["h"] / (np.sqrt(2.0) * p["eps"]))
    return p, phi, 0.9 + 0.1 * phi


@pytest.mark.parametrize("nx,ny", [(16, 16), (64, 16), (16, 128), (2048, 64), (4096, 16),
                                   (1024, 512), (512, 1024), (64, 4096), (4096, 128)])
def test_steps_match_the_oracle_at_the_edges_of_the_split(nx, ny):
    print(f"[case] {nx} x {ny}", flush=True)
    p, phi0, psi0 = rectangle(nx, ny)
    st = R.initial_state(phi0, psi0, p)
    with C.Context(p, phi0, psi0) as ctx:
        for _ in range(3):
            R.step(st)
            ctx.step(1)
        phi, psi = ctx.fields()
        sav, _ = ctx.savs()
    for got, ref in ((phi, st.phi), (psi, st.psi), (sav, st.sav)):
        assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("precision,graph", [("fp64", False), ("mixed", True)])
def test_one_wave_and_four_waves_per_unit_give_the_same_bits(precision, graph):
    # 2 segments x 4 bands x 4 waves per member: more than 2048 waves from 65 members on
    ms = [vesicle_member(64, 400 + i, dt=2.5e-8) for i in range(66)]
    print(f"[case] {len(ms)} members {precision} graph={graph}", flush=True)
    with C.Context.ensemble([m.params for m in ms], [m.phi0 for m in ms], [m.psi0 for m in ms],
                            precision, graph=graph) as many:
        many.step(9)
        for i in (0, 33, 65):
            with C.Context(ms[i].params, ms[i].phi0, ms[i].psi0, precision) as one:
                one.step(9)
                for a, b in zip((*many.fields(i), *many.savs(i)), (*one.fields(), *one.savs())):
                    assert np.array_equal(a, b), i
