"""Field queries to device memory (one kernel with the error bits) give the bytes that queries to
host memory give: both fields, either one alone, members of several grids, and destinations at an
8-byte offset; a state that is not finite is reported either way."""
import ctypes

import numpy as np
import pytest

from workloads import vesicle_member

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_10057_amd import ccmsav as C  # noqa: E402


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("offset", [0, 1])
def test_device_and_host_queries_agree(precision, offset):
    ms = [vesicle_member(n, 70 + n, dt=2.5e-8) for n in (16, 64, 64, 256)]
    with C.Context.ensemble([m.params for m in ms], [m.phi0 for m in ms], [m.psi0 for m in ms],
                            precision) as ctx:
        ctx.step(3)
        for i, m in enumerate(ms):
            print(f"[case] member {i} {precision} offset {offset}", flush=True)
            ref = ctx.fields(i)
            cells = m.phi0.size
            buf = torch.full((2, cells + 2), -7.0, device="cuda", dtype=torch.float64)
            phi, psi = (buf[f, offset:offset + cells].view(m.phi0.shape) for f in (0, 1))
            ctx.fields_into(phi, None, i)
            assert (psi == -7.0).all()
            ctx.fields_into(None, psi, i)
            for got, want in zip((phi, psi), ref):
                assert np.array_equal(got.cpu().numpy(), want)
            buf[:, offset:offset + cells] = 0.0
            ctx.fields_into(phi, psi, i)
            for got, want in zip((phi, psi), ref):
                assert np.array_equal(got.cpu().numpy(), want)
            rest = torch.cat([buf[:, :offset], buf[:, offset + cells:]], 1)
            assert (rest == -7.0).all()


def test_a_device_query_reports_a_state_that_is_not_finite():
    m = vesicle_member(64, 5)
    with C.Context(dict(m.params, dt=1e300), m.phi0, m.psi0) as ctx:
        ctx.step(3)
        phi = torch.empty(64, 64, device="cuda", dtype=torch.float64)
        with pytest.raises(C.CcmsavError) as host:
            ctx.fields()
        with pytest.raises(C.CcmsavError) as dev:
            ctx.fields_into(phi, phi.clone())
        assert dev.value.code == host.value.code


def test_contexts_beyond_the_pinned_words_query_as_well():
    # 256 contexts hold pinned words, further ones copy; closed ones give theirs back
    m = vesicle_member(16, 9, dt=2.5e-8)
    phi, psi = (torch.empty(16, 16, device="cuda", dtype=torch.float64) for _ in range(2))
    ctxs = [C.Context(m.params, m.phi0, m.psi0) for _ in range(260)]
    for ctx in ctxs[::2]:
        ctx.close()
    ctxs[::2] = [C.Context(m.params, m.phi0, m.psi0) for _ in ctxs[::2]]
    for ctx in ctxs:
        ctx.step(1)
    ref = ctxs[0].fields()
    for ctx in ctxs:
        phi.zero_()
        psi.zero_()
        ctx.fields_into(phi, psi)
        assert all(np.array_equal(a.cpu().numpy(), b) for a, b in zip((phi, psi), ref))
        ctx.close()


def hip():
    """The HIP runtime that the process runs on."""
    return ctypes.CDLL([line.split()[-1] for line in open("/proc/self/maps")
                        if "libamdhip64.so" in line][0])


def test_a_device_output_that_does_not_hold_the_field_is_refused():
    # an allocation of 12 MB for fields of 32 MB
    m = vesicle_member(64, 3)
    p = dict(m.params, nx=2048, ny=2048)
    phi = torch.full((2048, 2048), 0.3, device="cuda", dtype=torch.float64)
    marks = np.full(3 << 19, -7.0)
    small, size = ctypes.c_void_p(), ctypes.c_size_t(marks.nbytes)
    assert hip().hipMalloc(ctypes.byref(small), size) == 0
    assert hip().hipMemcpy(small, ctypes.c_void_p(marks.ctypes.data), size, 1) == 0
    with C.Context(p, phi, phi + 0.8) as ctx:
        ctx.step(1)
        query = C.load().ccmsav_get_fields_m
        for outs in ((small, None), (None, small), (phi.data_ptr(), small)):
            assert query(ctx._h, 0, *outs) == -3            # EHIP
            hip().hipGetLastError()                         # the runtime's refusal
            back = np.zeros_like(marks)
            assert hip().hipMemcpy(ctypes.c_void_p(back.ctypes.data), small, size, 2) == 0
            assert np.array_equal(back, marks)
        got = torch.empty_like(phi)
        ctx.fields_into(got, None)
        assert np.array_equal(got.cpu().numpy(), ctx.fields()[0])
    assert hip().hipFree(small) == 0


@pytest.mark.parametrize("shift", [0, 1, 777, 2048, 4095, -1, -2048])
def test_outputs_that_overlap_hold_psi(shift):
    # psi starts `shift` values behind phi and is written last
    m = vesicle_member(64, 8, dt=2.5e-8)
    with C.Context(m.params, m.phi0, m.psi0) as ctx:
        ctx.step(2)
        want_phi, want_psi = (torch.from_numpy(f.ravel()) for f in ctx.fields())
        for _ in range(20):
            buf = torch.zeros(3 * 4096, device="cuda", dtype=torch.float64)
            ctx.fields_into(buf[4096:8192], buf[4096 + shift:8192 + shift])
            want = torch.zeros(3 * 4096, dtype=torch.float64)
            want[4096:8192] = want_phi
            want[4096 + shift:8192 + shift] = want_psi
            assert torch.equal(buf.cpu(), want)


def test_an_error_that_another_call_left_does_not_fail_the_query():
    m = vesicle_member(64, 11, dt=2.5e-8)
    with C.Context(m.params, m.phi0, m.psi0) as ctx:
        ctx.step(2)
        want = ctx.fields()
        phi, psi = (torch.zeros(64, 64, device="cuda", dtype=torch.float64) for _ in range(2))
        host = np.zeros((64, 64))
        torch.cuda.synchronize()
        # a device number that does not exist sets the error state
        assert hip().hipSetDevice(9999) != 0
        ctx.fields_into(phi, psi)
        assert all(np.array_equal(a.cpu().numpy(), b) for a, b in zip((phi, psi), want))
        ctx.fields_into(host, None)
        assert np.array_equal(host, want[0])
    hip().hipGetLastError()
