"""Contexts in the least workspace that they accept: they take longer chunks and give the results of a full
workspace (2e-6 relative L2: float32 sums in another order, sqrt of the term count), without a write behind
their last byte."""
import ctypes

import pytest
import torch

from gpu_cases import DEV, blob_case, rel_l2, to_dev
from paper_1804_10541_amd import mfr
from test_gpu_plane import plane_case

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def derived_split():   # (another test's tile configuration may be in force)
    old = mfr.get_tile_config()
    mfr.set_tile_config(32, 16, 0, 0)
    yield
    mfr.set_tile_config(**old)


@pytest.mark.parametrize("m,my", [((24, 11, 146), (7, 4, 38)), ((64, 64, 24), (33, 33, 13)), ((33, 20, 70), (17, 11, 36)),
                                  ((206, 282, 1), (53, 72, 1)), ((300, 60, 1), (76, 31, 1))],
                         ids=lambda v: "x".join(map(str, v)))
def test_results_in_the_least_workspace(m, my):
    print(f"[gpu-case] least workspace {m} {my}", flush=True)
    if m[2] == 1:
        spec, R, T, u, probes = plane_case(3, m[:2], my[:2], n_probes=1)
    else:
        spec, R, T, u, probes = blob_case(3, m, my, alpha=0.3, n_probes=1)
    tR, tT, tu, tp = (to_dev(a) for a in (R, T, u, probes[0]))
    ctx = mfr.Context(spec, DEV)
    ctx.set_images(tR, tT)
    want = [ctx.gradient(tu, want_J=False)[0], ctx.hess_vec(tu, tp), ctx.jacobi_diag(tu)]
    J = ctx.objective(tu)[0]
    lib, h, grid, full = mfr.load(), ctypes.c_void_p(), mfr.make_grid(spec), mfr.workspace_size(spec)
    ws = torch.full((full + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    off = -ws.data_ptr() % 256

    def create(n):
        return lib.mfr_create(ctypes.byref(grid), None, ctypes.c_void_p(ws.data_ptr() + off), n, ctypes.byref(h))

    lo, nbytes = 0, full   # refused, accepted
    while nbytes - lo > 256:
        mid = (lo + nbytes) // 512 * 256
        if create(mid) == 0:
            lib.mfr_destroy(h)
            nbytes = mid
        else:
            lo = mid
    assert nbytes < full
    ws.fill_(0xA5)
    torch.cuda.synchronize()
    assert create(nbytes) == 0
    try:
        vp = lambda t: ctypes.c_void_p(t.data_ptr())   # noqa: E731
        got = [torch.empty_like(t) for t in want]
        Js = ctypes.c_double()
        torch.cuda.synchronize()
        assert lib.mfr_set_images(h, vp(tR), vp(tT)) == 0
        assert lib.mfr_gradient(h, vp(tu), None, vp(got[0])) == 0
        assert lib.mfr_hess_vec(h, vp(tu), vp(tp), vp(got[1])) == 0
        assert lib.mfr_jacobi_diag(h, vp(tu), vp(got[2])) == 0
        assert lib.mfr_objective(h, vp(tu), ctypes.byref(Js), None, None) == 0
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert rel_l2(a.cpu().numpy(), b.cpu().numpy()) <= 2e-6
        assert abs(Js.value - J) <= 1e-6 * abs(J)
        assert bool((ws[:off] == 0xA5).all()) and bool((ws[off + nbytes:] == 0xA5).all())
    finally:
        lib.mfr_destroy(h)
        ctx.close()
