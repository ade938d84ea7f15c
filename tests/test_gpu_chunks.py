"""The z split of the voxel-tile march: volumes for which the derived split takes few planes per
group, and a workspace that only the split into longer chunks fits.  Tolerance 2e-6 (relative L2)
against the float64 oracle, as for the node-plane reduction (float32 sums, sqrt of the term count)."""
import ctypes

import pytest
import torch

from gpu_cases import DEV, blob_case, gpu_eval, oracle_eval, rel_l2, to_dev
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,my", [((24, 20, 5), (7, 6, 3)), ((30, 14, 23), (11, 6, 12)), ((61, 29, 33), (16, 9, 5)),
                                  ((20, 20, 64), (6, 6, 33))], ids=lambda v: "x".join(map(str, v)))
def test_derived_split(m, my):
    print(f"[gpu-case] derived split {m} {my}", flush=True)
    spec, R, T, u, probes = blob_case(6, m, my, alpha=0.3, n_probes=1)
    a, b = gpu_eval(spec, R, T, u, probes), oracle_eval(spec, R, T, u, probes)
    assert abs(a["J"] - b["J"]) <= 1e-6 * abs(b["J"])
    for k in ("grad", "diag"):
        assert rel_l2(a[k], b[k]) <= 2e-6, k
    assert rel_l2(a["hv"][0], b["hv"][0]) <= 2e-6


def test_smaller_workspace_takes_longer_chunks():
    spec, R, T, u, probes = blob_case(7, (64, 64, 24), (33, 33, 13), alpha=0.3, n_probes=1)
    tR, tT, tu, tp = (to_dev(a) for a in (R, T, u, probes[0]))
    ctx = mfr.Context(spec, DEV)
    ctx.set_images(tR, tT)
    h0, d0 = ctx.hess_vec(tu, tp), ctx.jacobi_diag(tu)
    lib, nbytes = mfr.load(), mfr.workspace_size(spec) * 3 // 4
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device=DEV)
    ptr = ws.data_ptr() + (-ws.data_ptr()) % 256
    h = ctypes.c_void_p()
    grid = mfr.make_grid(spec)
    assert lib.mfr_create(ctypes.byref(grid), None, ctypes.c_void_p(ptr), nbytes, ctypes.byref(h)) == 0
    try:
        vp = lambda t: ctypes.c_void_p(t.data_ptr())   # noqa: E731
        q, d = torch.empty_like(tp), torch.empty_like(tp)
        torch.cuda.synchronize()
        assert lib.mfr_set_images(h, vp(tR), vp(tT)) == 0
        assert lib.mfr_hess_vec(h, vp(tu), vp(tp), vp(q)) == 0
        assert lib.mfr_jacobi_diag(h, vp(tu), vp(d)) == 0
        torch.cuda.synchronize()
        assert rel_l2(q.cpu().numpy(), h0.cpu().numpy()) <= 2e-6
        assert rel_l2(d.cpu().numpy(), d0.cpu().numpy()) <= 2e-6
        small = ctypes.c_void_p()
        assert lib.mfr_create(ctypes.byref(grid), None, ctypes.c_void_p(ptr), nbytes // 4, ctypes.byref(small)) == -2
    finally:
        lib.mfr_destroy(h)
        ctx.close()
