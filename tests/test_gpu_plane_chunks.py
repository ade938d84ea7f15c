"""The row split of the two-dimensional march: the derived split against chunks of 16 and of 5 rows,
which the other tests hold against the float64 oracle, for images of one and more x tiles, fewer rows
than a chunk and node rows that three chunks hold.  Tolerance 2e-6 (relative L2; float32 sums in
another order, sqrt of the term count), the objective 1e-6."""
import ctypes

import pytest
import torch

from gpu_cases import DEV, rel_l2, to_dev
from paper_1804_10541_amd import mfr
from synth import GridSpec
from test_gpu_plane import plane_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,my", [((40, 30), (11, 9)), ((300, 41), (76, 8)), ((255, 9), (65, 4)), ((20, 3), (6, 2)),
                                  ((64, 64), (33, 33))], ids=lambda v: "x".join(map(str, v)))
def test_derived_rows(m, my):
    print(f"[gpu-case] plane rows {m} {my}", flush=True)
    spec, R, T, u, probes = plane_case(3, m, my, n_probes=1)
    old, out = mfr.get_tile_config(), []
    try:
        for rows in (0, 16, 5):
            mfr.set_tile_config(32, 16, rows, 0)
            ctx = mfr.Context(spec, DEV)
            ctx.set_images(to_dev(R), to_dev(T))
            tu = to_dev(u)
            g, J = ctx.gradient(tu)
            out.append((J, g.cpu().numpy(), ctx.hess_vec(tu, to_dev(probes[0])).cpu().numpy(),
                        ctx.jacobi_diag(tu).cpu().numpy()))
            ctx.close()
    finally:
        mfr.set_tile_config(**old)
    for o in out[1:]:
        assert abs(o[0] - out[0][0]) <= 1e-6 * abs(out[0][0])
        for a, b in zip(o[1:], out[0][1:]):
            assert rel_l2(a, b) <= 2e-6


@pytest.mark.parametrize("m,my,nbytes", [((6, 3, 2), (4, 3, 2), 29184), ((24, 11, 146), (7, 4, 38), 444928),
                                         ((4, 8, 8), (5, 9, 9), 83200), ((206, 282, 1), (53, 72, 1), 732672)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_workspace_sizes_of_longer_chunks_are_still_taken(m, my, nbytes):
    """Sizes that were asked for before the split into short chunks: such a workspace gets long ones."""
    lib = mfr.load()
    grid = mfr.make_grid(GridSpec(m=m, h=(1.0, 1.0, 1.0), my=my, tau=0.1, rho=0.1, alpha=1.0))
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device=DEV)
    h = ctypes.c_void_p()
    ptr = ws.data_ptr() + (-ws.data_ptr()) % 256
    assert lib.mfr_create(ctypes.byref(grid), None, ctypes.c_void_p(ptr), nbytes, ctypes.byref(h)) == 0
    lib.mfr_destroy(h)
