"""The Jacobi diagonal where each column keeps its own sums (at least two voxels per cell in x and
y), at the grids where it can go wrong: cells of exactly two voxels, cells of mixed width, voxels on
a node (a weight of 0, which the sums divided by the weights leave to the general form), one cell in
all, one plane per cell, volumes narrower than a group and one column wider; and grids with cells of
a single voxel, which keep the general gather.  No regulariser, so that the image part is compared.
Tolerance 2e-6 (relative L2) against the float64 oracle: sums of squares of float32 products, a
rounding error of about 2^-24 times the square root of the roughly thirty operations of a product,
twice that for its square."""
import numpy as np
import pytest
import torch

from gpu_cases import DEV, blob_case, oracle_eval, rel_l2, to_dev
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu

CASES = [((32, 28, 24), (17, 15, 13)),    # two voxels per cell
         ((37, 31, 26), (16, 13, 9)),     # cells of two and three voxels
         ((33, 35, 17), (11, 15, 9)),     # voxels on nodes
         ((61, 29, 18), (16, 8, 19)),     # one plane per cell
         ((26, 22, 14), (2, 2, 2)),       # one cell
         ((31, 15, 130), (9, 5, 33)),     # one column and one row more than a group's own; chunks of many planes
         ((5, 4, 3), (2, 2, 2)),
         ((30, 14, 12), (8, 13, 4)),      # cells of one and two voxels in y: the general gather
         ((20, 18, 16), (21, 19, 17))]    # one voxel per cell


@pytest.mark.parametrize("distance", ["ngf", "ssd"])
@pytest.mark.parametrize("m,my", CASES, ids=lambda v: "x".join(map(str, v)))
def test_diagonal(m, my, distance):
    print(f"[gpu-case] diagonal march {m} {my} {distance}", flush=True)
    spec, R, T, u, probes = blob_case(8, m, my, h=(1.0, 1.2, 0.9), alpha=0.0, n_probes=0, distance=distance)
    ctx = mfr.Context(spec, DEV)
    ctx.set_images(to_dev(R), to_dev(T))
    d = ctx.jacobi_diag(to_dev(u))
    want = oracle_eval(spec, R, T, u, probes)["diag"]
    assert rel_l2(d.cpu().numpy(), want) <= 2e-6
    ctx.close()


def test_diagonal_keeps_a_bad_voxel_local():
    """A reference value that is not a number reaches the nodes its row and its neighbours' rows touch only."""
    spec, R, T, u, _ = blob_case(9, (48, 44, 40), (13, 12, 11), alpha=0.5, n_probes=0)
    bad = R.copy()
    bad[20, 21, 23] = np.nan
    ctx = mfr.Context(spec, DEV)
    tu, out = to_dev(u), []
    for r in (R, bad):
        ctx.set_images(to_dev(r), to_dev(T))
        out.append(ctx.jacobi_diag(tu))
    node = [v * (n - 1) // k for v, n, k in zip((20, 21, 23), spec.my[::-1], spec.m[::-1])]
    far = torch.ones(out[0].shape[1:], dtype=torch.bool, device=DEV)
    far[tuple(slice(max(n - 2, 0), n + 4) for n in node)] = False
    assert torch.equal(out[0][:, far], out[1][:, far])
    assert torch.isnan(out[1]).any()
    ctx.close()
