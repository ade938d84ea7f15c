"""The reduction of a finished P^T node plane on the matrix cores (voxel-tile kernel): node blocks
around the edges of its 16 x 16 node tiles, and an infinite or NaN voxel, whose zero conversion
weights must not carry it to the other nodes of a tile.

Tolerance 2e-6 (relative L2) against the float64 oracle: float32 products and sums of up to a few
hundred terms per node, rounding errors growing like the square root of their number (6e-8 x 16),
and the few float32 operations per voxel before them."""
import numpy as np
import pytest
import torch

from gpu_cases import DEV, blob_case, gpu_eval, oracle_eval, rel_l2, to_dev
from oracle import Grid
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu


# 32 x 16 columns per group (30 x 14 own): node columns per group from 2 to 33, rows from 2 to 17
@pytest.mark.parametrize("distance", ["ngf", "ssd"])
@pytest.mark.parametrize("m,my", [((31, 17, 9), (2, 2, 2)), ((62, 30, 12), (31, 16, 7)), ((60, 29, 10), (29, 15, 6)),
                                  ((64, 33, 11), (34, 18, 6)), ((40, 20, 7), (41, 21, 8)), ((33, 16, 5), (18, 17, 6))],
                         ids=lambda v: "x".join(map(str, v)))
def test_node_tiles(m, my, distance):
    print(f"[gpu-case] tile reduce {m} {my} {distance}", flush=True)
    spec, R, T, u, probes = blob_case(9, m, my, alpha=0.2, n_probes=1, distance=distance)
    a, b = gpu_eval(spec, R, T, u, probes, diag=False), oracle_eval(spec, R, T, u, probes, diag=False)
    assert rel_l2(a["grad"], b["grad"]) <= 2e-6
    assert rel_l2(a["hv"][0], b["hv"][0]) <= 2e-6


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_voxel_stays_local(bad):
    m, my = (40, 24, 20), (11, 7, 6)
    spec, R, T, u, probes = blob_case(4, m, my, alpha=0.0, n_probes=1)
    z, y, x = 9, 6, 14   # inside one group's own columns
    R[z, y, x] = bad
    ctx = mfr.Context(spec, DEV)
    ctx.set_images(to_dev(R), to_dev(T))
    g, _ = ctx.gradient(to_dev(u), want_J=False)
    h = ctx.hess_vec(to_dev(u), to_dev(probes[0]))
    torch.cuda.synchronize()
    g, h = g.cpu().numpy(), h.cpu().numpy()
    ctx.close()
    # rows of dr within one voxel see it, their columns lie one voxel further
    far = np.ones((my[2], my[1], my[0]), dtype=bool)
    grid = Grid.from_spec(spec)
    idx = []
    for k, c in enumerate((x, y, z)):
        n0, _ = grid.conversion_1d(k, np.arange(c - 2, c + 3))
        idx.append((n0.min(), n0.max() + 1))
    far[idx[2][0]:idx[2][1] + 1, idx[1][0]:idx[1][1] + 1, idx[0][0]:idx[0][1] + 1] = False
    assert np.isnan(g).any() and np.isnan(h).any()
    assert np.isfinite(g[:, far]).all() and np.isfinite(h[:, far]).all()
