"""Values near the ends of the float32 range in the voxel-tile kernel.  A sum over x of finite columns
that overflows stays with the nodes it belongs to: the zero weights of the reduction's second product
must not carry it over the tile."""
import numpy as np
import pytest
import torch

from gpu_cases import DEV, blob_case, to_dev
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu


def test_overflowing_sum_stays_local():
    m, my = (40, 24, 20), (11, 7, 6)
    spec, R, T, u, _ = blob_case(4, m, my, alpha=0.0, n_probes=0, distance="ssd")
    T = np.broadcast_to(np.arange(m[0], dtype=np.float32), T.shape).copy()   # derivative 1 along x
    ctx = mfr.Context(spec, DEV)
    ctx.set_images(to_dev(R), to_dev(T))
    tu = to_dev(u * 0.0)
    near = np.zeros(my[::-1], dtype=bool)
    near[1:5, 2:5, 3:8] = True   # the nodes of p and one further
    seen = 0
    for e in range(120, 128):    # from no overflow to overflowing columns
        p = np.zeros((3,) + my[::-1], dtype=np.float32)
        p[0, 2:4, 3, 4:7] = 2.0 ** e
        q = ctx.hess_vec(tu, to_dev(p))
        torch.cuda.synchronize()
        q = q.cpu().numpy()
        assert np.isfinite(q[:, ~near]).all(), e
        seen += not np.isfinite(q).all()
    assert 0 < seen < 8
    ctx.close()
