"""Values near the ends of the float32 range in the voxel-tile kernel.  A sum over x of finite columns
that overflows stays with the nodes it belongs to: the zero weights of the reduction's second product
must not carry it over the tile.  And the NGF derivatives do not change when images and edge parameters
are scaled together, down and up to gradients whose squares still are normal floats: tolerance 2e-6
(relative L2, as for the kernel's rows against the oracle; the scaling by a power of two itself is exact)."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_cases import DEV, blob_case, rel_l2, to_dev
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


@pytest.mark.parametrize("e", [-57, 57])
@pytest.mark.parametrize("amp", [1e-3, 1e3])
def test_scaled_images(e, amp):
    print(f"[gpu-case] images and edge parameters times 2^{e}, direction times {amp}", flush=True)
    spec, R, T, u, probes = blob_case(5, (40, 33, 21), (11, 9, 6), alpha=0.3, n_probes=1)
    out = []
    for k in (0, e):
        f = np.float32(2.0 ** k)
        ctx = mfr.Context(dataclasses.replace(spec, tau=spec.tau * 2.0 ** k, rho=spec.rho * 2.0 ** k), DEV)
        ctx.set_images(to_dev(R * f), to_dev(T * f))
        tu, tp = to_dev(u), to_dev(probes[0] * np.float32(amp))
        g, J = ctx.gradient(tu)
        out.append((J, g.cpu().numpy(), ctx.hess_vec(tu, tp).cpu().numpy()))
        torch.cuda.synchronize()
        ctx.close()
    assert abs(out[1][0] - out[0][0]) <= 1e-6 * abs(out[0][0])
    for a, b in zip(out[1][1:], out[0][1:]):
        assert rel_l2(a, b) <= 2e-6
