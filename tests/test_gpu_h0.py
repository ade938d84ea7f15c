"""The cosine transforms of the initial-matrix solve on the matrix cores, at the
edges of their tiles: half lengths around a tile of 16 rows, odd and even lengths,
lines that are no multiple of a group's 64, an axis of several row groups, and x
axes on both sides of the longest one that is transformed there and back in one
kernel.

Tolerance: each of the six orthonormal transforms sums at most H = ceil(n/2)
float32 products, a relative error of about sqrt(H) 2^-24 of its output's norm,
and the division weighs frequencies by at most kappa = max/min of the
denominators: kappa 6 sqrt(H) 2^-24, with gamma chosen so that kappa = 3."""
import math

import numpy as np
import pytest
import torch

from gpu_cases import DEV, rel_l2, to_dev
from oracle import Grid, lbfgs, plane
from paper_1804_10541_amd import mfr
from synth import GridSpec

pytestmark = pytest.mark.gpu

NODES = [(2, 3, 2), (3, 2, 5), (31, 6, 17), (32, 33, 4), (4, 64, 65), (129, 7, 6), (255, 5, 4), (256, 4, 3),
         (257, 4, 5), (258, 3, 4), (6, 300, 5), (5, 4, 257), (33, 18, 1), (257, 19, 1)]


@pytest.mark.parametrize("my", NODES, ids=["x".join(map(str, n)) for n in NODES])
def test_h0_solve_at_tile_edges(my):
    print(f"[gpu-case] h0 tile edges {my}", flush=True)
    flat = my[2] == 1
    m = tuple(max(k - 1, 2) for k in my[:2]) + (1 if flat else max(my[2] - 1, 2),)
    spec = GridSpec(m=m, h=(1.0, 1.0, 1.0), my=my, tau=0.1, rho=0.1, alpha=0.5)
    hy = [mk / (nk - 1) for mk, nk in zip(m, my) if nk > 1]
    lmax = sum(4.0 / s ** 2 for s in hy)
    gamma = 2.0 * spec.alpha * math.prod(hy) * lmax ** 2 / 2.0
    H = (max(my) + 1) // 2
    tol = 3.0 * 6.0 * math.sqrt(H) * 2.0 ** -24
    g = (plane.Grid2 if flat else Grid).from_spec(spec)
    h0 = lbfgs.H0Solver(g, gamma, plane.laplacian(g)) if flat else lbfgs.H0Solver(g, gamma)
    rng = np.random.default_rng(5)
    shape = (2, my[1], my[0]) if flat else (3, my[2], my[1], my[0])
    v = rng.standard_normal(shape).astype(np.float32)
    want = h0.apply(v.astype(np.float64))
    ctx = mfr.Context(spec, DEV)
    x = ctx.h0_solve(to_dev(v), gamma)
    assert x.shape == v.shape
    assert rel_l2(x.cpu().numpy(), want) <= tol
    t = to_dev(v)
    ctx.h0_solve(t, gamma, out=t)
    assert torch.equal(t, x)
    ctx.close()
