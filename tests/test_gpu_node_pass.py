"""The node pass that forms L L f from the 25 points of the twice applied Laplacian: grids of two
to five nodes per axis, where clamped neighbours of first and second order meet, and sizes around
its work-groups.  Constant images, so the regulariser is all there is; against the float64 oracle's
assembled operators.  Tolerance 2e-6 (relative L2): about ten float32 operations deep, each value
of the order of the result for a normal direction."""
import numpy as np
import pytest
import torch

from gpu_cases import DEV, rel_l2, to_dev
from oracle import Grid, curvature, diffusive, elastic
from paper_1804_10541_amd import mfr
from synth import GridSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reg", ["curvature", "diffusive", "elastic"])
@pytest.mark.parametrize("my", [(2, 3, 4), (4, 2, 3), (5, 4, 2), (3, 5, 5), (4, 8, 8), (3, 5, 17), (17, 16, 15)],
                         ids=lambda v: "x".join(map(str, v)))
def test_regulariser_products(my, reg):
    print(f"[gpu-case] node pass {my} {reg}", flush=True)
    m = tuple(2 * (k - 1) + 2 for k in my)
    spec = GridSpec(m=m, h=(1.0, 1.2, 0.9), my=my, tau=0.1, rho=0.1, alpha=0.7, regulariser=reg, lame_mu=1.3,
                    lame_lambda=0.4)
    rng = np.random.default_rng(2)
    p = rng.standard_normal((3, my[2], my[1], my[0])).astype(np.float32)
    ctx = mfr.Context(spec, DEV)
    img = torch.ones(m[2], m[1], m[0], device=DEV)
    big = torch.full_like(img, 1.0)
    ctx.set_images(img, big)
    u = to_dev(np.zeros_like(p))
    q = ctx.hess_vec(u, to_dev(p))
    g, _ = ctx.gradient(to_dev(p), want_J=False)   # S's gradient is linear in u
    S = ctx.objective(to_dev(p))[2]
    torch.cuda.synchronize()
    grid = Grid.from_spec(spec)
    mod = {"curvature": curvature, "diffusive": diffusive, "elastic": elastic}[reg]
    ref = spec.alpha * np.asarray(mod.hess_vec(grid, p.astype(np.float64)))
    # the zero extension outside a constant template gives the distance its own part at u = 0 and p
    ctx0 = mfr.Context(GridSpec(**{**spec.__dict__, "alpha": 0.0}), DEV)
    ctx0.set_images(img, big)
    q0 = ctx0.hess_vec(u, to_dev(p))
    g0, _ = ctx0.gradient(to_dev(p), want_J=False)
    torch.cuda.synchronize()
    f64 = lambda t: t.cpu().numpy().astype(np.float64)   # noqa: E731
    scale = max(1.0, np.linalg.norm(f64(q0)) / np.linalg.norm(ref), np.linalg.norm(f64(g0)) / np.linalg.norm(ref))
    assert rel_l2(f64(q) - f64(q0), ref) <= 2e-6 * scale
    assert rel_l2(f64(g) - f64(g0), ref) <= 2e-6 * scale
    assert abs(S - mod.energy(grid, p.astype(np.float64))) <= 2e-6 * S
    ctx.close()
    ctx0.close()
