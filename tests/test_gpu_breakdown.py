"""CG solves that break down (p.q <= 0 or not finite): the iterate returned is the one before the
failing step, bit for bit that of a solve limited to the iterations before it, for the synchronous
solve, its capturable twin and inside a batch.  Flat images leave the curvature term alone, whose
product with a direction near the largest float overflows after some iterations; edge parameters
far above the images' gradients leave a product that underflows to 0 in the first one."""
import pytest
import torch

from gpu_cases import DEV, blob_case, to_dev
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu


# node vectors of one work-group of the CG kernels, of a few, and of the most there are (1024)
@pytest.mark.parametrize("m,my", [((8, 8, 8), (4, 4, 4)), ((24, 20, 16), (9, 8, 7)), ((128, 128, 96), (65, 65, 49))],
                         ids=lambda v: "x".join(map(str, v)))
def test_iterate_before_the_failing_step(m, my):
    print(f"[gpu-case] CG breakdown {m} {my}", flush=True)
    spec, R, _, u, probes = blob_case(3, m, my, alpha=1.0, n_probes=1)
    flat = to_dev(R * 0.0 + 0.5)
    ctx = mfr.Context(spec, DEV)
    ctx.set_images(flat, flat.clone())
    tu = to_dev(u * 0.0)
    base = torch.cumsum(to_dev(probes[0]), dim=1) / 16.0   # rough and smooth parts: CG directions that grow
    found = 0
    for e in range(90, 128):
        b = base * 2.0 ** e
        s, info = ctx.pcg_solve(tu, b, max_iter=24, rtol=0.0, precond=0)
        if info["flag"] != 2:
            continue
        ref, lim = ctx.pcg_solve(tu, b, max_iter=info["iters"], rtol=0.0, precond=0)
        assert torch.equal(s.view(torch.int32), ref.view(torch.int32)) and lim["iters"] == info["iters"], e
        x, out = torch.empty_like(s), torch.empty(3, dtype=torch.float64, device=DEV)
        ctx.pcg_solve_async(tu, b, max_iter=24, rtol=0.0, precond=0, out=x, info=out)
        assert torch.equal(x.view(torch.int32), s.view(torch.int32)), e
        assert out.cpu().tolist() == [info["iters"], info["relres"], 2.0]
        found += bool(info["iters"] > 0 and torch.isfinite(s).all())
    assert found > 0   # at least one solve got past its first iteration
    ctx.close()


@pytest.mark.parametrize("use_graph", [False, True])
def test_a_pair_that_breaks_down_leaves_the_others_alone(use_graph):
    print(f"[gpu-case] CG breakdown in a batch, graph={use_graph}", flush=True)
    sizes = [((40, 28, 21), (11, 8, 6), 0.1), ((64, 48, 40), (33, 25, 21), 1e12), ((33, 40, 17), (9, 11, 5), 0.1)]
    cases = [blob_case(7 + i, m, my, tau=t, rho=t, alpha=0.0 if t > 1.0 else 1.0, n_probes=0)
             for i, (m, my, t) in enumerate(sizes)]
    opts = dict(gn_iters=3, pcg_max=10, pcg_rtol=1e-3, precond=0)
    ctx = mfr.Context(cases[1][0], DEV)
    ctx.set_images(to_dev(cases[1][1]), to_dev(cases[1][2]))
    step = ctx.gn_step(torch.zeros(ctx.node_shape(), device=DEV), pcg_max=10, pcg_rtol=1e-3,
                       precond=0)
    assert step["pcg_flag"] == 2 and step["pcg_iters"] == 0   # this pair does break down
    ctx.close()
    b = mfr.Batch([c[0] for c in cases], levels=1, device=DEV)
    b.set_images([to_dev(c[1]) for c in cases], [to_dev(c[2]) for c in cases])
    ub, rep = b.register(use_graph=use_graph, **opts)
    for k, (spec, R, T, _, _) in enumerate(cases):
        u1, r1 = mfr.register_multilevel(spec, to_dev(R), to_dev(T), levels=1, **opts)
        assert torch.equal(u1, ub[k]), k
        assert sum(r1["pcg_total"]) == rep["pcg_total"][k], k
        assert sum(r1["gn_done"]) == rep["gn_done"][k], k
    b.close()
