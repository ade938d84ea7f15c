"""Contexts beyond the pinned result pages (64 per process) copy their scalars instead: the same bits,
and the pages are lent again once contexts have ended."""
import pytest
import torch

from gpu_cases import DEV, ct_case, to_dev
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu


def _results(ctx, u, b):
    v = u.clone()
    J = ctx.objective(u)
    g, Jg = ctx.gradient(u)
    s, info = ctx.pcg_solve(u, b, max_iter=20, rtol=1e-2, precond=1)
    step = ctx.gn_step(v, pcg_max=6, pcg_rtol=1e-2, precond=1)
    lb = ctx.lbfgs(u.clone(), iters=2)
    torch.cuda.synchronize()
    return (J, Jg, info, step, {k: x for k, x in lb.items() if k != "seconds"}), (g, s, v)


def test_contexts_without_a_result_page():
    print("[gpu-case] 70 contexts at once", flush=True)
    spec, R, T, u, probes = ct_case(5, (24, 20, 16), (7, 6, 5), amp=0.5, n_probes=1)
    tR, tT, tu, tb = to_dev(R), to_dev(T), to_dev(u), to_dev(probes[0])
    ref = None
    for _ in range(2):   # the second time with the pages of the first
        ctxs = [mfr.Context(spec, DEV) for _ in range(70)]
        for k in (0, 63, 64, 69):   # the last ones have none
            ctxs[k].set_images(tR, tT)
            got = _results(ctxs[k], tu, tb)
            ref = ref or got
            assert got[0] == ref[0], k
            assert all(torch.equal(a, b) for a, b in zip(got[1], ref[1])), k
        for c in ctxs:
            c.close()
