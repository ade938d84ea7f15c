"""A learned preconditioner bound to a context leaves the calls that do not use it as they are: a
Jacobi-preconditioned solve and a Gauss-Newton step give the bits of an unbound context."""
import pytest
import torch

from gpu_cases import DEV, ct_case, to_dev
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,my", [((40, 36, 28), (11, 10, 8)), ((64, 48, 66), (17, 13, 17))],
                         ids=lambda v: "x".join(map(str, v)))
def test_jacobi_solves_do_not_see_a_bound_preconditioner(m, my):
    print(f"[gpu-case] Jacobi solves with a preconditioner bound {m} {my}", flush=True)
    spec, R, T, u, probes = ct_case(5, m, my, amp=0.5, n_probes=1)
    tu, tb, tR, tT = to_dev(u), to_dev(probes[0]), to_dev(R), to_dev(T)
    out = []
    for bound in (False, True):
        ctx = mfr.Context(spec, DEV)
        ctx.set_images(tR, tT)
        pc = mfr.LearnedPC(ctx) if bound else None
        s, info = ctx.pcg_solve(tu, tb, max_iter=12, rtol=0.0, precond=1)
        v = tu.clone()
        step = ctx.gn_step(v, pcg_max=8, pcg_rtol=0.0, precond=1)
        torch.cuda.synchronize()
        out.append((s, v, info, step))
        if pc is not None:
            pc.close()
        ctx.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert out[0][2] == out[1][2] and out[0][3] == out[1][3]
