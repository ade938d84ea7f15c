"""mfr_hess_vec_noalloc on problems close to its scratch array's size, whose full context workspace is
larger than the array while that of longer chunks is not: the product equals that of a context of
mfr_workspace_size bytes bit for bit."""
import pytest
import torch

from gpu_cases import DEV, blob_case, to_dev
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def derived_split():   # (another test's tile configuration may be in force)
    old = mfr.get_tile_config()
    mfr.set_tile_config(32, 16, 0, 0)
    yield
    mfr.set_tile_config(**old)


@pytest.mark.parametrize("m,my", [((78, 208, 89), (79, 36, 90)), ((241, 73, 59), (62, 74, 60))],
                         ids=lambda v: "x".join(map(str, v)))
def test_product_equals_that_of_a_full_context(m, my):
    print(f"[gpu-case] noalloc hess_vec at the array's limit {m} {my}", flush=True)
    spec, R, T, u, probes = blob_case(6, m, my, n_probes=1)
    assert mfr.workspace_size(spec) > 64 << 20   # (else the case shows nothing)
    tR, tT, tu, tp = (to_dev(a) for a in (R, T, u, probes[0]))
    ctx = mfr.Context(spec, DEV)
    ctx.set_images(tR, tT)
    want = ctx.hess_vec(tu, tp)
    got = torch.full_like(want, float("nan"))
    mfr.hess_vec_noalloc(spec, tR, tT, tu, tp, got)
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(got, want)
