"""Grids whose cells are deep along the march, so that several chunks of the derived split hold one
node plane: against the float64 oracle, float32 sums of up to a thousand terms per node.  Tolerance
2e-6 (relative L2) for the gradient, the product and the diagonal, 1e-6 for the objective."""
import pytest

from gpu_cases import blob_case, gpu_eval, oracle_eval, rel_l2
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def derived_split():   # (another test's tile configuration may be in force)
    old = mfr.get_tile_config()
    mfr.set_tile_config(32, 16, 0, 0)
    yield
    mfr.set_tile_config(**old)


@pytest.mark.parametrize("m,my", [((33, 20, 70), (9, 6, 2)), ((20, 17, 64), (5, 5, 3)), ((24, 31, 97), (4, 9, 4))],
                         ids=lambda v: "x".join(map(str, v)))
def test_deep_cells(m, my):
    print(f"[gpu-case] deep cells {m} {my}", flush=True)
    spec, R, T, u, probes = blob_case(8, m, my, alpha=0.3, n_probes=1)
    a, b = gpu_eval(spec, R, T, u, probes), oracle_eval(spec, R, T, u, probes)
    assert abs(a["J"] - b["J"]) <= 1e-6 * abs(b["J"])
    for k in ("grad", "diag"):
        assert rel_l2(a[k], b[k]) <= 2e-6, k
    assert rel_l2(a["hv"][0], b["hv"][0]) <= 2e-6
