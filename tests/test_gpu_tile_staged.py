"""Node values that the voxel-tile march reads through LDS a node plane ahead: cells of two planes
and of mixed depth, single-plane cells and blocks of too many nodes (which keep the direct loads), a
first and a last cell of one plane, chunks that begin inside a cell or at its first plane, and marches
of one cell.  Tolerance 2e-6 (relative L2) against the float64 oracle, as for the node-plane reduction
(float32 sums, sqrt of the term count); the objective 1e-6."""
import pytest

from gpu_cases import blob_case, gpu_eval, oracle_eval, rel_l2
from paper_1804_10541_amd import mfr

pytestmark = pytest.mark.gpu

CASES = [((34, 20, 24), (18, 11, 13), 24), ((34, 20, 24), (18, 11, 13), 9), ((31, 15, 26), (8, 5, 11), 26),
         ((31, 15, 26), (8, 5, 11), 13), ((30, 14, 17), (8, 5, 10), 17), ((24, 18, 15), (7, 5, 16), 15),
         ((40, 30, 22), (41, 31, 9), 22), ((20, 16, 12), (6, 5, 2), 12), ((20, 16, 12), (6, 5, 5), 4)]


@pytest.mark.parametrize("m,my,chunk", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_staged_node_planes(m, my, chunk):
    print(f"[gpu-case] staged node planes {m} {my} {chunk}", flush=True)
    spec, R, T, u, probes = blob_case(7, m, my, alpha=0.3, n_probes=1, h=(1.0, 1.1, 0.9))
    old = mfr.get_tile_config()
    mfr.set_tile_config(32, 16, chunk, 0)
    try:
        a = gpu_eval(spec, R, T, u, probes, diag=False)
    finally:
        mfr.set_tile_config(**old)
    b = oracle_eval(spec, R, T, u, probes, diag=False)
    assert abs(a["J"] - b["J"]) <= 1e-6 * abs(b["J"])
    assert rel_l2(a["grad"], b["grad"]) <= 2e-6
    assert rel_l2(a["hv"][0], b["hv"][0]) <= 2e-6
