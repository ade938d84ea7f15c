"""Rows of the voxel-tile kernel where their factors can go wrong: a template whose planes are too
large for 24-bit byte offsets, edge parameters so small that 1 / (|grad T| |grad R|) squared
overflows, and images of one plane to four.  Tolerance 2e-6 (relative L2) against the float64
oracle, as for the node-plane reduction (float32 sums, sqrt of the term count)."""
import numpy as np
import pytest

from gpu_cases import blob_case, gpu_eval, oracle_eval, rel_l2

pytestmark = pytest.mark.gpu


def _check(spec, R, T, u, probes):
    a, b = gpu_eval(spec, R, T, u, probes), oracle_eval(spec, R, T, u, probes)
    for k in ("grad", "diag"):
        assert rel_l2(a[k], b[k]) <= 2e-6, k
    assert rel_l2(a["hv"][0], b["hv"][0]) <= 2e-6
    return a, b


def test_large_template_planes():
    m, mT = (24, 20, 8), (2100, 2000, 3)
    hT = tuple(float(a) / b for a, b in zip(m, mT))
    spec, R, T, u, probes = blob_case(3, m, (7, 6, 4), alpha=0.3, n_probes=1, mT=mT, hT=hT, amp=0.3)
    a, b = gpu_eval(spec, R, T, u, probes, diag=False), oracle_eval(spec, R, T, u, probes, diag=False)
    # the float32 template coordinate carries 2^-24 mT cells: relative to a smooth template's
    # derivative scale (a tenth of the image) about 1e-3 of a cell, 1e-5 of a difference
    assert rel_l2(a["hv"][0], b["hv"][0]) <= 1e-3
    assert rel_l2(a["grad"], b["grad"]) <= 1e-3


@pytest.mark.parametrize("mz", [2, 3, 4])
def test_few_planes(mz):
    print(f"[gpu-case] tile rows {mz} planes", flush=True)
    _check(*blob_case(4, (33, 17, mz), (9, 6, 2), alpha=0.3, n_probes=1))


def test_flat_images_with_tiny_edge_parameters():
    spec, R, T, u, probes = blob_case(5, (34, 18, 12), (9, 6, 4), tau=1e-10, rho=1e-10, alpha=0.3, n_probes=1)
    flat = np.full_like(R, 0.25), np.full_like(T, 0.5)
    a, b = gpu_eval(spec, *flat, u * 0.0, probes), oracle_eval(spec, *flat, u * 0.0, probes)
    inner = (slice(None), slice(1, -1), slice(1, -1), slice(1, -1))
    assert np.isfinite(a["hv"][0]).all() and np.isfinite(a["grad"]).all()
    assert rel_l2(a["hv"][0][inner], b["hv"][0][inner]) <= 2e-6
