"""The device's fold and leaf analysis at the edges of their launches: leaf
counts around a wavefront (64), a block of four (256), a group (1024), the
shift's short path (8192) and its long one.  An adaptive run stopped after one
round of refinement reports the estimate of its partition; it must equal the
host finalize of the partition's records, evaluated in one pass.  The records
differ by the order of a leaf's samples over the round's passes alone (1e-11,
1e-9 of C(0) as in the adaptive tests)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2_leaves", [0, 5, 6, 8, 10, 13, 14])
@pytest.mark.parametrize("nx,prec", [(4, "fp64"), (10, "fp32")])
def test_estimate_of_the_partition(bfi, ctx, log2_leaves, nx, prec):
    lat = bfi.lattice(nx, 2, observable="averaged")
    n = 64
    cfg = bfi.adaptive_config(target_rel_err=1e-9, max_evals=5 * n << log2_leaves, n_min=n,
                              n_max=1 << 12, split_log2=log2_leaves, max_rounds=2,
                              refine_fraction=0.3, split_samples=n)
    got = bfi.bfi_integrate_adaptive(ctx, lat, prec, 5, -1.0, 1.0, cfg, leaf_capacity=1 << 17)
    part = got["partition"]
    assert len(part) >= 1 << log2_leaves
    want = bfi.bfi_finalize(lat, part, bfi.bfi_eval(ctx, lat, prec, 5, part))
    tol = 1e-11 if prec == "fp64" else 1e-5
    assert got["log_Z"] == pytest.approx(want["log_Z"], abs=tol)
    assert np.all(np.abs(got["C"] - want["C"]) <= 100 * tol * abs(want["C"][0]))
    assert got["Z_err"] == pytest.approx(want["Z_err"], rel=100 * tol)
    assert got["ess"] == pytest.approx(want["ess"], rel=100 * tol)
