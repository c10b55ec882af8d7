"""Record bits.  Refinement decides by sums that tie but for their last bits where
a few samples carry a leaf's weight, so their order and their roundings are part
of a run's result: a lane's scaled sum is one rounded product plus the lower
half's in a fused multiply-add, then lanes at distances 16, 8, 4, 2, 1, the
wavefronts in order, the items in order.  Digests of records and split
statistics in the three forms, and of an adaptive run's partition, on lists
with heavy-tailed weights (golden/record_bits.json, from the reduction by LDS
butterflies that first defined this order)."""
import hashlib
import json
import os

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "record_bits.json")
CASES = [(prec, nx, nt, obs, split) for prec in ("fp64", "fp32", "fp64s")
         for nx, nt, obs, split in ((3, 2, "anchor", True), (4, 2, "averaged", True),
                                    (10, 2, "anchor", True), (10, 2, "averaged", False),
                                    (16, 4, "anchor", False))]


def digest(arrays):
    h = hashlib.sha256()
    for a in arrays:
        h.update(np.ascontiguousarray(a).tobytes())
    return h.hexdigest()[:32]


def records(bfi, ctx, prec, nx, nt, obs, split):
    d = nx * nt
    sv = workloads.random_partition(d, 4.0 if nt == 2 else 3.0, 60, per_sub=1, seed=d)
    sv.n[:] = workloads.log_uniform_counts(60, 5, 15, seed=d + 1)
    got = bfi.bfi_eval(ctx, bfi.lattice(nx, nt, nu=0.7, observable=obs), prec, 9, sv,
                       bfi.launch(16, 256, 1), split=split)
    return got if split else (got,)


def adaptive(bfi, ctx, prec):
    cfg = bfi.adaptive_config(target_rel_err=1e-6, max_evals=1 << 24, n_min=1 << 10, n_max=1 << 18,
                              split_log2=8, max_rounds=12, round_evals=1 << 21,
                              split_samples=1 << 12)
    got = bfi.bfi_integrate_adaptive(ctx, bfi.lattice(10, 2, observable="averaged"), prec, 3, -4.0,
                                     4.0, cfg, bfi.launch(64, 256, 1), leaf_capacity=1 << 14)
    p = got["partition"]
    return np.array([got["Z"], got["rel_err"]]), got["C"], got["C_err"], p.ids, p.lo, p.hi, p.n


@pytest.mark.parametrize("prec,nx,nt,obs,split", CASES)
def test_record_bits(bfi, ctx, prec, nx, nt, obs, split):
    want = json.load(open(GOLDEN))
    key = f"{prec} {nx}x{nt} {obs} {int(split)}"
    assert digest(records(bfi, ctx, prec, nx, nt, obs, split)) == want[key]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp64s"])
def test_adaptive_run_bits(bfi, ctx, prec):
    assert digest(adaptive(bfi, ctx, prec)) == json.load(open(GOLDEN))[f"adaptive {prec}"]
