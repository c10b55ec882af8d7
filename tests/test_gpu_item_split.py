"""Work items cut smaller than the launch shape's to fill the chip (plain FP64,
samples_per_thread left open) against the launch shape's own items and the FP64
oracle.  The samples are the same, so two records differ by the order of
summation alone: at most n terms of relative rounding 2^-53 each side, so
n 2^-52 of a sum's L1 scale (n <= 2^18 here: 6e-11; 1e-10 as everywhere)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


def _close(got, want, nx, d=0):
    """Records (or records and split statistics) of the same samples."""
    assert np.array_equal(got[:, :2], want[:, :2])
    n, pw2 = want[:, 0:1], want[:, 4 + nx:4 + 2 * nx]
    scale = np.concatenate([want[:, 2:4], np.sqrt(n * pw2), pw2,
                            np.sqrt(pw2 * want[:, 3:4])], axis=1)
    assert np.all(np.abs(got[:, 2:] - want[:, 2:]) <= 1e-10 * scale)


def _lists(d):
    """Edges of the rule: one pair of samples, items of one sample per thread,
    a block's size and the default item's 16384 with their neighbours, counts
    from 2 to 2^18 in one list."""
    one = workloads.uniform_partition(d, 2.0, 0, per_sub=2)
    even = workloads.uniform_partition(d, 2.0, 3, per_sub=1)
    even.n[:] = [255, 256, 257, 16383, 16384, 16385, 2, 65537]
    ragged = workloads.random_partition(d, 2.0, 37, per_sub=1, seed=4)
    ragged.n[:] = workloads.log_uniform_counts(37, 1, 18, seed=9)
    ragged.offset[:] = np.arange(37, dtype=np.uint64) * np.uint64(2**30 + 7)
    return one, even, ragged


@pytest.mark.parametrize("nx,nt", [(2, 1), (4, 2), (10, 2), (16, 4)])
def test_smaller_items_same_sums(bfi, ctx, nx, nt):
    lat = bfi.lattice(nx, nt, nu=0.6)
    for sv in _lists(nx * nt):
        print(f"items: {nx}x{nt} {len(sv)} subvolumes {int(sv.n.sum())} samples", flush=True)
        got = bfi.bfi_eval(ctx, lat, "fp64", 3, sv)
        _close(got, bfi.bfi_eval(ctx, lat, "fp64", 3, sv, bfi.launch(64, 256, 1)), nx)
        want = oracle.sums(oracle.lattice(nx, nt, nu=0.6), 3, sv.ids, sv.lo, sv.hi, sv.n,
                           sv.offset)
        _close(got, np.insert(want, 1, 0.0, axis=1), nx)
        same = bfi.bfi_eval_noalloc(ctx, lat, "fp64", 3, sv)
        assert np.array_equal(got.view(np.uint64), same.view(np.uint64))


def test_split_pairs_and_samplers(bfi, ctx):
    shape = bfi.launch(64, 256, 1)
    for sv in _lists(20):
        lat = bfi.lattice(10, 2, observable="averaged")
        (a, sa), (b, sb) = (bfi.bfi_eval(ctx, lat, "fp64", 5, sv, l, split=True)
                            for l in (None, shape))
        _close(a, b, 10)
        assert np.all(np.abs(sa - sb)[:, 1:21] <= 1e-10 * b[:, 2:3])
        assert np.all(np.abs(sa - sb)[:, 21:] <= 1e-10 * b[:, 3:4])
        pairs = bfi.lattice(10, 2, antithetic=True)
        _close(bfi.bfi_eval(ctx, pairs, "fp64", 5, sv), bfi.bfi_eval(ctx, pairs, "fp64", 5, sv, shape),
               10)
    lat = bfi.lattice(4, 2)
    ids = np.array([1, 2, (1 << 63) + 1], np.uint64)
    n = [2, 70_001, 300]
    _close(bfi.bfi_is_eval(ctx, lat, "fp64", 2, -4.0, 4.0, 0.9, ids, n),
           bfi.bfi_is_eval(ctx, lat, "fp64", 2, -4.0, 4.0, 0.9, ids, n, 0, shape), 4)
    shells = bfi.Shells([1, 2, 3], [0.0, 1.0, 2.0], [1.0, 2.0, 3.0], [2, 100_001, 257])
    _close(bfi.bfi_sph_eval(ctx, lat, "fp64", 2, 4.0, shells),
           bfi.bfi_sph_eval(ctx, lat, "fp64", 2, 4.0, shells, shape), 4)
    box = workloads.uniform_partition(6, 1.0, 3, per_sub=100_003)
    f = bfi.integrand_nsphere(6)
    for a, b in zip(bfi.bfi_integrand_eval(ctx, f, 1, box),
                    bfi.bfi_integrand_eval(ctx, f, 1, box, shape)):
        np.testing.assert_allclose(a, b, rtol=1e-10)


def test_launch_shape_items_kept(bfi, ctx):
    """Items of the launch shape: the shifted forms, a given samples_per_thread,
    and lists long enough to fill the chip."""
    lat = bfi.lattice(4, 2)
    sv = workloads.uniform_partition(8, 2.0, 4, per_sub=40_000)

    def items(prec, launch, sub=sv):
        plan = bfi.bfi_plan_create(ctx, lat, prec, sub, launch)
        try:
            return bfi.bfi_plan_info(plan)["n_items"]
        finally:
            bfi.bfi_plan_destroy(plan)

    per = -(-40_000 // (64 * 256))
    shape = bfi.launch(64, 256, 1)
    assert items("fp32", None) == items("fp64s", None) == items("fp64", shape) == 16 * per
    assert items("fp64", None) > 16 * per
    long = workloads.uniform_partition(8, 2.0, 4, per_sub=1 << 26)
    assert items("fp64", bfi.launch(0, 256, 1), long) == 16 * (1 << 26) // (64 * 256)
