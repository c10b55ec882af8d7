"""Memory of blocking calls: the context's block, grown from call to call, and
the call's own where the block is taken by another thread or too small for it.
The records are those of a plan, which has memory of its own, bit for bit."""
import threading

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _plan_records(bfi, ctx, lat, prec, sv, seed):
    plan = bfi.bfi_plan_create(ctx, lat, prec, sv)
    try:
        bfi.bfi_plan_run(plan, seed)
        return bfi.bfi_plan_partials(plan, len(sv), lat.nx)
    finally:
        bfi.bfi_plan_destroy(plan)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_sizes_in_turn(bfi, prec):
    """Below, above (200000 subvolumes of 20 dimensions: 76 MB of point maps,
    ids and items in FP64) and below the block's limit again, on one context,
    with a refused call between."""
    c = bfi.bfi_context_create(0)
    try:
        lat = bfi.lattice(10, 2)
        for k, (count, n) in enumerate([(3, 500), (5000, 3), (200_000, 2), (7, 40_000), (1, 2)]):
            print(f"scratch: {prec} {count} subvolumes of {n}", flush=True)
            sv = workloads.uniform_partition(20, 4.0, 0, per_sub=n)
            sv = bfi.Subvolumes(np.arange(1, count + 1), np.repeat(sv.lo, count, 0),
                                np.repeat(sv.hi, count, 0), n, 0, 20)
            got = bfi.bfi_eval(c, lat, prec, k + 1, sv)
            assert np.array_equal(got, _plan_records(bfi, c, lat, prec, sv, k + 1))
            few = bfi.Subvolumes(sv.ids, sv.lo, sv.hi, 1, 0, 20)
            with pytest.raises(bfi.BfiError):
                bfi.bfi_eval(c, lat, prec, 1, few)
    finally:
        bfi.bfi_context_destroy(c)


def test_calls_of_several_threads(bfi, ctx):
    """Calls that overlap on one context: each has the records of the same call
    alone."""
    lat = bfi.lattice(10, 2, nu=0.5)
    lists = [workloads.random_partition(20, 4.0, 20 + 30 * t, per_sub=3000 + 700 * t, seed=t)
             for t in range(4)]
    alone = [bfi.bfi_eval(ctx, lat, "fp64", t + 1, sv, split=True) for t, sv in enumerate(lists)]
    bad = []

    def work(t):
        for _ in range(25):
            got = bfi.bfi_eval(ctx, lat, "fp64", t + 1, lists[t], split=True)
            if not all(np.array_equal(a, b) for a, b in zip(got, alone[t])):
                bad.append(t)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
