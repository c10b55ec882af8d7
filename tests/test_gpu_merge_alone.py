"""A subvolume's record and split statistics depend on its own work items alone,
not on what is merged beside them: with a launch shape given, and in the shifted
forms with any, the same bits alone, beside a much larger subvolume, and in a list
long enough for another choice of wavefronts.  Item counts at the edges of the
merge's runs (1 | 16 | 17 | 64 | 65 items).  Plain FP64 with samples_per_thread
left open is the exception: the items follow the list, so the sums may differ by
the order of summation, n 2^-52 of their L1 scale (n < 2^18: 6e-11; 1e-10)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

ITEMS = [1, 2, 15, 16, 17, 33, 40, 63, 64, 65, 66, 100, 129, 250, 511]


def _list(d, block, items, seed):
    sv = workloads.random_partition(d, 2.0, len(items), per_sub=2, seed=seed)
    sv.n[:] = np.asarray(items, np.uint64) * np.uint64(block) - np.uint64(1)
    return sv


def _part(bfi, sv, keep):
    d = sv.lo.shape[1]
    return bfi.Subvolumes(sv.ids[keep], sv.lo[keep], sv.hi[keep], sv.n[keep], sv.offset[keep], d)


@pytest.mark.parametrize("nx,nt", [(4, 2), (10, 2)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp64s"])
@pytest.mark.parametrize("split", [False, True])
def test_alone_and_beside_others(bfi, ctx, nx, nt, prec, split):
    lat = bfi.lattice(nx, nt, nu=0.6)
    block = 256 if split else 64
    shape = bfi.launch(1, block, 1)

    def records(sv):
        got = bfi.bfi_eval(ctx, lat, prec, 3, sv, shape, split=split)
        return np.concatenate(got, axis=1) if split else got

    each = ITEMS * 8
    sv = _list(nx * nt, block, each + [3000], seed=nx)
    whole = records(sv)
    for keep in ([k] for k in range(0, len(each), 7)):
        assert np.array_equal(records(_part(bfi, sv, keep)).view(np.uint64),
                              whole[keep].view(np.uint64)), each[keep[0]]
    small = np.arange(len(each))
    assert np.array_equal(records(_part(bfi, sv, small)).view(np.uint64),
                          whole[small].view(np.uint64))
    # 2049 subvolumes and more: the average decides the wavefronts
    order = np.concatenate([np.arange(len(sv)), np.zeros(2049, int)])
    long = records(_part(bfi, sv, order))
    assert np.array_equal(long[:len(sv)].view(np.uint64), whole.view(np.uint64))


@pytest.mark.parametrize("split", [False, True])
def test_open_shape_beside_a_larger_one(bfi, ctx, split):
    lat = bfi.lattice(10, 2, nu=0.6)
    sv = workloads.random_partition(20, 2.0, 2, per_sub=50_000, seed=3)
    sv.n[1] = 1 << 25
    for shape in (None, bfi.launch(0, 256, -1)):
        both = bfi.bfi_eval(ctx, lat, "fp64", 3, sv, shape, split=split)
        alone = bfi.bfi_eval(ctx, lat, "fp64", 3, _part(bfi, sv, [0]), shape, split=split)
        if split:
            (both, both_s), (alone, alone_s) = both, alone
            assert np.all(np.abs(both_s[0] - alone_s[0])[1:21] <= 1e-10 * alone[0, 2])
            assert np.all(np.abs(both_s[0] - alone_s[0])[21:] <= 1e-10 * alone[0, 3])
        n, w2, pw2 = alone[0, 0], alone[0, 3], alone[0, 14:24]
        scale = np.concatenate([alone[0, 2:4], np.sqrt(n * pw2), pw2, np.sqrt(pw2 * w2)])
        assert np.array_equal(both[0, :2], alone[0, :2])
        assert np.all(np.abs(both[0, 2:] - alone[0, 2:]) <= 1e-10 * scale)
