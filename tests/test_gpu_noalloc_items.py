"""bfi_eval_noalloc equals bfi_eval bit for bit also where plain FP64 items cut
shorter than the launch shape's would not fit the allocation-free entry's array
(32 MiB) and the launch shape's do: 16x4, 64-thread blocks, about 9500 subvolumes of
2 samples beside one long enough to be cut (27 to 33 MB with the launch shape's
items, up to 34 with shorter ones), below, inside and above that window."""
import numpy as np
import pytest


pytestmark = pytest.mark.gpu


def _layout(count, items, d=64, rec=4 + 3 * 16):
    """Bytes of the array as the header lists its regions."""
    regions = [count * 8] * 3 + [count * d * 8] * 4 + [count * d * 4] * 2 + \
        [256, (count + 1) * 4, items * 32, items * rec * 8, count * rec * 8, 4]
    return sum(-(-r // 256) * 256 for r in regions)


@pytest.mark.parametrize("count", [8000, 9500, 9700])
@pytest.mark.parametrize("long", [327_680, 2_441_406, 28_421_691])
def test_same_items_at_the_arrays_limit(bfi, ctx, count, long):
    lat = bfi.lattice(16, 4, nu=0.5)
    rng = np.random.Generator(np.random.PCG64(count))
    lo = rng.uniform(-1.0, 0.0, (count, 64))
    n = np.full(count, 2)
    n[-1] = long
    sv = bfi.Subvolumes(np.arange(1, count + 1), lo, lo + 0.5, n, 0, 64)
    shape = bfi.launch(0, 64, -1)
    print(f"noalloc items: {count} subvolumes, one of {long}", flush=True)
    want = bfi.bfi_eval(ctx, lat, "fp64", 3, sv, shape)
    if _layout(count, count - 1 + -(-long // (64 * 64))) > 32 << 20:
        with pytest.raises(bfi.BfiError, match="scratch"):
            bfi.bfi_eval_noalloc(ctx, lat, "fp64", 3, sv, shape)
        return
    got = bfi.bfi_eval_noalloc(ctx, lat, "fp64", 3, sv, shape)
    assert np.array_equal(got.view(np.uint64), want.view(np.uint64))
