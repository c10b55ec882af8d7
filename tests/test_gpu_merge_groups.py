"""The merge of work-item records with one, four and sixteen wavefronts per
subvolume: against numpy's merge of the items' own records, which come from the
same samples listed as one subvolume per item.  Items per subvolume around the
edges of a batch (16 items), of the rule (16, 64) and of the runs' lengths, empty
runs among them (65 items are 13 runs of 5 for 16 wavefronts).  The sums are
compensated on both sides, so they agree to a few roundings; 1e-13 of each
sum's L1 scale."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ITEM = 64  # samples per item: 64-thread blocks, one sample per thread


@pytest.mark.parametrize("items", [1, 2, 7, 8, 9, 16, 17, 18, 31, 63, 64, 65, 66, 97, 511, 1030])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_merge_of_items(bfi, ctx, items, prec):
    d, nx = 8, 4
    lat = bfi.lattice(4, 2)
    lo, hi = np.full((1, d), -2.0), np.full((1, d), 2.0)
    launch = bfi.launch(1, ITEM, 1)
    whole = bfi.Subvolumes([5], lo, hi, ITEM * items, 3, d)
    each = bfi.Subvolumes(np.full(items, 5), np.repeat(lo, items, 0), np.repeat(hi, items, 0), ITEM,
                          3 + ITEM * np.arange(items), d)
    got = bfi.bfi_eval(ctx, lat, prec, 7, whole, launch)[0]
    rec = bfi.bfi_eval(ctx, lat, prec, 7, each, launch)
    sigma = rec[:, 1].min()
    assert got[0] == ITEM * items and got[1] == sigma
    first = np.zeros(rec.shape[1], bool)
    first[[2] + list(range(4, 4 + nx))] = True
    for f in range(2, rec.shape[1]):
        factor = np.exp((sigma - rec[:, 1]) * (1.0 if first[f] else 2.0))
        terms = rec[:, f] * factor
        assert abs(got[f] - math.fsum(terms)) <= 1e-13 * math.fsum(np.abs(terms)), f
