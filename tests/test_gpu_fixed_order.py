"""Calls whose results are decisions by split statistics: their sums keep the
launch shape's order, whatever the size of the list.  Leaves with a few weighty
samples make dimensions tie but for the last bits, so another order would
suggest another dimension: bitwise comparison with the launch shape given."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("dim,per_sub", [(2, 300_001), (12, 20_000), (16, 37_047)])
def test_nsphere_suggestions(bfi, ctx, dim, per_sub):
    sv = workloads.random_partition(dim, 1.0, 40, per_sub=per_sub, seed=dim)
    f = bfi.integrand_nsphere(dim)
    assert _same(bfi.bfi_integrand_eval(ctx, f, 3, sv),
                 bfi.bfi_integrand_eval(ctx, f, 3, sv, bfi.launch(64, 256, 1)))


@pytest.mark.parametrize("distance", [None, 2])
def test_lattice_suggestions(bfi, ctx, distance):
    lat = bfi.lattice(10, 2, nu=0.5)
    sv = workloads.random_partition(20, 4.0, 60, per_sub=40_000, seed=8)
    f = bfi.integrand_burgers(lat, "fp64", distance)
    value, err, dim = bfi.bfi_integrand_eval(ctx, f, 3, sv)
    assert _same((value, err, dim),
                 bfi.bfi_integrand_eval(ctx, f, 3, sv, bfi.launch(64, 256, 1)))
