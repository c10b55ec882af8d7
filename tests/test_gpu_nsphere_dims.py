"""The N-sphere kernels, one per dimension, against the oracle's points in numpy:
every remainder of the dimension by the four words of a Philox block, sample
ranges on both sides of and across a 2^32 boundary of the Philox counter, boxes
inside, outside and across the ball."""
import math

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", range(1, 17))
def test_every_dimension(bfi, ctx, dim):
    n, blocks = 700, -(-dim // 4)
    edge = 2**32 // blocks  # first sample whose counters lie past (or across) 2^32
    lists = [(-0.9, 1.1, 0), (0.0, 0.2 / math.sqrt(dim), edge - n // 2), (1.0, 2.0, edge + 3),
             (-1.0, 1.0, edge - n)]
    sv = workloads.SubvolumeList(
        np.arange(5, 5 + len(lists)).astype(np.uint64),
        np.array([[b[0]] * dim for b in lists]), np.array([[b[1]] * dim for b in lists]),
        np.full(len(lists), n, np.uint64), np.array([b[2] for b in lists], np.uint64))
    value, err, split = bfi.bfi_integrand_eval(ctx, bfi.integrand_nsphere(dim), 9, sv)
    for s, (lo, hi, first) in enumerate(lists):
        u = oracle.points(dim, 9, 5 + s, [lo] * dim, [hi] * dim,
                          np.arange(first, first + n).astype(np.uint64))
        r2 = np.zeros(n)
        for k in range(dim):
            r2 += u[:, k] ** 2
        f = np.sqrt(np.maximum(1.0 - r2, 0.0))
        vol = (hi - lo) ** dim
        mean = math.fsum(f) / n
        var = max(math.fsum(f * f) - n * mean * mean, 0.0) / (n - 1)
        # r2 carries dim + 1 roundings of at most 2^-53 each, so f = sqrt(1 - r2)
        # is off by at most (dim + 1) 2^-53 / (2 f) and its sum by their sum
        tol = 2e-16 * (n * mean + (dim + 1) * np.sum(1.0 / np.maximum(f[f > 0], 1e-8))) * n
        assert abs(value[s] - vol * mean) <= vol / n * tol + 1e-300
        assert err[s] == pytest.approx(vol * math.sqrt(var / n), rel=1e-7, abs=1e-12)
        assert 0 <= split[s] < dim
