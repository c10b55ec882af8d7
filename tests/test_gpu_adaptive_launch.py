"""An adaptive run takes its items through the queue, as a block each, or as the
library chooses, as its launch shape says: the same run bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("per_thread,block", [(1, 256), (64, 256)])
def test_queue_and_blocks(bfi, ctx, prec, per_thread, block):
    lat = bfi.lattice(4, 2, observable="averaged")
    runs = []
    for persistent in (1, 0, -1):
        cfg = bfi.adaptive_config(target_rel_err=1e-9, max_evals=1 << 23, n_min=1 << 10,
                                  n_max=1 << 16, split_log2=6, max_rounds=8, split_samples=1 << 12)
        print(f"adaptive launch: {prec} {per_thread}x{block} persistent {persistent}", flush=True)
        runs.append(bfi.bfi_integrate_adaptive(ctx, lat, prec, 2, -4.0, 4.0, cfg,
                                               bfi.launch(per_thread, block, persistent),
                                               leaf_capacity=1 << 14))
    a = runs[0]
    for b in runs[1:]:
        assert a["rounds"] == b["rounds"] >= 3 and a["Z"] == b["Z"]
        assert np.array_equal(a["C"], b["C"]) and np.array_equal(a["C_err"], b["C_err"])
        assert np.array_equal(a["partition"].ids, b["partition"].ids)
        assert np.array_equal(a["partition"].n, b["partition"].n)
