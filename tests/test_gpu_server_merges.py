"""Requests that finish together merge in one launch of up to sixteen lists per
kernel: a single list, one less and one more than a launch holds and two
launches' worth, of one, four and sixteen wavefronts per subvolume mixed, with
records on both sides of the 64 KiB that a merge writes to host memory itself.
The sums of a list do not depend on what merges beside it: bit for bit the
result of the request served alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (lattice, split_log2, evaluations): items per subvolume up to 16, up to 64 and
# beyond; 2048 subvolumes of 10x2 are 557 KB of records, 256 of 4x2 are 32 KB
KINDS = [((4, 2), 4, 1 << 16), ((4, 2), 0, 1 << 20), ((8, 2), 0, 1 << 22),
         ((10, 2), 11, 1 << 17), ((4, 2), 8, 1 << 16)]


@pytest.mark.parametrize("count", [1, 15, 17, 32])
def test_finished_together(bfi, ctx, count):
    reqs = []
    for i in range(count):
        (nx, nt), k, n = KINDS[(i * 3) % len(KINDS)]
        reqs.append(bfi.request(bfi.lattice(nx, nt), "fp32" if i % 2 else "fp64", i + 1, 3.0, k, n))
    server = bfi.bfi_server_create(ctx, bfi.server_config(memory_budget=4 << 30, max_requests=64))
    try:
        tickets = [bfi.bfi_server_submit(server, r) for r in reqs]
        together = [bfi.bfi_server_wait(server, t, 60.0)[0] for t in tickets]
        for i in list(range(0, count, 4)) + [count - 1]:
            alone = bfi.bfi_server_wait(server, bfi.bfi_server_submit(server, reqs[i]), 60.0)[0]
            for name in ("Z", "Z_err", "log_Z", "ess", "C", "C_err"):
                assert np.array_equal(alone[name], together[i][name]), (i, name)
    finally:
        bfi.bfi_server_destroy(server)
