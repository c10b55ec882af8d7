"""The merge's order of summation, on records made so that it shows: items whose
fields cancel over forty orders of magnitude, so that any other order gives other
numbers.  A subvolume's items form one run (up to 16 items), four (up to 64) or
sixteen, each summed in item order with Neumaier compensation and the runs' sums
and compensations then in order -- by its own number of items, alone, beside a
much larger subvolume, and in a list so long that fewer wavefronts share the runs.
Where sums decide (no item counts given to the launch) every subvolume is one run.
The launch function is called in the library itself; expected values are the same
steps in numpy, bit for bit."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
SYMBOL = "_ZN3bfi12launch_mergeERKNS_9MergeArgsEP12ihipStream_t"
ITEMS = [1, 2, 15, 16, 17, 33, 63, 64, 65, 66, 97, 250, 1030]


class MergeArgs(C.Structure):
    _fields_ = [(k, C.c_void_p) for k in ("item_rec", "item_split", "sub_first", "sub_rec",
                                          "sub_split")] + \
               [(k, C.c_uint32) for k in ("nsub", "nitems", "most")] + \
               [(k, C.c_int32) for k in ("nx", "d")]


def _add(total, v):
    s, c = total
    t = s + v
    return t, c + np.where(np.abs(s) >= np.abs(v), (s - t) + v, (v - t) + s)


def _merged(rows, runs):
    zero = np.zeros(rows.shape[1])
    per = -(-len(rows) // runs)
    parts = []
    for k in range(runs):
        part = (zero, zero)
        for row in rows[k * per:(k + 1) * per]:
            part = _add(part, row)
        parts.append(part)
    if runs == 1:
        return parts[0][0] + parts[0][1]
    total = (zero, zero)
    for s, c in parts:
        total = _add(_add(total, s), c)
    return total[0] + total[1]


def _runs(items):
    return 1 if items <= 16 else 4 if items <= 64 else 16


@pytest.mark.parametrize("nx,d,split", [(4, 8, False), (10, 20, True), (16, 64, False)])
@pytest.mark.parametrize("decides", [False, True])
@pytest.mark.parametrize("beside", ["alone", "larger", "long list"])
def test_order_of_the_sums(bfi, ctx, nx, d, split, decides, beside):
    torch = pytest.importorskip("torch")
    rec, spl = 4 + 3 * nx, 2 * d if split else 0
    counts = ITEMS + {"alone": [], "larger": [3000], "long list": [1] * 2100}[beside]
    lists = [ITEMS[k:k + 1] for k in range(len(ITEMS))] if beside == "alone" else [counts]
    rows = {}
    for n in counts:  # the same items whatever the list
        g = np.random.Generator(np.random.PCG64([nx, n]))
        v = g.choice([-1.0, 1.0], (n, rec + spl)) * 10.0 ** g.uniform(-20, 20, (n, rec + spl))
        v[1::2] = np.where(g.random((len(v[1::2]), rec + spl)) < 0.7, -v[0:2 * len(v[1::2]):2],
                           v[1::2])
        v = v[g.permutation(n)]
        v[:, 0], v[:, 1] = 64.0, 0.0  # samples, shift
        rows[n] = v
    merge = getattr(bfi.load(), SYMBOL)
    merge.restype, merge.argtypes = C.c_int, [C.POINTER(MergeArgs), C.c_void_p]
    for counts in lists:
        all_rows = np.concatenate([rows[n] for n in counts])
        first = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in
               (all_rows[:, :rec], all_rows[:, rec:], first)]
        out = torch.zeros((len(counts), rec), dtype=torch.float64, device="cuda")
        out_s = torch.zeros((len(counts), 1 + spl), dtype=torch.float64, device="cuda")
        a = MergeArgs(dev[0].data_ptr(), dev[1].data_ptr() if split else None, dev[2].data_ptr(),
                      out.data_ptr(), out_s.data_ptr() if split else None, len(counts),
                      0 if decides else int(sum(counts)), 0 if decides else max(counts), nx, d)
        torch.cuda.synchronize()
        print(f"merge order: {len(counts)} subvolumes, {sum(counts)} items", flush=True)
        assert merge(C.byref(a), None) == 0
        torch.cuda.synchronize()
        got = np.concatenate([out.cpu().numpy(), out_s.cpu().numpy()[:, 1:]], axis=1)
        for k, n in enumerate(counts[:len(ITEMS)]):
            want = _merged(rows[n], 1 if decides else _runs(n))
            want[1] = 0.0
            assert np.array_equal(got[k].view(np.uint64), want.view(np.uint64)), n
