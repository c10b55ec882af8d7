"""The work that a user of the library has it do, as cases that can be timed.

Every case is one call (or one batch of calls) of the public entry points on a
synthetic input: lattice, box, partition, sample counts and Philox seed.  Sizes
are those of the benchmark workloads (4x2, 10x2 and 16x4 lattices), of the
serving mix (budgets 2^16 .. 2^26), of the adaptive loop (ragged per-leaf
counts with split statistics) and of the paper's own integrand runs (10^6
samples per subvolume), and sizes between them.

``exact`` evaluates the same estimator in 64 bits with plain torch: Philox4x32-10
words, the point map, the action of the discretised equation, the weights, the
sums of each subvolume's record and the delta-method finalize.
"""
import math
import os

import numpy as np
import torch

import paper_1803_07560_amd as bfi

_TUNED = os.path.join(os.path.dirname(bfi.__file__), "tuned_gfx950.json")
_LEAVES = 1 << 14  # leaves that the adaptive runs are given room for
_context = None


def _ctx():
    """One context per process with the committed launch table, as the benchmark
    and a long-running program keep it."""
    global _context
    if _context is None:
        _context = bfi.bfi_context_create(0)
        bfi.bfi_tune_load(_context, _TUNED)
    return _context


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest request of the serving mix, called alone: latency
        {"name": "integrate_4x2_fp32", "kind": "integrate", "nx": 4, "nt": 2, "nu": 1.0,
         "obs": "anchor", "pairs": False, "prec": "fp32", "box": 4.0, "split_log2": 4,
         "budget": 1 << 16},
        # an ordinary one-off estimate, a round number of samples in decimal
        {"name": "integrate_10x2_fp64", "kind": "integrate", "nx": 10, "nt": 2, "nu": 0.5,
         "obs": "anchor", "pairs": False, "prec": "fp64", "box": 1.0, "split_log2": 6,
         "budget": 3_000_001},
        # the paper's idea: refinement where the error is, with its host rounds
        {"name": "adaptive_10x2_fp32", "kind": "adaptive", "nx": 10, "nt": 2, "nu": 1.0,
         "obs": "averaged", "pairs": False, "prec": "fp32", "box": 4.0, "split_log2": 10,
         "budget": 1 << 28},
        # a burst of requests on the continuous-batching server
        {"name": "server_burst_fp32", "kind": "server", "prec": "fp32", "requests": 16,
         "budget_lo_log2": 16, "budget_hi_log2": 22},
        # the headline benchmark: resident plan, captured replay, FP64
        {"name": "plan_10x2_fp64", "kind": "plan", "nx": 10, "nt": 2, "nu": 1.0,
         "obs": "anchor", "pairs": False, "prec": "fp64", "box": 4.0, "split_log2": 10,
         "budget": 1 << 30, "graph": True},
        # its FP32 form through to Z and C(r): run, records to the host, finalize
        {"name": "plan_10x2_fp32", "kind": "estimate", "nx": 10, "nt": 2, "nu": 1.0,
         "obs": "anchor", "pairs": False, "prec": "fp32", "box": 1.0, "split_log2": 10,
         "budget": 1 << 28, "graph": True},
        # antithetic pairs on the middle lattice of the serving mix
        {"name": "plan_8x2_pairs_fp64", "kind": "plan", "nx": 8, "nt": 2, "nu": 1.0,
         "obs": "anchor", "pairs": True, "prec": "fp64", "box": 4.0, "split_log2": 8,
         "budget": 1 << 27, "graph": False},
        # the large lattice
        {"name": "plan_16x4_fp64", "kind": "plan", "nx": 16, "nt": 4, "nu": 0.5,
         "obs": "anchor", "pairs": False, "prec": "fp64", "box": 3.0, "split_log2": 10,
         "budget": 1 << 27, "graph": True},
        # an adaptive round by hand: uneven leaves, ragged counts, split statistics
        {"name": "eval_split_10x2_fp64", "kind": "eval", "nx": 10, "nt": 2, "nu": 1.0,
         "obs": "averaged", "pairs": False, "prec": "fp64", "box": 4.0, "leaves": 301,
         "count_lo_log2": 10, "count_hi_log2": 17, "split": True},
        # the Gaussian-proposal sampler in the form the benchmark runs it
        {"name": "is_10x2_fp32", "kind": "is", "nx": 10, "nt": 2, "nu": 1.0, "obs": "anchor",
         "pairs": False, "prec": "fp32", "box": 4.0, "budget": 1 << 26, "streams": 256,
         "fraction": 0.9},
        # the sampler in spherical coordinates, pilot and main pass
        {"name": "sph_10x2_fp64", "kind": "sph", "nx": 10, "nt": 2, "nu": 1.0, "obs": "anchor",
         "pairs": False, "prec": "fp64", "box": 4.0, "budget": 1 << 24, "shells": 64,
         "fraction": 0.125},
        # one generation of the paper's subdivision driver on its test integrand
        {"name": "nsphere_6d", "kind": "nsphere", "dim": 6, "leaves": 32, "samples": 1_000_000},
    ]


def _log2_uniform(rng, lo, hi):
    """An integer between 2^lo and 2^hi, spread over the logarithm."""
    return int(round(2.0 ** rng.uniform(lo, hi)))


def draw(rng):
    kind = rng.choice(["integrate", "integrate", "plan", "estimate", "eval", "is", "sph",
                       "nsphere", "server", "adaptive"])
    prec = rng.choice(["fp64", "fp64", "fp32"])
    nu = math.exp(rng.uniform(math.log(0.05), math.log(2.0)))
    nx, nt = rng.choice([(3, 2), (4, 2), (5, 3), (8, 2), (10, 2), (16, 4)])
    obs = rng.choice(["anchor", "anchor", "averaged"])
    if kind == "server":
        return {"kind": kind, "prec": prec, "requests": rng.randint(3, 16),
                "budget_lo_log2": 14, "budget_hi_log2": rng.randint(18, 22)}
    if kind == "nsphere":
        return {"kind": kind, "dim": rng.randint(1, 16), "leaves": rng.randint(1, 64),
                "samples": _log2_uniform(rng, 12, 20)}
    small = (nx, nt) if nx * nt <= 32 else (10, 2)
    if kind in ("is", "sph"):
        case = {"kind": kind, "nx": small[0], "nt": small[1], "nu": nu, "obs": obs,
                "pairs": False, "prec": prec, "box": rng.choice([1.0, 2.5, 4.0]),
                "budget": _log2_uniform(rng, 17, 26)}
        if kind == "is":
            return case | {"streams": rng.randint(1, 256), "fraction": rng.choice([0.5, 0.9])}
        return case | {"shells": rng.randint(8, 128), "fraction": 0.125}
    if kind == "eval":
        lo = rng.randint(4, 10)
        return {"kind": kind, "nx": small[0], "nt": small[1], "nu": nu, "obs": obs,
                "pairs": False, "prec": prec, "box": rng.choice([1.0, 4.0]),
                "leaves": _log2_uniform(rng, 0, 10), "count_lo_log2": lo,
                "count_hi_log2": lo + rng.randint(1, 8), "split": rng.random() < 0.6}
    if kind == "adaptive":
        return {"kind": kind, "nx": small[0], "nt": small[1], "nu": nu, "obs": "averaged",
                "pairs": False, "prec": prec, "box": 4.0, "split_log2": rng.randint(4, 10),
                "budget": _log2_uniform(rng, 24, 28)}
    pairs = rng.random() < 0.25 and nx * nt <= 32
    case = {"kind": kind, "nx": nx, "nt": nt, "nu": nu, "obs": obs, "pairs": pairs,
            "prec": prec, "box": rng.choice([1.0, 3.0, 4.0]) if kind == "plan" else 1.0}
    if kind == "integrate":
        return case | {"split_log2": rng.randint(0, 8), "budget": _log2_uniform(rng, 13, 26)}
    big = 26 if nx * nt > 32 else 28
    return case | {"split_log2": rng.randint(0, 11), "budget": _log2_uniform(rng, 18, big),
                   "graph": rng.random() < 0.5}


# ------------------------------------------------------------------- inputs

def _lattice(case):
    return bfi.lattice(case["nx"], case["nt"], nu=case["nu"], observable=case["obs"],
                       antithetic=case["pairs"])


def _halves(d, box, k, dims=None):
    """2^k equal subvolumes of [-box, box]^d, halving dimension t mod d at level t."""
    count = 1 << k
    lo, hi = np.full((count, d), -box), np.full((count, d), box)
    b = np.arange(count)
    for t in range(k):
        j = t % d
        mid = 0.5 * (lo[:, j] + hi[:, j])
        up = ((b >> (k - 1 - t)) & 1).astype(bool)
        lo[up, j], hi[~up, j] = mid[up], mid[~up]
    return np.uint64(count) + b.astype(np.uint64), lo, hi


def _counts(total, count):
    return np.array([total // count + (i < total % count) for i in range(count)], np.uint64)


def _uneven(d, box, leaves, seed):
    """`leaves` boxes of an uneven bisection tree, in the order of their heap ids."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = [(1, np.full(d, -box), np.full(d, box))]
    while len(out) < leaves:
        hid, lo, hi = out.pop(int(rng.integers(len(out))))
        if hid >= 1 << 61:
            out.append((hid, lo, hi))
            continue
        j = int(rng.integers(d))
        mid = 0.5 * (lo[j] + hi[j])
        hi_a, lo_b = hi.copy(), lo.copy()
        hi_a[j] = lo_b[j] = mid
        out += [(2 * hid, lo, hi_a), (2 * hid + 1, lo_b, hi)]
    out.sort(key=lambda t: t[0])
    return (np.array([t[0] for t in out], np.uint64), np.stack([t[1] for t in out]),
            np.stack([t[2] for t in out]))


def _subs(case, seed):
    """(ids, lo, hi, n) of a case over subvolumes, as numpy arrays."""
    kind = case["kind"]
    if kind == "nsphere":
        d, count = case["dim"], case["leaves"]
        ids, lo, hi = _uneven(d, 1.0, count, seed)
        return ids, lo, hi, np.full(count, case["samples"], np.uint64)
    d = case["nx"] * case["nt"]
    if kind == "eval":
        ids, lo, hi = _uneven(d, case["box"], case["leaves"], seed)
        rng = np.random.Generator(np.random.PCG64(seed + 1))
        e = rng.uniform(case["count_lo_log2"], case["count_hi_log2"], size=len(ids))
        return ids, lo, hi, np.maximum(2, np.round(2.0 ** e)).astype(np.uint64)
    ids, lo, hi = _halves(d, case["box"], case["split_log2"])
    total = case["budget"] // 2 if case["pairs"] else case["budget"]
    return ids, lo, hi, _counts(total, len(ids))


def _requests(case, seed):
    """A burst of the serving mix: the four lattices in turn, viscosity and
    budget spread over their logarithms."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    for i in range(case["requests"]):
        nx, nt = ((4, 2), (8, 2), (10, 2), (16, 4))[i % 4]
        nu = float(math.exp(rng.uniform(math.log(0.05), math.log(2.0))))
        budget = 2.0 ** rng.uniform(case["budget_lo_log2"], case["budget_hi_log2"])
        out.append({"kind": "integrate", "nx": nx, "nt": nt, "nu": nu, "obs": "anchor",
                    "pairs": False, "prec": case["prec"], "box": 1.0,
                    "split_log2": 4, "budget": int(round(budget / 16.0)) * 16,
                    "seed": int(rng.integers(1, 1 << 40))})
    return out


class _Plan:
    """A resident plan, destroyed with the state that keeps it."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        bfi.bfi_plan_destroy(self.handle)


class _Server:
    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        bfi.bfi_server_destroy(self.handle)


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case, "ctx": _ctx(), "seed": int(seed) + 1}
    if kind == "server":
        state["server"] = _Server(bfi.bfi_server_create(
            state["ctx"], bfi.server_config(memory_budget=8 << 30, max_requests=256)))
        state["requests"] = [
            bfi.request(_lattice(r), r["prec"], r["seed"], r["box"], r["split_log2"], r["budget"])
            for r in _requests(case, seed)]
        return state
    if kind == "nsphere":
        state["integrand"] = bfi.integrand_nsphere(case["dim"])
    else:
        state["lat"] = _lattice(case)
    if kind in ("plan", "estimate", "eval", "nsphere"):
        ids, lo, hi, n = _subs(case, seed)
        state["subs"] = bfi.Subvolumes(ids, lo, hi, n, 0, lo.shape[1])
    if kind in ("plan", "estimate"):
        state["plan"] = _Plan(bfi.bfi_plan_create(
            state["ctx"], state["lat"], case["prec"], state["subs"],
            bfi.launch(use_graph=int(case["graph"]))))
        state["out"] = torch.empty((len(state["subs"]), bfi.partial_len(case["nx"])),
                                   dtype=torch.float64, device="cuda")
    if kind == "adaptive":
        budget = case["budget"]
        state["config"] = bfi.adaptive_config(
            target_rel_err=1e-6, max_evals=budget, n_min=1 << 12, n_max=1 << 20,
            split_log2=case["split_log2"], max_rounds=24, refine_fraction=0.5,
            round_evals=budget // 8, split_samples=1 << 14)
    return state


# --------------------------------------------------------------------- runs

def _plain(result):
    """A result without the values that say nothing about the estimate."""
    return {k: result[k] for k in ("Z", "Z_err", "log_Z", "ess", "n_evals", "C", "C_err")}


def _together(results):
    """Results of several requests, one array for each value."""
    return {k: np.concatenate([np.atleast_1d(r[k]) for r in results]) for k in results[0]}


def run(state):
    case, ctx, seed = state["case"], state["ctx"], state["seed"]
    kind = case["kind"]
    if kind == "integrate":
        return _plain(bfi.bfi_integrate(ctx, state["lat"], case["prec"], seed, -case["box"],
                                        case["box"], case["split_log2"], case["budget"]))
    if kind == "plan":
        bfi.bfi_plan_run(state["plan"].handle, seed, state["out"])
        return state["out"]
    if kind == "estimate":
        bfi.bfi_plan_run(state["plan"].handle, seed)
        rec = bfi.bfi_plan_partials(state["plan"].handle, len(state["subs"]), case["nx"])
        return _plain(bfi.bfi_finalize(state["lat"], state["subs"], rec))
    if kind == "eval":
        got = bfi.bfi_eval(ctx, state["lat"], case["prec"], seed, state["subs"],
                           split=case["split"])
        return list(got) if case["split"] else [got]
    if kind == "nsphere":
        value, err, dim = bfi.bfi_integrand_eval(ctx, state["integrand"], seed, state["subs"])
        return {"value": value, "err": err, "dim": dim}
    if kind == "is":
        return _plain(bfi.bfi_integrate_is(ctx, state["lat"], case["prec"], seed, -case["box"],
                                           case["box"], case["budget"], case["fraction"],
                                           case["streams"]))
    if kind == "sph":
        return _plain(bfi.bfi_integrate_sph(ctx, state["lat"], case["prec"], seed, case["box"],
                                            case["shells"], case["budget"], case["fraction"]))
    if kind == "server":
        srv = state["server"].handle
        tickets = [bfi.bfi_server_submit(srv, r) for r in state["requests"]]
        return _together([_plain(bfi.bfi_server_wait(srv, t, 120.0)[0]) for t in tickets])
    got = bfi.bfi_integrate_adaptive(ctx, state["lat"], case["prec"], seed, -case["box"],
                                     case["box"], state["config"], leaf_capacity=_LEAVES)
    # the partition in arrays of one size, whatever number of leaves the run ends with
    leaves = np.zeros((2, _LEAVES), np.int64)
    part = got["partition"]
    leaves[0, :len(part)], leaves[1, :len(part)] = part.ids, part.n
    return _plain(got) | {"rel_err": got["rel_err"], "rounds": got["rounds"],
                          "leaves": got["leaves"], "evals": got["evals"], "partition": leaves}


# --------------------------------------------------------------------- work

def _per_evaluation(case):
    """Floating-point operations of one evaluation: point map, action, weight
    (a 13-term exponential) and the record's sums."""
    nx, d = case["nx"], case["nx"] * case["nt"]
    r = nx // 2 + 1 if case["obs"] == "averaged" else nx
    ops = 2 * d + 10 * d + 36 + 3 + 6 * r
    if case["obs"] == "averaged":
        ops += 2 * d * r
    if case.get("split"):
        ops += 4 * d
    if case["kind"] in ("is", "sph"):
        ops += 40 * d  # a normal per variable: logarithm, root, sine or cosine
    if case["kind"] == "is":
        ops += 2 * d * (nx + case["nt"]) + 3 * d
    return ops


def work(case):
    kind = case["kind"]
    if kind == "server":
        parts = [work(r) for r in _requests(case, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if kind == "nsphere":
        n, count, d = case["samples"] * case["leaves"], case["leaves"], case["dim"]
        return {"bytes": count * (24 + 16 * d + 20), "flops": n * (8 * d + 20)}
    d, rec = case["nx"] * case["nt"], 8 * bfi.partial_len(case["nx"])
    if kind == "eval":
        count = case["leaves"]
        n = count * 2.0 ** (0.5 * (case["count_lo_log2"] + case["count_hi_log2"]))
    else:
        n = case["budget"]
        count = (2 * case["streams"] if kind == "is" else case["shells"] if kind == "sph"
                 else 1 << case["split_log2"])
    out = rec + (8 * bfi.split_len(d) if case.get("split") else 0)
    return {"bytes": count * (24 + 16 * d + out), "flops": n * _per_evaluation(case)}


# -------------------------------------------------- the same in 64-bit torch

_M32 = 0xFFFFFFFF


def _philox(index, blocks, ids, seed):
    """Philox4x32-10 words (4 * blocks, m) of samples `index` of streams `ids`."""
    dev = index.device
    q = index[None, :] * blocks + torch.arange(blocks, device=dev)[:, None]
    c0, c1 = q & _M32, (q >> 32) & _M32
    c2 = (ids & _M32)[None, :].expand_as(c0)
    c3 = ((ids >> 32) & _M32)[None, :].expand_as(c0)
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((b >> 32) & _M32) ^ c1 ^ k0, b & _M32,
                          ((a >> 32) & _M32) ^ c3 ^ k1, a & _M32)
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return torch.stack((c0, c1, c2, c3), 1).reshape(4 * blocks, -1)


def _unit(x):
    return x.double() * 2.0 ** -32 + 2.0 ** -33


def _normals(words, d):
    """Box-Muller: coordinate k from the pair of words 2 floor(k/2), 2 floor(k/2) + 1."""
    pairs = (d + 1) // 2
    radius = torch.sqrt(-2.0 * torch.log(_unit(words[0:2 * pairs:2])))
    turn = 2.0 * math.pi * _unit(words[1:2 * pairs:2])
    z = torch.stack((radius * torch.cos(turn), radius * torch.sin(turn)), 1)
    return z.reshape(2 * pairs, -1)[:d]


def _action(u, case):
    """The action of lattice fields u (nt, nx, m), D = a = tau = g = 1."""
    right, left = torch.roll(u, -1, 1), torch.roll(u, 1, 1)
    res = (torch.roll(u, -1, 0) - u + 0.5 * u * (right - left)
           - case["nu"] * (right - 2.0 * u + left))
    return 0.5 * (res * res).sum((0, 1))


def _products(u, case):
    """p_r of lattice fields u (nt, nx, m): (nx, m)."""
    if case["obs"] == "anchor":
        return u[0, 0][None] * u[0]
    return torch.stack([(u * torch.roll(u, -r, 1)).mean((0, 1)) for r in range(case["nx"])])


def _rows(w, pw):
    """Summands of a record after its count and shift, for weights w and products p_r w."""
    return torch.cat((w[None], (w * w)[None], pw, pw * pw, pw * w))


def _pieces(n, most):
    """The samples of streams of n[s] samples in pieces: (owner, index) tensors."""
    owner, index, size = [], [], 0
    for s, k in enumerate(int(v) for v in n):
        start = 0
        while start < k:
            take = min(k - start, most - size)
            owner.append(torch.full((take,), s, dtype=torch.int64, device="cuda"))
            index.append(torch.arange(start, start + take, device="cuda"))
            start += take
            size += take
            if size == most:
                yield torch.cat(owner), torch.cat(index)
                owner, index, size = [], [], 0
    if size:
        yield torch.cat(owner), torch.cat(index)


def _records(case, seed, ids, n, summands, rows, offset=None):
    """Sums over every stream's samples: summands(owner, index, ids) -> (rows, m)."""
    width = case["dim"] if case["kind"] == "nsphere" else case["nx"] * case["nt"]
    id64 = torch.from_numpy(ids.view(np.int64)).cuda()
    first = torch.zeros(len(ids), dtype=torch.int64, device="cuda")
    if offset is not None:
        first += torch.from_numpy(offset.astype(np.int64)).cuda()
    total = torch.zeros((len(ids), rows), dtype=torch.float64, device="cuda")
    for owner, index in _pieces(n, (1 << 24) // max(width, 4)):
        values = summands(owner, index + first[owner], id64[owner])
        low, high = int(owner[0]), int(owner[-1])
        if high - low < 256:  # streams are consecutive: a slice for each
            ends = torch.searchsorted(owner, torch.arange(low, high + 1, device="cuda"),
                                      right=True).tolist()
            for s, a, b in zip(range(low, high + 1), [0] + ends, ends):
                total[s] += values[:, a:b].sum(1)
        else:
            total.index_add_(0, owner, values.t().contiguous())
    head = torch.zeros((len(ids), 2), dtype=torch.float64, device="cuda")
    head[:, 0] = torch.from_numpy(n.astype(np.float64)).cuda()
    return torch.cat((head, total), 1).cpu().numpy()


def _box_records(case, seed, ids, lo, hi, n):
    """Records (and split statistics) of the plain sampler over boxes."""
    nx, nt = case["nx"], case["nt"]
    d, blocks = nx * nt, (nx * nt + 3) // 4
    scale = torch.from_numpy((hi - lo) * 2.0 ** -32).cuda().t().contiguous()
    base = torch.from_numpy(lo.copy()).cuda().t().contiguous() + 0.5 * scale
    split = bool(case.get("split"))

    def weigh(words, owner):
        u = (words.double() * scale[:, owner] + base[:, owner]).view(nt, nx, -1)
        w = torch.exp(-_action(u, case))
        return w, _products(u, case) * w

    def summands(owner, index, id64):
        words = _philox(index, blocks, id64, seed)[:d]
        w, pw = weigh(words, owner)
        if case["pairs"]:
            w2, pw2 = weigh(_M32 - words, owner)
            w, pw = 0.5 * (w + w2), 0.5 * (pw + pw2)
        rows = _rows(w, pw)
        if split:
            up = (words >> 31).double()
            rows = torch.cat((rows, up * w, up * (w * w)))
        return rows

    rec = 2 + 3 * nx
    got = _records(case, seed, ids, n, summands, rec + (2 * d if split else 0))
    return got[:, :2 + rec], got[:, 2 + rec:]


def _finalize(nx, rec, volume, per_sample=1):
    """Z, C(r) and their errors from unshifted records (the delta method)."""
    n, sw, sw2 = rec[:, 0], rec[:, 2], rec[:, 3]
    sp, sp2, spw = (rec[:, 4 + k * nx:4 + (k + 1) * nx] for k in range(3))
    v2 = volume ** 2 / (n * (n - 1.0))
    z = np.float64(math.fsum(volume * sw / n))
    var_z = v2 * (sw2 - sw * sw / n)
    num = np.array([math.fsum(volume * sp[:, r] / n) for r in range(nx)])
    c = num / z
    err = []
    for r in range(nx):
        var_n = v2 * (sp2[:, r] - sp[:, r] ** 2 / n)
        cov = v2 * (spw[:, r] - sp[:, r] * sw / n)
        err.append(math.sqrt(max(math.fsum(var_n - 2.0 * c[r] * cov + c[r] ** 2 * var_z), 0.0)))
    return {"Z": z, "Z_err": math.sqrt(max(math.fsum(var_z), 0.0)), "log_Z": float(np.log(z)),
            "ess": z * z / math.fsum((volume / n) ** 2 * sw2),
            "n_evals": float(n.sum()) * per_sample, "C": c, "C_err": np.array(err) / abs(z)}


def _exact_boxes(case, seed, input_seed):
    ids, lo, hi, n = _subs(case, input_seed)
    rec, split = _box_records(case, seed, ids, lo, hi, n)
    kind = case["kind"]
    if kind == "plan":
        return rec if case["prec"] == "fp64" else None
    if kind == "eval":
        if case["prec"] != "fp64":
            return None  # a shifted record's scale is the kernel's choice
        if not case["split"]:
            return [rec]
        return [rec, np.concatenate((np.zeros((len(ids), 1)), split), 1)]
    return _finalize(case["nx"], rec, np.prod(hi - lo, 1), 2 if case["pairs"] else 1)


def _exact_nsphere(case, seed, input_seed):
    ids, lo, hi, n = _subs(case, input_seed)
    d = case["dim"]
    scale = torch.from_numpy((hi - lo) * 2.0 ** -32).cuda().t().contiguous()
    base = torch.from_numpy(lo.copy()).cuda().t().contiguous() + 0.5 * scale

    def summands(owner, index, id64):
        words = _philox(index, (d + 3) // 4, id64, seed)[:d]
        x = words.double() * scale[:, owner] + base[:, owner]
        f = torch.sqrt(torch.clamp(1.0 - (x * x).sum(0), min=0.0))
        up = (words >> 31).double()
        return torch.cat((f[None], (f * f)[None], up * f, up * (f * f)))

    rec = _records(case, seed, ids, n, summands, 2 + 2 * d)
    k, s1, s2 = rec[:, 0], rec[:, 2], rec[:, 3]
    volume = np.prod(hi - lo, 1)
    var = np.maximum(s2 - s1 * s1 / k, 0.0) / (k - 1.0)
    half, up1, up2 = 0.5 * k[:, None], rec[:, 4:4 + d], rec[:, 4 + d:]
    low1, low2 = s1[:, None] - up1, s2[:, None] - up2
    spread = (np.sqrt(np.maximum(up2 / half - (up1 / half) ** 2, 0.0))
              + np.sqrt(np.maximum(low2 / half - (low1 / half) ** 2, 0.0)))
    return {"value": volume * s1 / k, "err": volume * np.sqrt(var / k),
            "dim": np.argmin(spread, 1).astype(np.int32)}


def _fourier(n):
    """The real orthonormal Fourier basis of period n, one vector a row."""
    m = np.arange(n)
    rows = [np.full(n, 1.0 / math.sqrt(n))]
    for b in range(1, n):
        k = (b + 1) // 2
        if n % 2 == 0 and b == n - 1:
            rows.append((-1.0) ** m / math.sqrt(n))
        else:
            f = np.cos if b % 2 else np.sin
            rows.append(math.sqrt(2.0 / n) * f(2.0 * math.pi * ((k * m) % n) / n))
    return np.stack(rows)


def _exact_is(case, seed):
    nx, nt, box = case["nx"], case["nt"], case["box"]
    d, c, alpha, budget = nx * nt, case["nu"], case["fraction"], case["budget"]
    kt, kx = (np.arange(nt) + 1) // 2, (np.arange(nx) + 1) // 2
    mt = (2.0 * np.cos(2.0 * math.pi * kt / nt) - 2.0)[:, None]
    mx = (2.0 * np.cos(2.0 * math.pi * kx / nx) - 2.0)[None, :]
    lam = (-mt - c * mt * mx + c * c * mx * mx).reshape(-1)
    reach = math.sqrt(d * box * box)
    flat = lam[0] * reach ** 2 < 4.0
    scale = np.where(lam * reach ** 2 <= 1.0, reach, 1.0 / np.sqrt(np.maximum(lam, 1e-300)))
    log_k = float(np.sum(0.5 * math.log(2.0 * math.pi) + np.log(scale)))
    if flat:
        scale[0] = reach
        log_k = math.log(2.0 * reach) + float(
            np.sum(0.5 * math.log(2.0 * math.pi) + np.log(scale[1:])))
    basis = torch.from_numpy(np.kron(_fourier(nt), _fourier(nx))).cuda()
    width = torch.from_numpy(scale).cuda()[:, None]
    log_ga = math.log(alpha)
    log_un = math.log1p(-alpha) + log_k - d * math.log(2.0 * box)
    step = 2.0 * box * 2.0 ** -32
    first = 1 if flat else 0

    def weigh(u, half_z2, inside):
        f = u.view(nt, nx, -1)
        mix = torch.logaddexp(log_ga - half_z2, torch.full_like(half_z2, log_un))
        w = torch.where(inside, torch.exp(-(_action(f, case) + mix)), 0.0)
        return _rows(w, _products(f, case) * w)

    def gaussian(owner, index, id64):
        words = _philox(index, (2 * ((d + 1) // 2) + 4) // 4, id64, seed)
        z = _normals(words, d)
        a = z * width
        if flat:
            a[0] = reach * (2.0 * _unit(words[2 * ((d + 1) // 2)]) - 1.0)
        u = basis.t() @ a
        return weigh(u, 0.5 * (z[first:] ** 2).sum(0), (u.abs() <= box).all(0))

    def uniform(owner, index, id64):
        words = _philox(index, (d + 3) // 4, id64, seed)[:d]
        u = words.double() * step + (0.5 * step - box)
        z = (basis @ u) / width
        return weigh(u, 0.5 * (z[first:] ** 2).sum(0),
                     torch.ones(u.shape[1], dtype=torch.bool, device=u.device))

    share = int(math.floor(alpha * budget + 0.5))
    recs = []
    for total, bit, summands in ((share, 0, gaussian), (budget - share, 1 << 63, uniform)):
        ids = np.array([bit + 1 + i for i in range(case["streams"])], np.uint64)
        recs.append(_records(case, seed, ids, _counts(total, case["streams"]), summands,
                             2 + 3 * nx))
    rec = np.concatenate(recs)
    return _finalize(nx, rec, math.exp(log_k) * rec[:, 0] / budget)


def _exact_sph(case, seed):
    nx, nt, box, count = case["nx"], case["nt"], case["box"], case["shells"]
    d, budget = nx * nt, case["budget"]
    rmax = box * math.sqrt(float(d))
    low = np.array([rmax * s / count for s in range(count)])
    high = np.array([rmax * (s + 1) / count for s in range(count)])
    inner = (low / high) ** d
    volume = np.exp(0.5 * d * math.log(math.pi) - math.lgamma(0.5 * d + 1.0)
                    + d * np.log(high)) * (1.0 - inner)
    outer_t, inner_t = torch.from_numpy(high).cuda(), torch.from_numpy(inner).cuda()
    pairs = (d + 1) // 2

    def summands(owner, index, id64):
        words = _philox(index, (2 * pairs + 4) // 4, id64, seed)
        z = _normals(words, d)
        t = inner_t[owner]
        rho = outer_t[owner] * (t + _unit(words[2 * pairs]) * (1.0 - t)) ** (1.0 / d)
        u = z * (rho / torch.sqrt((z * z).sum(0)))
        f = u.view(nt, nx, -1)
        w = torch.where((u.abs() <= box).all(0), torch.exp(-_action(f, case)), 0.0)
        return _rows(w, _products(f, case) * w)

    ids = np.arange(1, count + 1).astype(np.uint64)
    pilot = int(case["fraction"] * budget) // count
    rec = _records(case, seed, ids, np.full(count, pilot, np.uint64), summands, 2 + 3 * nx)
    mean, square = rec[:, 2] / pilot, rec[:, 3] / pilot
    share = volume * np.sqrt(np.maximum(square - mean * mean, 0.0))
    rest = max(budget - pilot * count, 0)
    more = (share / share.sum() * rest).astype(np.uint64)
    keep = more >= 2
    if keep.any():
        rec[keep] += _records(case, seed, ids[keep], more[keep],
                              lambda owner, index, id64: summands(id64 - 1, index, id64),
                              2 + 3 * nx, np.full(int(keep.sum()), pilot))
    return _finalize(nx, rec, volume)


def exact(case, seed):
    kind, philox_seed = case["kind"], int(seed) + 1
    if kind == "adaptive":
        return None
    if kind == "server":
        return _together([_exact_boxes(r, r["seed"], 0) for r in _requests(case, seed)])
    if kind == "nsphere":
        return _exact_nsphere(case, philox_seed, seed)
    if case["budget" if "budget" in case else "leaves"] * case["nx"] * case["nt"] > 24 << 30:
        return None  # beyond about ten seconds
    if kind == "is":
        return _exact_is(case, philox_seed)
    if kind == "sph":
        return _exact_sph(case, philox_seed)
    return _exact_boxes(case, philox_seed, seed)
