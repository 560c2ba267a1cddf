"""What a user of the planner has it do, as cases that can be timed and compared.

A case names one use of the public entry points (`op`) and the training iteration whose
allocation trace it works on (schedule, layers, micro-batches, sizes).  Traces imitate profiled
iterations the way workloads/traces.py does -- few distinct sizes, persistent / scoped / transient
tensors, pipeline schedules, recomputation, routed experts -- but are drawn from a seed, so that
every seed is another iteration.  A tick of several events is a profiler with a coarse clock.
"""
from __future__ import annotations

import bisect
import heapq
import math

import numpy as np
import torch

import paper_2507_16274_amd as S

ROUND = 512                                   # trace producers round sizes up to this many bytes
SMALL = (512, 1024, 1536, 2048, 3072, 4096, 6144, 8192, 12288, 16384, 24576, 32768, 40960, 49152, 57344, 65536)
RECOMPUTED = (1, 2, 4, 5, 7, 8, 10)           # of a layer's 12 forward tensors, those dropped and made again

TRACE = {"kind": "dense", "layers": 32, "chunks": 1, "micro_batches": 8, "hidden": 4096, "seq": 4096, "heads": 32,
         "experts": 0, "small": 0, "persistent": 0, "tick": 1}


def _case(name, op, **more):
    return {"name": name, "op": op, **TRACE, **more}


def listed():
    dense = {"kind": "dense", "layers": 32, "micro_batches": 8, "hidden": 4096, "seq": 4096, "heads": 32}
    recompute = {"kind": "recompute", "layers": 80, "micro_batches": 8, "hidden": 8192, "seq": 4096, "heads": 64}
    moe = {"kind": "moe", "layers": 16, "micro_batches": 8, "hidden": 4096, "seq": 8192, "experts": 64, "heads": 0}
    interleaved = {"kind": "interleaved", "layers": 16, "chunks": 4, "micro_batches": 8, "hidden": 8192, "seq": 8192,
                   "small": 183, "heads": 0}
    return [
        # a two-layer model, planned interactively or in a test: launches are all there is
        _case("plan_tiny", "plan", kind="tiny", layers=2, micro_batches=1, hidden=512, seq=512, heads=0, plans=64, offsets=True),
        # one pipeline stage of a dense model: the ordinary call
        _case("plan_dense", "plan", plans=1024, offsets=True, **dense),
        # the same stage at a sequence length that is no power of two: sizes share a small granule only
        _case("plan_ragged", "plan", plans=512, offsets=True, **{**dense, "seq": 4000}),
        # a deep stage with selective recomputation
        _case("plan_recompute", "plan", plans=512, offsets=True, **recompute),
        # an expert-parallel stage: over a thousand distinct sizes, a third of the requests long-lived
        _case("plan_moe", "plan", plans=256, offsets=True, **moe),
        # the largest: an interleaved schedule with 200k requests under the whole family of orders
        _case("plan_interleaved", "plan", plans=4096, offsets=True, **interleaved),
        # the check of a finished plan before it is handed to an allocator (a few decisions are damaged)
        _case("validate_best", "validate", plans=1, **interleaved),
        # what the plans are judged by: the lower bound of the trace and Eq. 2 of every plan
        _case("bounds_dense", "bounds", plans=1024, **dense),
        # candidate orders for a search over the largest trace
        _case("orders_interleaved", "orders", plans=256, **interleaved),
        # the memory-layers of the HomoSize groups of the largest trace
        _case("layers_interleaved", "layers", **interleaved),
        # dynamic requests of an iteration asking for the room that is idle during their lifetime
        _case("reusable_interleaved", "reusable", windows=4096, most=64, **interleaved),
        # all candidate fusions of HomoPhase groups of a stage
        _case("fuse_interleaved", "fuse", **interleaved),
    ]


def _spread(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _requests(c):
    """About how many requests the trace of a case has."""
    passes = c["layers"] * c["chunks"] * c["micro_batches"]
    per = {"tiny": 48, "dense": 24, "recompute": 31, "moe": 6 + 6 * c["experts"], "interleaved": 24 + 2 * c["small"]}[c["kind"]]
    return passes * per + c["persistent"]


def draw(rng):
    op = rng.choice(("plan", "plan", "plan", "plan", "plan", "validate", "validate", "bounds", "orders", "layers", "reusable", "fuse"))
    kind = rng.choice(("tiny", "dense", "dense", "recompute", "moe", "interleaved"))
    c = {"op": op, **TRACE, "kind": kind}
    if kind == "tiny":
        c.update(layers=rng.randint(1, 8), micro_batches=1, hidden=512, seq=rng.choice((512, 384, 1000)), heads=0)
    elif kind == "dense":
        c.update(layers=_spread(rng, 2, 48), micro_batches=rng.randint(1, 8), hidden=rng.choice((2048, 4096, 5120, 8192)),
                 seq=rng.choice((2048, 4096, 4096, 4000, 8192)), heads=rng.choice((0, 32)), persistent=rng.choice((0, 0, 64, 256)),
                 tick=rng.choice((1, 1, 1, 4)))
    elif kind == "recompute":
        c.update(layers=_spread(rng, 4, 80), micro_batches=rng.randint(2, 8), hidden=8192, seq=4096, heads=64,
                 tick=rng.choice((1, 1, 1, 8)))
    elif kind == "moe":
        c.update(layers=_spread(rng, 1, 16), micro_batches=rng.randint(2, 8), hidden=4096, seq=rng.choice((4096, 8192)), heads=0,
                 experts=rng.choice((8, 16, 32, 64)), persistent=rng.choice((0, 0, 128)), tick=rng.choice((1, 1, 8)))
    else:
        c.update(layers=_spread(rng, 2, 16), chunks=rng.choice((2, 4)), micro_batches=rng.choice((4, 8)), hidden=8192,
                 seq=rng.choice((4096, 8192)), heads=0, small=rng.randint(61, 183))
    n = _requests(c)
    if op == "plan":
        most = min(2048, 8 * 10 ** 6 // n, 5 * 10 ** 11 // (n * n))
        if kind == "interleaved" and n > 12000:
            most = min(2048, 2 * 10 ** 8 // n)
        c.update(plans=_spread(rng, 1, max(1, most)), offsets=rng.random() < 0.5)
    elif op == "validate":
        c.update(plans=_spread(rng, 1, max(1, min(2048, 2 * 10 ** 10 // (n * n)))))
    elif op == "bounds":
        c.update(plans=_spread(rng, 1, 4096))
    elif op == "orders":
        c.update(plans=_spread(rng, 1, max(1, min(4096, 5 * 10 ** 7 // n))))
    elif op == "reusable":
        c.update(windows=_spread(rng, 1, 4096), most=rng.choice((16, 64)))
    return c


# ---------------------------------------------------------------------------------------------
# traces

def _schedule(c):
    """(forward?, micro-batch, chunk) in execution order: 1F1B, interleaved when there are chunks."""
    m, v = c["micro_batches"], c["chunks"]
    if v == 1:
        total, f, b = m, (lambda k: (True, k, 0)), (lambda k: (False, k, 0))
        warm = min(3, m)
    else:
        depth, total = 4, m * v
        mb = lambda k: (k // (depth * v)) * depth + k % depth                                   # noqa: E731
        f = lambda k: (True, mb(k), (k // depth) % v)                                           # noqa: E731
        b = lambda k: (False, mb(k), v - 1 - (k // depth) % v)                                  # noqa: E731
        warm = min((depth - 1) * 2 + (v - 1) * depth, total)
    seq = [f(k) for k in range(warm)]
    for k in range(total - warm):
        seq += [f(warm + k), b(k)]
    return seq + [b(k) for k in range(total - warm, total)]


def _trace(c, seed):
    """size, t_alloc, t_free, t_end and the phases of allocation and release, as numpy arrays."""
    kind, layers = c["kind"], c["layers"]
    rng = np.random.default_rng([seed, 17, layers, c["micro_batches"], c["seq"], c["small"], c["experts"]])
    act = c["seq"] * c["hidden"] * 2
    score = c["heads"] * c["seq"] * c["seq"] // 2
    many = 2 * _requests(c) + 4096
    longest = 3 if kind == "tiny" else 5
    next_size = iter((rng.choice((1, 2, 3, 4) if kind == "tiny" else (1, 3, 4, 8), many) * act).tolist()).__next__
    next_small = iter(rng.choice(SMALL, many if c["small"] else 1).tolist()).__next__
    if c["op"] == "fuse":                     # the groups, and so the shapes of the outputs, are the model's: only sizes are drawn anew
        rng = np.random.default_rng(17)
    next_life = iter(rng.integers(1, longest + 1, many).tolist()).__next__
    next_coin = iter(rng.random(many).tolist()).__next__
    size, ta, tf, ps, pe = [], [], [], [], []
    due, clock, phase = {}, 0, 0

    def free(i):
        nonlocal clock
        tf[i], pe[i] = clock, phase
        clock += 1

    def alloc(s):
        nonlocal clock
        i = len(size)
        for j in due.pop(i, ()):
            free(j)
        size.append(s)
        ta.append(clock)
        tf.append(-1)
        ps.append(phase)
        pe.append(-1)
        clock += 1
        return i

    def transient(s):                         # released after a few more allocations
        i = alloc(s)
        due.setdefault(i + next_life() + 1, []).append(i)

    scoped, again, routed, to_the_end = {}, {}, {}, []
    persistent = [alloc(next_size()) for _ in range(c["persistent"])]
    schedule = _schedule(c)
    last = {ch: k for k, (fwd, _, ch) in enumerate(schedule) if not fwd}
    for phase, (fwd, mb, ch) in enumerate(schedule):
        span = range(ch * layers, (ch + 1) * layers)
        for layer in span if fwd else reversed(span):
            at = (mb, layer)
            if fwd:
                keep = scoped[at] = []
                if kind in ("tiny", "dense"):
                    for j in range(12):
                        s = score if score and j == 5 else next_size()
                        transient(s) if next_coin() < 0.3 else keep.append(alloc(s))
                elif kind == "recompute":
                    dropped = []
                    for j in range(12):
                        s = score if score and j == 5 else next_size()
                        i = alloc(s)
                        (dropped if j in RECOMPUTED else keep).append(i)
                    for i in reversed(dropped):
                        free(i)
                    again[at] = [size[i] for i in dropped]
                elif kind == "moe":
                    for j in range(6):
                        s = next_size()
                        transient(s) if next_coin() < 0.3 else keep.append(alloc(s))
                    tokens = rng.multinomial(2 * c["seq"], rng.dirichlet(np.full(c["experts"], 0.5))).tolist()
                    routed[at] = sizes = [max(1, t) * c["hidden"] * 2 for t in tokens]
                    for s in sizes:
                        keep.append(alloc(s))
                        transient(s)
                        keep.append(alloc(s))
                else:
                    for j in range(12 + c["small"]):
                        if j % 16 == 0 and j < 192:
                            s = next_size()
                            transient(s) if next_coin() < 0.3 else keep.append(alloc(s))
                        else:
                            transient(next_small())
            else:
                keep = scoped.pop(at)
                remade = [alloc(s) for s in again.pop(at, ())]
                if kind == "moe":
                    for s in reversed(routed.pop(at)):
                        for _ in range(3):
                            transient(s)
                        if keep:
                            free(keep.pop())
                elif kind == "interleaved":
                    for j in range(12 + c["small"]):
                        if j % 16 == 0 and j < 192:
                            transient(next_size())
                            if keep:
                                free(keep.pop())
                        else:
                            transient(next_small())
                else:
                    for j in range(12):
                        transient(score if score and j == 5 else next_size())
                        if kind == "tiny":
                            to_the_end.append(alloc(next_size()))          # weight gradient
                        if keep:
                            free(keep.pop())
                while keep:
                    free(keep.pop())
                for i in reversed(remade):
                    free(i)
        if not fwd and kind == "interleaved" and last[ch] == phase:
            to_the_end.append(alloc(25 << 20))                              # gradient bucket
    phase = len(schedule)                                                  # optimizer step
    for _ in range(layers * c["chunks"]):
        if kind == "tiny":
            for _ in range(12):
                transient(next_size())
        elif kind == "interleaved":
            transient(24 * c["hidden"] * c["hidden"] * 4)
    for k in sorted(due):
        for i in due[k]:
            free(i)
    for i in reversed(to_the_end):
        free(i)
    for i in reversed(persistent):
        free(i)
    size = (np.asarray(size, np.int64) + ROUND - 1) // ROUND * ROUND
    ta, tf = np.asarray(ta, np.int64) // c["tick"], np.asarray(tf, np.int64) // c["tick"]
    tf = np.maximum(tf, ta + 1)               # a lifetime below the clock's tick still holds its memory for one
    return size, ta.astype(np.int32), tf.astype(np.int32), int(tf.max()), np.asarray(ps), np.asarray(pe)


def _online_plan(size, ta, tf):
    """Addresses an online first-fit allocator would have handed out: a finished plan without conflicts."""
    n = len(size)
    when = np.concatenate([tf.astype(np.int64) * 2, ta.astype(np.int64) * 2 + 1])
    events = np.argsort(when, kind="stable").tolist()
    s, at = size.tolist(), [0] * n
    holes, ends = [0], [1 << 62]              # free ranges by address
    for e in events:
        if e >= n:
            i = e - n
            k = 0
            while ends[k] - holes[k] < s[i]:
                k += 1
            at[i] = holes[k]
            holes[k] += s[i]
            if holes[k] == ends[k]:
                del holes[k], ends[k]
        else:
            lo, hi = at[e], at[e] + s[e]
            k = bisect.bisect_left(holes, lo)
            if k < len(holes) and holes[k] == hi:
                holes[k] = lo
                if k and ends[k - 1] == lo:
                    ends[k - 1] = ends[k]
                    del holes[k], ends[k]
            elif k and ends[k - 1] == lo:
                ends[k - 1] = hi
            else:
                holes.insert(k, lo)
                ends.insert(k, hi)
    return np.asarray(at, np.int64)


def _plans(c, seed, size, ta, tf):
    """P finished plans [P][n], a few decisions of every other one damaged."""
    base = _online_plan(size, ta, tf)
    P, n = c["plans"], len(size)
    plans = base[None, :] + (np.arange(P, dtype=np.int64) * ROUND)[:, None]
    rng = np.random.default_rng([seed, 23])
    for p in range(0, P, 2):
        i, j = rng.integers(0, n, 8), rng.integers(0, n, 8)
        plans[p, i] = plans[p, j]
    return plans


def _windows(c, seed, t_end):
    """Half-open windows: short spans of a layer are common, spans of a quarter iteration exist."""
    rng = np.random.default_rng([seed, 29])
    k = c["windows"]
    length = np.clip(np.exp(rng.uniform(math.log(2.0), math.log(max(2.0, t_end // 4)), k)).astype(np.int64), 1, t_end)
    lo = rng.integers(0, t_end, k)
    hi = np.minimum(lo + length, t_end)
    return np.stack([np.minimum(lo, hi - 1), hi], axis=1).astype(np.int32)


def _pairs(ps, pe):
    """Candidate fusions: members, where each pair begins, the first group's share, the largest pair.
    A pair is two HomoPhase groups, the second allocated in the phase in which the first is released."""
    key = ps * (1 << 20) + pe
    order = np.argsort(key, kind="stable")
    groups = np.split(order, np.flatnonzero(np.diff(key[order])) + 1)
    ends = [(int(ps[g[0]]), int(pe[g[0]])) for g in groups]
    pairs = [(g, h) for g in range(len(groups)) for h in range(len(groups))
             if g != h and ends[g][1] == ends[h][0] and len(groups[g]) + len(groups[h]) <= 4900]
    sizes = [len(groups[g]) + len(groups[h]) for g, h in pairs]
    members = np.concatenate([groups[x] for pair in pairs for x in pair])
    begin = np.concatenate([[0], np.cumsum(sizes)])
    return members.astype(np.int32), begin.astype(np.int32), np.asarray([len(groups[g]) for g, _ in pairs], np.int32), max(sizes)


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def prepare(case, seed):
    size, ta, tf, t_end, ps, pe = _trace(case, seed)
    s = {"case": case, "trace": (_gpu(size), _gpu(ta), _gpu(tf), t_end), "cache": {}, "seed": 1000 + seed}
    op = case["op"]
    if op == "plan":
        s["orders"] = S.stalloc_make_orders(*s["trace"], case["plans"], seed=s["seed"])["orders"]
    elif op == "validate":
        s["plans"] = _gpu(_plans(case, seed, size, ta, tf))
    elif op == "bounds":
        s["extents"] = _gpu(_extents(case, seed, size))
    elif op == "reusable":
        s["plan"] = _gpu(_online_plan(size, ta, tf))
        s["windows"] = _gpu(_windows(case, seed, t_end))
        s["places"] = torch.arange(case["most"], dtype=torch.int32, device="cuda")
    elif op == "layers":
        s["places"] = torch.arange(len(size), dtype=torch.int32, device="cuda")
    elif op == "fuse":
        members, begin, first, largest = _pairs(ps, pe)
        s["pairs"] = (_gpu(members), _gpu(begin), _gpu(first), largest)
    return s


def _extents(c, seed, size):
    rng = np.random.default_rng([seed, 31])
    return rng.integers(int(size.max()), int(size.sum()) + 1, c["plans"]) // ROUND * ROUND


def run(s):
    op, trace, kept = s["case"]["op"], s["trace"], {"workspace_cache": s["cache"]}
    if op == "plan":
        r = S.stalloc_plan(*trace, s["orders"], want_offsets=s["case"]["offsets"], **kept)
        return {k: r[k] for k in ("offsets", "peaks", "best_offsets", "best_plan", "status")}
    if op == "validate":
        r = S.stalloc_validate(*trace, s["plans"], **kept)
        return {k: r[k] for k in ("conflicts", "first_pair", "status")}
    if op == "bounds":
        r = S.stalloc_lower_bound(*trace, **kept)
        t = S.stalloc_tmp(*trace, s["extents"], workspace_cache=s.setdefault("cache2", {}))
        return {"lower_bound": r["lower_bound"], "t_at_max": r["t_at_max"], "tmp": t["tmp"]}
    if op == "orders":
        r = S.stalloc_make_orders(*trace, s["case"]["plans"], seed=s["seed"], **kept)
        return {"orders": r["orders"], "status": r["status"]}
    if op == "layers":
        r = S.stalloc_memory_layers(*trace, **kept)
        spare = s["places"] >= r["n_layers"]                                 # places of the tables that hold no layer
        return {"layer_of": r["layer_of"], "n_layers": r["n_layers"], "layer_size": r["layer_size"].masked_fill_(spare, 0),
                "layer_t_alloc": r["layer_t_alloc"].masked_fill_(spare, 0), "layer_t_free": r["layer_t_free"].masked_fill_(spare, 0)}
    if op == "reusable":
        r = S.stalloc_reusable_space(*trace, s["plan"], s["windows"], s["case"]["most"], **kept)
        spare = s["places"] >= r["counts"][:, None]                          # places of a row that hold no interval
        return {"ranges": r["ranges"].masked_fill_(spare[:, :, None], 0), "counts": r["counts"], "idle_bytes": r["idle_bytes"]}
    r = S.stalloc_fuse_groups(*trace, *s["pairs"], **kept)
    return {k: r[k] for k in ("order", "addr", "extents", "accepted", "status")}


def work(case):
    """Bytes that must move; the arithmetic is on integers, so there are no floating-point operations to count."""
    n, op = _requests(case), case["op"]
    trace = 16 * n
    if op == "plan":
        return {"bytes": trace + (12 if case["offsets"] else 4) * n * case["plans"] + 8 * case["plans"] + 8 * n, "flops": 0}
    if op == "validate":
        return {"bytes": trace + 8 * n * case["plans"] + 16 * case["plans"], "flops": 0}
    if op == "bounds":
        return {"bytes": 2 * trace + 16 * case["plans"], "flops": 0}
    if op == "orders":
        return {"bytes": trace + 4 * n * case["plans"], "flops": 0}
    if op == "layers":
        return {"bytes": trace + 8 * n, "flops": 0}
    if op == "reusable":
        return {"bytes": trace + 8 * n + case["windows"] * (20 + 16 * case["most"]), "flops": 0}
    return {"bytes": trace + 16 * 3 * n, "flops": 0}


def tolerance(case):
    """Whole numbers everywhere but in the products of Eq. 2: exact sums, then at most eight roundings in double precision."""
    return {"rel": 1e-15, "max": 4e-15, "differ": 0.0} if case["op"] == "bounds" else "exact"


# ---------------------------------------------------------------------------------------------
# what run returns, from plain numpy

def _mix(x):
    with np.errstate(over="ignore"):
        z = x + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _orders(plans, seed, size, ta, tf):
    n = len(size)
    number = np.arange(n, dtype=np.uint64)
    rank = np.searchsorted(-np.unique(size)[::-1], -size).astype(np.uint64)
    rows = np.empty((plans, n), np.int32)
    for p in range(plans):
        if p == 0:
            row = np.lexsort((ta, -size))
        elif p == 1:
            row = np.lexsort((-size, -(tf.astype(np.int64) - ta)))
        elif p == 2:
            row = np.argsort(ta, kind="stable")
        else:
            with np.errstate(over="ignore"):
                key = _mix(number * np.uint64(0xD1342543DE82EF95) + _mix(np.asarray([seed + p], np.uint64))[0])
                if p % 2 == 0:
                    key = ((rank + np.uint64(1)) << np.uint64(32)) + (key >> np.uint64(31))
            row = np.argsort(key, kind="stable")
        rows[p] = row
    return rows


def _place(order, size, ta, tf):
    """Each request in turn at the lowest address at which it conflicts with no earlier one."""
    at, done = np.zeros(len(size), np.int64), np.zeros(len(size), bool)
    for i in order.tolist():
        k = np.flatnonzero(done & (ta < tf[i]) & (ta[i] < tf))
        k = k[np.argsort(at[k], kind="stable")]
        reach = np.maximum.accumulate(np.concatenate([[0], at[k] + size[k]]))
        fits = np.flatnonzero(at[k] - reach[:-1] >= size[i])
        at[i] = reach[fits[0]] if len(fits) else reach[-1]
        done[i] = True
    return at


def _layers(size, ta, tf):
    layer_of, tables, opened = np.empty(len(size), np.int32), [], 0
    for s in np.unique(size)[::-1]:
        group = np.flatnonzero(size == s)
        group = group[np.argsort(ta[group], kind="stable")]
        busy, idle, first, end = [], [], [], []                             # idle: released last on top
        for i in group.tolist():
            back = []
            while busy and busy[0][0] <= ta[i]:
                back.append(heapq.heappop(busy))
            for t, layer in sorted(back, key=lambda b: (b[0], -b[1])):
                idle.append(layer)
            if idle:
                layer = idle.pop()
            else:
                layer = len(first)
                first.append(int(ta[i]))
                end.append(0)
            end[layer] = int(tf[i])
            heapq.heappush(busy, (int(tf[i]), layer))
            layer_of[i] = opened + layer
        tables.append((np.full(len(first), s, np.int64), np.asarray(first, np.int32), np.asarray(end, np.int32)))
        opened += len(first)
    return layer_of, tuple(np.concatenate([t[k] for t in tables]) for k in range(3))


def exact(case, seed):
    op = case["op"]
    n = _requests(case)
    if op == "fuse" or (op == "plan" and n * n * case["plans"] > 2 * 10 ** 8) or (op == "orders" and n * case["plans"] > 6 * 10 ** 7) \
            or (op == "validate" and case["plans"] > 1 and n * n * case["plans"] > 2 * 10 ** 9):
        return None
    size, ta, tf, t_end, _, _ = _trace(case, seed)
    n = len(size)
    if op == "plan":
        orders = _orders(case["plans"], 1000 + seed, size, ta, tf)
        plans = np.stack([_place(o, size, ta, tf) for o in orders])
        peaks = (plans + size).max(axis=1)
        best = int(np.argmin(peaks))
        return {"offsets": plans if case["offsets"] else None, "peaks": peaks, "best_offsets": plans[best],
                "best_plan": np.asarray([best], np.int32), "status": np.zeros(1, np.int32)}
    if op == "validate":
        plans = _plans(case, seed, size, ta, tf)
        by = np.argsort(ta, kind="stable")
        a, f, z = ta[by], tf[by], size[by]
        stop = np.searchsorted(a, f, side="left")                           # starts before my release
        count, first = np.zeros(len(plans), np.int64), np.full((len(plans), 2), -1, np.int32)
        for p, plan in enumerate(plans):
            lo = plan[by]
            hi = lo + z
            best = None
            for k in range(len(by)):
                e = stop[k]
                hit = np.flatnonzero((lo[k + 1:e] < hi[k]) & (lo[k] < hi[k + 1:e])) if e > k + 1 else ()
                if len(hit):
                    count[p] += len(hit)
                    for j in by[k + 1 + hit].tolist():
                        pair = (min(int(by[k]), j), max(int(by[k]), j))
                        best = pair if best is None or pair < best else best
            if best is not None:
                first[p] = best
        return {"conflicts": count, "first_pair": first, "status": np.zeros(1, np.int32)}
    if op == "bounds":
        net = np.zeros(t_end + 1, np.int64)
        np.add.at(net, ta, size)
        np.add.at(net, tf, -size)
        live = np.cumsum(net)[:t_end]
        used = sum(s * t for s, t in zip(size.tolist(), (tf.astype(np.int64) - ta).tolist()))
        span = int(tf.max()) - int(ta.min())
        return {"lower_bound": live.max(keepdims=True), "t_at_max": np.asarray([np.argmax(live)], np.int32),
                "tmp": np.asarray([used / (e * span) for e in _extents(case, seed, size).tolist()])}
    if op == "orders":
        return {"orders": _orders(case["plans"], 1000 + seed, size, ta, tf), "status": np.zeros(1, np.int32)}
    if op == "layers":
        layer_of, tables = _layers(size, ta, tf)
        m = len(tables[0])
        s, a, f = (np.concatenate([t, np.zeros(n - m, t.dtype)]) for t in tables)
        return {"layer_of": layer_of, "n_layers": np.asarray([m], np.int32), "layer_size": s, "layer_t_alloc": a, "layer_t_free": f}
    plan = _online_plan(size, ta, tf)                                       # reusable
    by = np.argsort(plan, kind="stable")
    lo, a, f = plan[by], ta[by], tf[by]
    hi = lo + size[by]
    most, windows = case["most"], _windows(case, seed, t_end)
    ranges, counts = np.zeros((len(windows), most, 2), np.int64), np.zeros(len(windows), np.int32)
    idle = np.zeros(len(windows), np.int64)
    for w, (w_lo, w_hi) in enumerate(windows.tolist()):
        k = np.flatnonzero((a < w_hi) & (w_lo < f))
        reach = np.maximum.accumulate(np.concatenate([[lo[0]], hi[k]]))
        start = np.concatenate([lo[k], [hi.max()]])
        gap = np.flatnonzero(start > reach)
        counts[w], idle[w] = len(gap), int((start[gap] - reach[gap]).sum())
        gap = gap[:most]
        ranges[w, :len(gap), 0], ranges[w, :len(gap), 1] = reach[gap], start[gap]
    return {"ranges": ranges, "counts": counts, "idle_bytes": idle}
