"""Parity of the sorted-list kernel (and, up to 512 requests in up to 4096 plans, of the kernel for short traces) with the CPU oracle where its batches of 64 requests and its equally long chunks of the
list can go wrong: lengths around whole batches and chunks, orders whose batches are one chain of clashes, requests that
see many holes beside blocks that cover most of the list, more plans than workgroups, plans handed on to 64-bit addresses, and both
sides of each layout's LDS limit."""

import numpy as np
import pytest

from helpers import random_trace
from test_gpu_parity import _T, _compare_plans, _gpu_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_16274_amd as S
    return S


def _trace(rng, n, kind):
    """Sizes of one to three, a few of forty, one in fifty as large as some thirty others: `compact` in a granule that they
    all share, `narrow` and `wide` odd numbers of bytes that take 32 and 64 bits."""
    size, ts, te, t_end = random_trace(rng, n, t_max=max(4, n // 3), sizes=[1, 2, 3, 3, 40])
    size[rng.random(n) < 0.02] = 100
    if kind == "compact":
        size = size * np.uint64(4096)
    else:
        size = size * np.uint64(2 ** 31 + 8 if kind == "wide" else 2 ** 10) + np.uint64(1)
    return _T(size, ts, te, t_end)


def _orders(rng, tr, n):
    by_time = np.argsort(tr.t_alloc, kind="stable")
    return np.stack([rng.permutation(n), by_time, by_time[::-1], np.argsort(-tr.size.astype(np.int64), kind="stable")]).astype(np.uint32)


BITS = {"compact": 16, "narrow": 32, "wide": 64}


@pytest.mark.parametrize("kind", ["compact", "narrow", "wide"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 256, 257, 321, 577, 2049])
def test_lengths_around_batches_and_chunks(S, oracle, kind, n):
    rng = np.random.default_rng([n, BITS[kind]])
    tr = _trace(rng, n, kind)
    got, _, _ = _compare_plans(S, oracle, tr, _orders(rng, tr, n), method="allpairs")
    if n >= 64:                                                   # (few requests may suit the bitmap kernel)
        assert got["info"]["kernel"] == "list_lds" and got["info"]["address_bits"] == BITS[kind]


MANY = 4097                                                       # plans; up to 4096 of up to 512 requests go to the kernel for short traces
NEXT_PLAN = {16: 14, 32: 14, 64: 15}                              # words of the workspace that plans are handed out by (kAccNextPlan, kAccNextWide)


def _compare_many(S, oracle, tr, orders, P=MANY, kernel=None):
    """`orders` over and over, P plans in all.  The sorted-list kernel hands out plans beyond one per workgroup, which no other does."""
    import torch
    rows = np.arange(P) % len(orders)
    dev = torch.from_numpy(np.ascontiguousarray(orders[rows]).view(np.int32)).cuda()
    plan = S.stalloc_plan(*S.trace_to_device(tr), tr.t_end, dev)
    S.check_status(plan)
    info = S.stalloc_plan_report(plan)
    a, ext = oracle.plan_many(tr.size, tr.t_alloc, tr.t_free, orders, method="allpairs")
    assert np.array_equal(plan["peaks"].cpu().numpy().view(np.uint64), ext[rows])
    offsets = torch.from_numpy(a.view(np.int64)).cuda()
    assert torch.equal(plan["offsets"], offsets[torch.from_numpy(rows).cuda()])
    assert int(plan["best_plan"].item()) == int(np.argmin(ext))
    if kernel:
        assert info["kernel"] == kernel
    if kernel == "list_lds":
        words = plan["workspace"][:16 * 8].view(torch.int64).cpu()
        assert int(words[NEXT_PLAN[info["address_bits"]]]) > 0, "plans were handed out"
    return info


@pytest.mark.parametrize("kind", ["compact", "narrow", "wide"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 256, 257, 321, 511, 512])
def test_short_lengths_in_many_plans(S, oracle, kind, n):
    """The lengths around batches and chunks that only a call of more than 4096 plans takes to this kernel."""
    rng = np.random.default_rng([n, BITS[kind]])
    tr = _trace(rng, n, kind)
    info = _compare_many(S, oracle, tr, _orders(rng, tr, n), kernel="list_lds" if n >= 64 else None)
    assert n < 64 or info["address_bits"] == BITS[kind]


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 300, 512])
def test_short_lengths_in_many_plans_of_the_bitmap_kernel(S, oracle, n):
    rng = np.random.default_rng([n, 4])
    size, ts, te, t_end = random_trace(rng, n, t_max=max(4, n // 3), sizes=[1, 2, 3, 8])
    tr = _T(size * np.uint64(4096), ts, te, t_end)
    _compare_many(S, oracle, tr, _orders(rng, tr, n), kernel="bitmap")


@pytest.mark.parametrize("kind", ["narrow", "wide"])
def test_more_plans_than_workgroups(S, oracle, kind):
    rng = np.random.default_rng(71)
    n = 577
    tr = _trace(rng, n, kind)
    info = _compare_many(S, oracle, tr, _orders(rng, tr, n), P=2500, kernel="list_lds")
    assert info["address_bits"] == BITS[kind]


@pytest.mark.parametrize("n", [3000, 8900])
def test_blocks_that_concern_no_request_of_a_batch(S, oracle, n):
    """Requests that live for a dozen allocations, one in a hundred for long: in an order by size whole groups of blocks lie at other times than
    the batch, in orders by time and at random few do; lists in LDS and in the workspace."""
    rng = np.random.default_rng([77, n])
    ts = np.arange(n) * 2
    te = ts + 2 * rng.integers(1, 12, n) + np.where(rng.random(n) < 0.01, n // 4, 0)
    size = (rng.choice([1, 2, 5, 1000, 70000], n) * 512 + 1).astype(np.uint64)
    tr = _T(size, ts.astype(np.uint32), te.astype(np.uint32), int(te.max()))
    orders = np.concatenate([_orders(rng, tr, n), np.lexsort((ts, -size.astype(np.int64)))[None].astype(np.uint32)])
    got, _, _ = _compare_plans(S, oracle, tr, orders, method="lists")
    assert got["info"]["kernel"] == ("list_lds" if n == 3000 else "list_memory") and got["info"]["address_bits"] == 32


@pytest.mark.parametrize("beyond", [0, 1])
def test_both_sides_of_the_lds_limit(S, oracle, beyond):
    n = S.lib.stalloc_plan_lds_capacity() + beyond
    rng = np.random.default_rng(72)
    tr = _trace(rng, n, "narrow")
    got, _, _ = _compare_plans(S, oracle, tr, _orders(rng, tr, n)[:2], method="lists")
    assert got["info"]["kernel"] == ("list_memory" if beyond else "list_lds")


def _longest_with(S, rng, kind, lo, hi, **want):
    """Length of the longest trace that is placed with the given figures in its report (those of `lo` are, those of `hi` not)."""
    def holds(n):
        tr = _trace(rng, n, kind)
        info = _gpu_plan(S, tr, np.arange(n, dtype=np.uint32)[None])["info"]
        return all(info[k] == v for k, v in want.items())
    assert holds(lo) and not holds(hi)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if holds(mid) else (lo, mid)
    return lo


def test_both_sides_of_the_packed_list_s_limit(S, oracle):
    rng = np.random.default_rng(73)
    last = _longest_with(S, rng, "compact", 3000, 4200, kernel="list_lds", address_bits=16)
    for n, bits in ((last, 16), (last + 1, 32)):
        tr = _trace(rng, n, "compact")
        got, _, _ = _compare_plans(S, oracle, tr, _orders(rng, tr, n), method="lists")
        assert got["info"]["kernel"] == "list_lds" and got["info"]["address_bits"] == bits


def test_both_sides_of_the_limit_of_lists_with_64_bit_addresses(S, oracle):
    rng = np.random.default_rng(74)
    last = _longest_with(S, rng, "wide", 3000, 6000, kernel="list_lds")
    for n, kernel in ((last, "list_lds"), (last + 1, "list_memory")):
        tr = _trace(rng, n, "wide")
        got, _, _ = _compare_plans(S, oracle, tr, _orders(rng, tr, n), method="lists")
        assert got["info"]["kernel"] == kernel and got["info"]["address_bits"] == 64


def _outgrows(size, order, at):
    """The sizes of a batch of 64 on top of all before it need not fit 32 bits."""
    end = np.maximum.accumulate((at + size)[order])
    return any(int(end[b - 1] if b else 0) + int(size[order[b:b + 64]].sum()) >= 2 ** 32 for b in range(0, len(size), 64))


@pytest.mark.parametrize("n_clique, n_extra, kernel", [(1000, 2000, "list_lds"), (2000, 5500, "list_memory")])
def test_some_of_more_plans_than_workgroups_outgrow_32_bit_counts(S, oracle, n_clique, n_extra, kernel):
    """Odd byte sizes that stack up to nearly 2^32: a workgroup that gives up a plan tried with 32-bit counts takes the next one
    that is handed out, and those given up, some of each workgroup's, are placed again with 64-bit addresses."""
    rng = np.random.default_rng(75)
    unit = 2 ** 21
    size = np.concatenate([rng.integers(unit // 2, unit * 3 // 2, n_clique), rng.integers(unit // 4, unit * 2, n_extra)]).astype(np.uint64)
    size[:n_clique] = size[:n_clique].astype(np.float64) * (0.97 * 2 ** 32 / float(size[:n_clique].sum()))
    size |= np.uint64(1)
    ts = np.concatenate([np.zeros(n_clique, np.int64), rng.integers(0, 20 * n_extra, n_extra)])
    te = np.concatenate([np.full(n_clique, 21 * n_extra, np.int64), ts[n_clique:] + rng.integers(1, 60, n_extra)])
    n, P = n_clique + n_extra, 600
    tr = _T(size, ts.astype(np.uint32), te.astype(np.uint32), int(te.max()))
    some = [rng.permutation(n) for _ in range(3)]
    some += [np.argsort(ts, kind="stable"), np.argsort(-size.astype(np.int64), kind="stable"), np.arange(n)[::-1]]
    some = np.stack(some).astype(np.uint32)
    rows = np.arange(P) % len(some)
    a, ext = oracle.plan_many(tr.size, tr.t_alloc, tr.t_free, some, method="lists")
    wide = np.asarray([_outgrows(size, o, x) for o, x in zip(some, a)])
    assert 0 < wide.sum() < len(some)
    got = _gpu_plan(S, tr, some[rows])
    info = got["info"]
    assert got["status"] == 0 and info["kernel"] == kernel and info["address_bits"] == 32
    assert info["plans_64bit"] == int(wide[rows].sum())
    assert np.array_equal(got["peaks"], ext[rows]) and np.array_equal(got["offsets"], a[rows])


@pytest.mark.parametrize("fill", [0.80, 0.95])
def test_short_plans_that_outgrow_32_bit_counts_among_many(S, oracle, fill):
    """A clique of odd sizes with a sum of `fill` x 2^32 bytes and half as many requests in between, tried with 32-bit counts by the sorted-list
    kernel: plans go on to 64-bit addresses where the sizes of a batch on top of all before it need not fit."""
    rng = np.random.default_rng(78)
    n = 300
    size = rng.integers(1, 1 << 20, n).astype(np.float64)
    size = (size * (fill * 2 ** 32 / size[:200].sum())).astype(np.uint64) | np.uint64(1)
    ts = np.r_[np.zeros(200, np.int64), rng.integers(0, 90, 100)]
    te = np.r_[np.full(200, 100), ts[200:] + rng.integers(1, 9, 100)]
    tr = _T(size, ts.astype(np.uint32), te.astype(np.uint32), 100)
    orders = np.stack([rng.permutation(n) for _ in range(20)]).astype(np.uint32)
    info = _compare_many(S, oracle, tr, orders, kernel="list_lds")
    a, _ = oracle.plan_many(tr.size, tr.t_alloc, tr.t_free, orders, method="allpairs")
    wide = np.asarray([_outgrows(tr.size, o, x) for o, x in zip(orders, a)])
    assert info["address_bits"] == 32 and info["plans_64bit"] == int(wide[np.arange(MANY) % 20].sum()) and wide.any() == (fill > 0.9)


@pytest.mark.parametrize("narrow", [8, 40, 400])
def test_whole_batches_go_through_one_crowded_chunk_of_a_list_in_the_workspace(S, oracle, narrow):
    """Blocks that stay alternate with blocks that go, one hole each; what comes later wants those holes, all of a batch the same one
    first.  `narrow` holes in a row suit the few small requests only: with fewer than a request's noted holes the search ends among
    them or goes on in the next chunk, with more it falls back on the list.  Wholly free holes and half-filled ones are both met."""
    rng = np.random.default_rng([76, narrow])
    n_base, n = 4800, S.lib.stalloc_plan_lds_capacity() + 321
    n_late = n - n_base
    unit = 2 ** 12
    size = rng.integers(2, 6, n).astype(np.uint64)
    size[1:n_base:2] = np.where(np.arange(n_base // 2) // narrow % 2 == 0, 1, size[1:n_base:2])
    size[n_base:] = np.where(rng.random(n_late) < 0.3, 1, size[n_base:])
    size = size * np.uint64(unit) + np.uint64(1)
    ts = np.concatenate([np.zeros(n_base, np.int64), 10 + np.arange(n_late)])
    te = np.concatenate([np.where(np.arange(n_base) % 2 == 0, 2 * n, 5), ts[n_base:] + rng.integers(500, 1500, n_late)])
    tr = _T(size, ts.astype(np.uint32), te.astype(np.uint32), int(te.max()))
    late = n_base + rng.permutation(n_late)
    orders = np.stack([np.arange(n), np.concatenate([np.arange(n_base), late])]).astype(np.uint32)
    got, _, _ = _compare_plans(S, oracle, tr, orders, method="lists")
    assert got["info"]["kernel"] == "list_memory" and got["info"]["address_bits"] == 32
