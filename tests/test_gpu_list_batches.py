"""Parity of the sorted-list kernel with the CPU oracle where its batches of 64 requests and its equally long chunks of the
list can go wrong: lengths around whole batches and chunks, orders whose batches are one chain of clashes, requests that
see many holes beside blocks that cover most of the list, more plans than workgroups, and both sides of the LDS limit."""

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


@pytest.mark.parametrize("kind", ["narrow", "wide"])
def test_more_plans_than_workgroups(S, oracle, kind):
    rng = np.random.default_rng(71)
    n, P = 200, 700
    tr = _trace(rng, n, kind)
    orders = np.stack([_orders(rng, tr, n)[k % 4] for k in range(P)])
    _compare_plans(S, oracle, tr, orders, method="allpairs")


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
