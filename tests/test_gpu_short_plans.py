"""Short traces, which a wave places with the list of blocks in its registers: lengths around the register sets of 64 blocks,
every width of address, orders whose requests are one chain, errors, and both sides of what the kernel takes."""
import numpy as np
import pytest

from helpers import random_trace
from test_gpu_list_batches import BITS, _orders, _trace
from test_gpu_parity import _T, _compare_plans, _gpu_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_16274_amd as S
    return S


@pytest.mark.parametrize("kind", ["compact", "narrow", "wide"])
@pytest.mark.parametrize("n", [2, 62, 66, 127, 130, 191, 192, 193, 255, 320, 385, 449, 511, 512, 513])
def test_lengths_around_register_sets(S, oracle, n, kind):
    rng = np.random.default_rng([n, BITS[kind], 3])
    tr = _trace(rng, n, kind)
    got, _, _ = _compare_plans(S, oracle, tr, _orders(rng, tr, n), method="allpairs")
    assert n < 62 or got["info"]["address_bits"] == BITS[kind]


@pytest.mark.parametrize("n", [64, 200, 512])
@pytest.mark.parametrize("t_end", [65535, 65536, 2 ** 31 - 1])
def test_times_up_to_the_end_and_blocks_up_to_the_largest_address(S, oracle, n, t_end):
    """Lifetimes that end with the last timestamp that 16 bits hold and beyond; a sum of 65 535 granules, one short of what
    16-bit counts cannot hold, stacked to the top by requests that all live together at first."""
    rng = np.random.default_rng([n, t_end % 1000])
    size = rng.integers(1, 65535 // n, n)
    size[0] += 65535 - size.sum()
    ts = np.where(rng.random(n) < 0.7, 0, rng.integers(0, t_end, n))
    te = np.where(rng.random(n) < 0.7, t_end, np.minimum(ts + rng.integers(1, 1000, n), t_end))
    tr = _T((size * 512).astype(np.uint64), ts.astype(np.uint32), te.astype(np.uint32), t_end)
    got, _, _ = _compare_plans(S, oracle, tr, _orders(rng, tr, n), method="allpairs")
    assert got["info"]["address_bits"] == (16 if t_end < 65536 else 32)


@pytest.mark.parametrize("P", [1, 1023, 4096, 4097])
def test_numbers_of_plans(S, oracle, P):
    rng = np.random.default_rng(P)
    n = 70
    tr = _trace(rng, n, "narrow")
    some = np.stack([rng.permutation(n) for _ in range(50)]).astype(np.uint32)
    _compare_plans(S, oracle, tr, some[np.arange(P) % 50], method="allpairs")


@pytest.mark.parametrize("fill", [0.5, 0.93, 1.2])
def test_plans_that_outgrow_32_bit_counts(S, oracle, fill):
    """A clique of odd sizes with a sum of `fill` x 2^32 bytes, and half as many requests in between."""
    rng = np.random.default_rng(7)
    n = 150
    size = rng.integers(1, 1 << 20, n).astype(np.float64)
    size = (size * (fill * 2 ** 32 / size[:100].sum())).astype(np.uint64) | np.uint64(1)
    ts = np.r_[np.zeros(100, np.int64), rng.integers(0, 90, 50)]
    te = np.r_[np.full(100, 100), ts[100:] + rng.integers(1, 9, 50)]
    tr = _T(size, ts.astype(np.uint32), te.astype(np.uint32), 100)
    orders = np.stack([rng.permutation(n) for _ in range(20)]).astype(np.uint32)
    got, _, ext = _compare_plans(S, oracle, tr, orders, method="allpairs")
    assert got["info"]["address_bits"] == 32
    above = int((ext > np.uint64(2 ** 32 - 1)).sum())
    assert got["info"]["plans_64bit"] == above and (above > 0 or fill < 1) and (above == 0 or fill > 0.5)


@pytest.mark.parametrize("n", [5, 64, 300])
def test_errors(S, n):
    """A malformed trace or order is reported as by the other kernels, whichever plan it is in."""
    rng = np.random.default_rng(n)
    size, ts, te, t_end = random_trace(rng, n)
    order = np.stack([rng.permutation(n) for _ in range(6)]).astype(np.uint32)

    def status(size=size, ts=ts, te=te, t_end=t_end, order=order):
        return _gpu_plan(S, _T(size, ts, te, t_end), order)["status"]

    worse = order.copy()
    worse[4, n - 1] = n
    none, dead, much = size.copy(), te.copy(), size.copy()
    none[n // 2], dead[n - 1], much[0] = 0, ts[n - 1], 1 << 63
    assert status() == 0
    assert status(order=worse) == 6
    assert status(size=none) == 2 and status(te=dead) == 2 and status(t_end=int(te.max()) - 1) == 2
    assert status(size=much) == 3 and status(size=much, order=worse) == 3
