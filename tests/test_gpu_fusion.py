"""Parity of stalloc_fuse_groups (fusion of two HomoPhase groups, Sec. 5.1) with the CPU oracle, through
the C ABI: order, every address, the three extents and the accept flag of every candidate pair, bit by bit."""
import numpy as np
import pytest

from workloads import Trace, make_trace
from workloads.groups import candidate_pairs, flatten_pairs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_16274_amd as S
    return S


def _fuse(S, tr, members, begin, count1, largest):
    import torch
    size, ta, tf = S.trace_to_device(tr)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).cuda()
    out = S.stalloc_fuse_groups(size, ta, tf, tr.t_end, dev(members), dev(begin), dev(count1), largest)
    torch.cuda.synchronize()
    return {"status": int(out["status"].item()), "order": out["order"].cpu().numpy().view(np.uint32),
            "addr": out["addr"].cpu().numpy().view(np.uint64), "extents": out["extents"].cpu().numpy().view(np.uint64),
            "accepted": out["accepted"].cpu().numpy()}


def _compare(S, oracle, tr, groups, pairs):
    members, begin, count1, largest = flatten_pairs(groups, pairs)
    got = _fuse(S, tr, members, begin, count1, largest)
    assert got["status"] == 0
    n_acc = 0
    for k, (g, h) in enumerate(pairs):
        want = oracle.fuse_groups(tr.size, tr.t_alloc, tr.t_free, groups[g], groups[h])
        lo, hi = int(begin[k]), int(begin[k + 1])
        assert np.array_equal(got["order"][lo:hi], want["order"]), (k, g, h)
        assert np.array_equal(got["addr"][lo:hi], want["a"]), (k, g, h)
        assert np.array_equal(got["extents"][k], want["extent"]), (k, g, h)
        assert bool(got["accepted"][k]) == want["accepted"], (k, g, h)
        n_acc += int(want["accepted"])
    return n_acc


@pytest.mark.parametrize("cfg", [1, 2, 3, 5])
def test_every_candidate_pair_of_a_training_trace(S, oracle, cfg):
    tr = make_trace(cfg)
    groups, pairs = candidate_pairs(tr.p_alloc, tr.p_free)
    assert len(pairs) >= 5
    n_acc = _compare(S, oracle, tr, groups, pairs)
    if cfg in (2, 5):
        assert 0 < n_acc < len(pairs)          # both outcomes of the accept test occur


def _random_trace(rng, n, t_end, sizes):
    ts = rng.integers(0, t_end - 1, n)
    te = np.minimum(ts + rng.integers(1, max(2, t_end // 3), n), t_end)
    return Trace(name="random", size=rng.choice(np.asarray(sizes, dtype=np.uint64), n), t_alloc=ts.astype(np.uint32),
                 t_free=te.astype(np.uint32), t_end=t_end)


@pytest.mark.parametrize("seed", range(6))
def test_random_groups_with_arbitrary_lifetimes(S, oracle, seed):
    """Groups that are no HomoPhase groups at all (lifetimes overlap freely, equal keys abound): the
    kernel's sorts, its pointer walk and the leftovers on top against the oracle's."""
    rng = np.random.default_rng(4200 + seed)
    n = 3000
    tr = _random_trace(rng, n, t_end=int(rng.choice([6, 40, 900])), sizes=[512, 1024, 1536, 4096, 1 << 20, 3 << 30])
    groups, pairs = [], []
    for k in range(40):
        n1, n2 = int(rng.integers(1, 300)), int(rng.integers(1, 300))
        ids = rng.choice(n, n1 + n2, replace=False).astype(np.uint32)
        groups += [ids[:n1], ids[n1:]]
        pairs.append((2 * k, 2 * k + 1))
    _compare(S, oracle, tr, groups, pairs)


def test_single_requests_equal_extents_and_sizes_near_2_to_the_62(S, oracle):
    size = np.asarray([1 << 61, 1 << 61, 512, 512, (1 << 61) - 512, 1024], dtype=np.uint64)
    ts = np.asarray([0, 2, 0, 1, 1, 0], dtype=np.uint32)
    te = np.asarray([2, 4, 1, 3, 4, 4], dtype=np.uint32)
    tr = Trace(name="edge", size=size, t_alloc=ts, t_free=te, t_end=4)
    groups = [np.asarray(g, dtype=np.uint32) for g in ([0], [1], [2], [3], [0, 2], [4, 3], [5], [1, 4])]
    pairs = [(0, 1), (1, 0), (2, 3), (3, 2), (4, 5), (5, 4), (6, 7), (7, 6), (0, 6), (2, 0)]
    _compare(S, oracle, tr, groups, pairs)


def test_a_large_pair_at_the_lds_limit_and_errors(S, oracle):
    import torch
    rng = np.random.default_rng(77)
    n = 6000
    tr = _random_trace(rng, n, t_end=64, sizes=[512, 2048, 65536])
    ids = rng.permutation(n).astype(np.uint32)
    groups = [ids[:2500], ids[2500:4900]]
    _compare(S, oracle, tr, groups, [(0, 1), (1, 0)])
    # beyond the LDS limit: refused on the host
    members, begin, count1, largest = flatten_pairs([ids[:3000], ids[3000:]], [(0, 1)])
    with pytest.raises(S.StallocError) as err:
        _fuse(S, tr, members, begin, count1, largest)
    assert err.value.code == 9
    # a pair larger than announced, an empty group, a request number >= n: reported by the device
    members, begin, count1, largest = flatten_pairs(groups, [(0, 1)])
    assert _fuse(S, tr, members, begin, count1, 100)["status"] == 9
    assert _fuse(S, tr, members, begin, np.asarray([0], dtype=np.uint32), largest)["status"] == 1
    bad = members.copy(); bad[17] = n
    assert _fuse(S, tr, bad, begin, count1, largest)["status"] == 6
    # pairs that reach beyond the member list, or backwards: reported, nothing read or written out there
    assert _fuse(S, tr, members, np.asarray([0, len(members) + 1], dtype=np.uint32), count1, largest)["status"] == 1
    assert _fuse(S, tr, members, np.asarray([4000, 100], dtype=np.uint32), count1, largest)["status"] == 1


@pytest.mark.parametrize("kind", ["before", "after", "stack", "free"])
@pytest.mark.parametrize("n1,n2", [(64, 65), (700, 63), (130, 1500), (1, 129), (900, 900), (127, 129), (128, 129)])
def test_groups_before_after_and_inside_each_other(S, oracle, n1, n2, kind):
    """The smaller group entirely earlier or later than the larger one (lifetimes meet in one phase only), with
    lifetimes nested like a stack's, and free: requests that fit for good, that sleep and that need a
    look, around the 64 requests a wave takes at a time."""
    rng = np.random.default_rng(n1 * 7 + n2)
    n = n1 + n2
    if kind == "free":
        ts = rng.integers(0, 900, n)
        te = ts + rng.integers(1, 300, n)
    else:
        meet = rng.permutation(2 * n)[:n] + 2 * n                 # the phase in which both are alive
        first, second = (slice(0, n1), slice(n1, n)) if kind != "before" else (slice(n1, n), slice(0, n1))
        ts, te = meet.copy(), meet.copy()
        k1, k2 = first.stop - first.start, second.stop - second.start
        ts[first] = np.sort(rng.integers(0, 2 * n, k1))
        te[second] = np.sort(rng.integers(4 * n, 6 * n, k2))
        if kind == "stack":
            te[first] = np.sort(te[first])[::-1]
            te[second] = te[second][::-1]
            ts[second] = np.sort(ts[second])
    size = rng.choice([512, 1024, 4096, 1 << 20], n).astype(np.uint64)
    tr = Trace(name="phases", size=size, t_alloc=ts.astype(np.uint32), t_free=te.astype(np.uint32), t_end=int(te.max()))
    ids = np.arange(n, dtype=np.uint32)
    _compare(S, oracle, tr, [ids[:n1], ids[n1:]], [(0, 1), (1, 0)])


def test_sizes_that_would_wrap_end_with_a_status(S):
    """Requests near 2^61 bytes listed several times, and beside entries that name no request: starts that would not
    ascend.  Reported, and the call returns; without the repetition the same requests are placed."""
    n = 68
    size = np.full(n, 512, dtype=np.uint64)
    size[:2] = 1 << 61
    ts, te = np.zeros(n, np.uint32), np.full(n, 200, np.uint32)
    te[0], te[1], te[66], te[67], ts[67] = 100, 300, 10, 400, 20
    tr = Trace(name="wrap", size=size, t_alloc=ts, t_free=te, t_end=400)
    small = np.asarray([67], dtype=np.uint32)
    larger = np.concatenate([[1], np.arange(2, 66), [66]]).astype(np.uint32)
    for extra, status in (([0], 0), ([0] * 7, 3), ([0] + [n] * 6, 6), ([0] + [0xffffffff] * 6, 6), ([0] * 7 + [n], 6)):
        both = np.concatenate([larger, np.asarray(extra, dtype=np.uint32)])
        for pair in ((both, small), (small, both)):
            members, begin, count1, largest = flatten_pairs(list(pair), [(0, 1)])
            got = _fuse(S, tr, members, begin, count1, largest)
            assert got["status"] == status
            if status == 0:
                assert got["extents"][0, 2] == (1 << 62) + 65 * 512
