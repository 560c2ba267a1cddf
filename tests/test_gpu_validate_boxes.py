"""The form of stalloc_validate that sorts short-lived requests by time and long-lived ones by address, where it can go wrong: requests
numbered by allocation time or not, lengths and shares of long-lived requests around whole tiles, plans that are gone through
in several groups; against the all-pairs form."""
import numpy as np
import pytest

from test_gpu_validate_near import _all_pairs

pytestmark = pytest.mark.gpu


def _trace(rng, n, longs):
    """`longs` of the requests live for a quarter of the trace, the others for up to a dozen allocations."""
    ts = np.sort(rng.permutation(4 * n)[:n])
    life = rng.integers(1, 40, n)
    life[rng.permutation(n)[:longs]] = rng.integers(n // 2, n, longs) if longs else 0
    size = np.where(life > 40, 4000, 1) * rng.integers(1, 50, n)
    return size.astype(np.uint64), ts.astype(np.uint32), (ts + life).astype(np.uint32), 5 * n


@pytest.mark.parametrize("numbered", ["by time", "at random"])
@pytest.mark.parametrize("n, longs, P", [(900, 64, 2100), (1024, 65, 1600), (1025, 0, 1500), (4096, 63, 100), (4097, 1280, 95), (4097, 4097, 95),
                                         (20011, 700, 6), (20011, 4161, 190), (70001, 300, 1), (150001, 40000, 1)])
def test_forms_agree(n, longs, P, numbered):
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng([n, longs])
    size, ts, te, t_end = _trace(rng, n, longs)
    if numbered == "at random":
        mixed = rng.permutation(n)
        size, ts, te = size[mixed], ts[mixed], te[mixed]
    # each plan puts the long-lived one after the other, the short-lived at low addresses: conflicts between neighbours in either
    many = min(P, 8)
    plans = np.empty((many, n), np.int64)
    for p in range(many):
        order = rng.permutation(n)
        at = np.cumsum(np.where(size[order] > 50, size[order], 0))
        plans[p, order] = np.where(size[order] > 50, at * 9 // 10, rng.integers(0, 4000, n))
    dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32))]
    given = torch.from_numpy(plans).cuda()[torch.arange(P, device="cuda") % many].contiguous()
    out = S.stalloc_validate(*dev, t_end, given)
    S.check_status(out)
    conflicts, first, status = _all_pairs(S, dev, t_end, given[:many].contiguous())
    assert int(status.item()) == 0 and (longs == 0 or int(conflicts.sum()) > 0)
    where = torch.arange(P, device="cuda") % many
    assert torch.equal(out["conflicts"], conflicts[where]) and torch.equal(out["first_pair"], first[where])


def test_one_wave_finds_more_pairs_than_32_bits_count():
    """7.5 million requests, all alive at once.  1216 of them cover all addresses from their start on, 64 that share a start in front
    of every 6143 * 64 others that keep clear of one another: in order of address every 6144th tile is one of theirs, and with a
    plan's tiles dealt out to 6144 waves in turn the same wave gets them all, 4.8e9 pairs."""
    import torch
    import paper_2507_16274_amd as S
    spans, each, segment = 19, 6143 * 64, 64 << 13          # (64 of 2^11 buckets of addresses a span)
    n, end = spans * (each + 64), (1 << 24) + 1
    start = torch.arange(spans, device="cuda")[:, None] * segment
    offsets = torch.cat([start.expand(spans, 64), start + 8192 + torch.arange(each, device="cuda")], dim=1)
    size = torch.cat([(end - start).expand(spans, 64), torch.ones((spans, each), dtype=torch.int64, device="cuda")], dim=1)
    assert int((offsets + size)[:, 64:].max()) <= spans * segment < end and int((offsets[:, -1] - start[:, 0]).max()) < segment
    once = torch.ones(n, dtype=torch.int32, device="cuda")
    out = S.stalloc_validate(size.reshape(n).contiguous(), once - 1, once, 1, offsets.reshape(1, n).contiguous())
    S.check_status(out)
    meet = sum(64 * ((spans - g) * (each + 64) - 64) + 64 * 63 // 2 for g in range(spans))          # with what begins at or behind their start
    assert meet > 1 << 32
    assert int(out["conflicts"].item()) == meet and out["first_pair"].tolist() == [[0, 1]]


@pytest.mark.parametrize("n, longs, P", [(4097, 1280, 95), (20011, 20011, 6), (70001, 40000, 1)])
def test_addresses_far_off(n, longs, P):
    """Damaged decisions near 2^62 or at 0, and starts far from 0 in all: the same conflicts, and about the same time -- the buckets that
    the long-lived requests are put into follow the addresses that most of them have."""
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng([n, longs, 7])
    size, ts, te, t_end = _trace(rng, n, longs)
    order = rng.permutation(n)
    plan = np.empty(n, np.int64)
    at = np.cumsum(np.where(size[order] > 50, size[order], 0)).astype(np.int64)
    plan[order] = np.where(size[order] > 50, at * 9 // 10, rng.integers(0, 4000, n))
    high = plan + (1 << 61)
    plans = {"as it is": plan, "all far from 0": high}
    for name, base, far in (("one far above", plan, [1 << 62]), ("three far above", plan, [1 << 62, 1 << 61, (1 << 63) - (1 << 20)]),
                            ("one far below", high, [0]), ("both", high, [0, (1 << 62) + (1 << 61)])):
        bent = base.copy()
        bent[np.flatnonzero(size > 50)[-len(far):] if longs else [0]] = far
        plans[name] = bent
    plans["none apart"] = np.full(n, 5, np.int64)
    dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32))]
    took = {}
    for name, one in plans.items():
        given = torch.from_numpy(one).cuda().expand(P, n).contiguous()
        kept = {}
        out = S.stalloc_validate(*dev, t_end, given, workspace_cache=kept)
        S.check_status(out)
        conflicts, first, status = _all_pairs(S, dev, t_end, given[:1].contiguous())
        assert int(status.item()) == 0, name
        assert (out["conflicts"] == conflicts).all() and (out["first_pair"] == first).all(), name
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for _ in range(10):
            begin.record()
            S.stalloc_validate(*dev, t_end, given, workspace_cache=kept)
            end.record()
            end.synchronize()
            took[name] = min(took.get(name, 1e9), begin.elapsed_time(end))
    del took["none apart"]                                            # (nearly all pairs that are alive together conflict)
    assert max(took.values()) < 1.7 * took["as it is"] + 0.03, took     # ms; 2.4 and 3.4 times in the larger two while they did not
