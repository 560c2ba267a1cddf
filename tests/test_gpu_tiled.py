"""The bitmap kernel with tables per tile of time (from 1024 requests on, sizes of at most 31 granules) against the
oracle: trace lengths around the limits of its two shapes, distinct and tied times, requests that live for one
tile, for part of one and for all of them, plans that outgrow its tables and are placed by the other bitmap
kernel, malformed orders."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _path(plan):
    """(shape or None when the tiled variant declined the trace, tiles, plans it handed on): words 11 and 12 of the
    accumulators at the start of the workspace (kAccTiles, kAccTilesMissed; the report does not tell the two bitmap
    kernels apart)."""
    import torch
    word, missed = (int(x) for x in plan["workspace"][:16 * 8].view(torch.int64)[11:13].cpu())
    return (word >> 1 & 0x7f, word >> 8 & 0xff, missed) if word & 1 else (None, 0, missed)


def _trace(rng, n, kind):
    """kind: how long requests live and how their times fall."""
    if kind == "tied":
        ts = rng.integers(0, n // 6, n)
        te = ts + rng.integers(1, 30, n)
    elif kind == "persistent":                                    # some alive throughout, from the first to the last tile
        ts = rng.integers(0, 2 * n - 8, n)
        te = ts + rng.integers(1, 7, n)
        ts[: n // 40], te[: n // 40] = 0, 2 * n
    elif kind == "stack":                                         # scoped: released in reverse order, transients in between
        ts, te = np.arange(n), np.arange(n) + rng.integers(1, 6, n)
        k = np.flatnonzero(rng.random(n) < 0.3)
        te[k] = 2 * n - np.arange(len(k))
    else:                                                         # all lengths
        ts = rng.integers(0, 2 * n - 2, n)
        te = np.minimum(ts + np.exp(rng.uniform(0, np.log(2 * n), n)).astype(np.int64) + 1, 2 * n)
    return ts.astype(np.uint32), te.astype(np.uint32)


@pytest.mark.parametrize("kind", ["tied", "persistent", "stack", "mixed"])
@pytest.mark.parametrize("n,most", [(1024, 31), (2049, 8), (4097, 3), (6144, 8), (9001, 8), (17000, 2), (3071, 8), (3072, 31), (3073, 31), (4096, 8), (16383, 2),
                                     (16384, 2)])
def test_plans_match_the_oracle(oracle, n, most, kind):
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(n + len(kind))
    ts, te = _trace(rng, n, kind)
    # few large requests and many small ones; 4096-byte granules (the odd sizes keep them)
    size = (rng.choice([1, 2, most], n, p=[0.6, 0.3, 0.1]) * 4096).astype(np.uint64)
    if n > 9000:                                                  # (the sum of sizes has to suit the bitmap kernels at all)
        te = np.minimum(te, ts + 3000).astype(np.uint32)
    t_end = int(te.max())
    orders = np.stack([rng.permutation(n) for _ in range(4)] + [np.lexsort((ts, -size.astype(np.int64))), np.argsort(size, kind="stable"),
                                                                  np.argsort(ts, kind="stable")]).astype(np.uint32)
    dev = lambda x, t: torch.from_numpy(np.ascontiguousarray(x).view(t)).cuda()
    plan = S.stalloc_plan(dev(size, np.int64), dev(ts, np.int32), dev(te, np.int32), t_end, dev(orders, np.int32))
    S.check_status(plan)
    assert S.stalloc_plan_report(plan)["kernel"] == "bitmap"
    shape, tiles, missed = _path(plan)
    large = (n, kind) in {(3072, "stack"), (16383, "stack"), (16384, "stack"), (17000, "stack"), (17000, "mixed")}
    assert shape == (1 if large else 0) and tiles >= (8 if large else 12) and missed == 0
    a, ext = oracle.plan_many(size, ts, te, orders, threads=7, method="lists")
    assert np.array_equal(plan["peaks"].cpu().numpy().view(np.uint64), ext)
    assert np.array_equal(plan["offsets"].cpu().numpy().view(np.uint64), a)
    assert int(plan["best_plan"].item()) == int(np.argmin(ext))


def test_a_trace_without_enough_tiles_is_declined(oracle):
    """A few timestamps: no eight tiles of time."""
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(5)
    n = 3300
    ts = rng.integers(0, 5, n)
    te, size = (ts + rng.integers(1, 3, n)).astype(np.uint32), rng.integers(1, 4, n).astype(np.uint64)
    orders = np.stack([rng.permutation(n) for _ in range(3)]).astype(np.uint32)
    dev = lambda x, t: torch.from_numpy(np.ascontiguousarray(x).view(t)).cuda()
    plan = S.stalloc_plan(dev(size, np.int64), dev(ts.astype(np.uint32), np.int32), dev(te, np.int32), int(te.max()), dev(orders, np.int32))
    S.check_status(plan)
    assert S.stalloc_plan_report(plan)["kernel"] == "bitmap" and _path(plan)[0] is None
    a, ext = oracle.plan_many(size, ts.astype(np.uint32), te, orders, threads=7, method="lists")
    assert np.array_equal(plan["offsets"].cpu().numpy().view(np.uint64), a)


def test_orders_that_all_leave_holes_are_left_to_the_other_kernel(oracle):
    """Every plan outgrows the tables: beyond the first plans, which run side by side, none is tried; the addresses
    are those of plans that were never tried."""
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(12)
    k = 1300
    n = 2 * k + k // 2
    ts, te, size = np.zeros(n, np.int64), np.zeros(n, np.int64), np.full(n, 512, np.uint64)
    early, kept, late = np.arange(0, 2 * k, 2), np.arange(1, 2 * k, 2), np.arange(2 * k, n)
    ts[:2 * k] = rng.integers(0, 1000, 2 * k)
    te[early], te[kept] = 2000, rng.integers(4000, 4200, k)
    ts[late], te[late], size[late] = 2000 + rng.integers(0, 50, k // 2), 4000, 1024
    ts, te = ts.astype(np.uint32), te.astype(np.uint32)
    tall = np.arange(n)
    orders = np.stack([np.concatenate([np.roll(tall[:2 * k], 2 * int(rng.integers(0, k))), rng.permutation(late)])
                       for _ in range(2500)]).astype(np.uint32)
    dev = lambda x, t: torch.from_numpy(np.ascontiguousarray(x).view(t)).cuda()
    args = (dev(size, np.int64), dev(ts, np.int32), dev(te, np.int32), int(te.max()))
    plan = S.stalloc_plan(*args, dev(orders, np.int32))
    S.check_status(plan)
    shape, _, missed = _path(plan)
    side_by_side = 3 * torch.cuda.get_device_properties(0).multi_processor_count
    assert shape == 0 and 16 < missed < 2500 and missed <= 2 * side_by_side
    rows = [0, 1, side_by_side + 5, 2499]
    a, ext = oracle.plan_many(size, ts, te, orders[rows], threads=7, method="lists")
    assert np.array_equal(plan["peaks"].cpu().numpy().view(np.uint64)[rows], ext)
    assert np.array_equal(plan["offsets"].cpu().numpy().view(np.uint64)[rows], a)
    assert not S.stalloc_validate(*args, plan["offsets"])["conflicts"].any()


def test_plans_that_outgrow_the_tables_are_placed_all_the_same(oracle):
    """Unit blocks of two kinds placed in turn, one kind released early, then blocks of two units that do not fit
    the holes in between: an extent of one and a half times the largest number of live granules, beside
    orders that stay close to it."""
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(11)
    k = 1300
    early, kept, late = np.arange(0, 2 * k, 2), np.arange(1, 2 * k, 2), np.arange(2 * k, 2 * k + k // 2)
    n = 2 * k + k // 2
    ts, te, size = np.zeros(n, np.int64), np.zeros(n, np.int64), np.full(n, 512, np.uint64)
    ts[:2 * k] = rng.integers(0, 1000, 2 * k)
    te[early], te[kept] = 2000, rng.integers(4000, 4200, k)
    ts[late], te[late], size[late] = 2000 + rng.integers(0, 50, k // 2), 4000, 1024
    ts, te = ts.astype(np.uint32), te.astype(np.uint32)
    tall = np.concatenate([np.arange(2 * k), late])
    orders = np.stack([tall, np.lexsort((ts, -size.astype(np.int64))), np.concatenate([tall[4:2 * k], late, tall[:4]])] +
                      [rng.permutation(n) for _ in range(300)] + [tall]).astype(np.uint32)
    dev = lambda x, t: torch.from_numpy(np.ascontiguousarray(x).view(t)).cuda()
    args = (dev(size, np.int64), dev(ts, np.int32), dev(te, np.int32), int(te.max()))
    plan = S.stalloc_plan(*args, dev(orders, np.int32))
    S.check_status(plan)
    shape, _, missed = _path(plan)
    assert shape == 0 and missed == 3
    rows = list(range(8)) + [302, 303]
    a, ext = oracle.plan_many(size, ts, te, orders[rows], threads=7, method="lists")
    lb, _ = oracle.lower_bound(size, ts, te, int(te.max()))
    assert (ext * 8 > lb * 9 + 8 * 32 * 5 * 512).sum() == 3, "which plans outgrow the tables"
    assert np.array_equal(plan["peaks"].cpu().numpy().view(np.uint64)[rows], ext)
    assert np.array_equal(plan["offsets"].cpu().numpy().view(np.uint64)[rows], a)
    conflicts = S.stalloc_validate(*args, plan["offsets"])["conflicts"]
    assert not conflicts.any()
    bad = orders[:3].copy()                                       # repeated entries: unspecified, but nothing else may break
    bad[1] = bad[1][0]
    bad[2][7] = n
    plan = S.stalloc_plan(*args, dev(bad, np.int32))
    assert int(plan["status"].item()) == 6
    torch.cuda.synchronize()


@pytest.mark.parametrize("least, most", [(1, 2), (1, 31), (24, 31), (31, 31)])
@pytest.mark.parametrize("n, alive", [(1100, 12), (1500, 60), (3001, 80), (4100, 60)])
def test_chains_of_clashing_requests(oracle, n, alive, least, most):
    """Orders in which nearly every request meets the one before it (by time, by release, by size), so that a chain of them is settled one
    after the other: places within the 64 granules from a candidate's word on, and, with large sizes in tall stacks, mostly beyond, where they
    are looked for in the bitmap, and random orders, which leave such chains again."""
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng([n, alive, least, most])
    ts = np.sort(rng.integers(0, 2 * n, n))
    te = ts + rng.integers(1, 4 * alive, n)
    size = (rng.integers(least, most + 1, n) * 512).astype(np.uint64)
    size[0] = 512                                                 # (the granule)
    mixed = rng.permutation(n)
    mixed[: n // 2].sort()                                        # first by time, then at random
    by_size = np.lexsort((ts, -size.astype(np.int64)))
    orders = np.stack([np.arange(n), np.arange(n)[::-1], np.argsort(te, kind="stable"), by_size, mixed, rng.permutation(n)]).astype(np.uint32)
    ts, te = ts.astype(np.uint32), te.astype(np.uint32)
    dev = lambda x, t: torch.from_numpy(np.ascontiguousarray(x).view(t)).cuda()
    plan = S.stalloc_plan(dev(size, np.int64), dev(ts, np.int32), dev(te, np.int32), int(te.max()), dev(orders, np.int32))
    S.check_status(plan)
    assert S.stalloc_plan_report(plan)["kernel"] == "bitmap" and _path(plan)[0] == 0
    a, ext = oracle.plan_many(size, ts, te, orders, threads=6, method="lists")
    assert np.array_equal(plan["peaks"].cpu().numpy().view(np.uint64), ext)
    assert np.array_equal(plan["offsets"].cpu().numpy().view(np.uint64), a)
