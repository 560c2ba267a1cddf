"""stalloc_validate on calls large enough for the forms that leave out pairs that cannot meet (n * n * P >= 3e8), against the
oracle and against the all-pairs form, which a call with a smaller call's workspace gets."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

WORK = 1_500_000_000                                          # n * n * P


def _trace(rng, n, kind):
    t_end = {"dense": 40, "ties": n // 8 + 4, "mixed": 2 * n, "sparse": 1000 * n}[kind]
    ts = rng.integers(0, t_end - 1, n)
    life = np.exp(rng.uniform(0, np.log(t_end), n)).astype(np.int64) if kind != "dense" else rng.integers(1, 40, n)
    te = np.minimum(ts + np.maximum(life, 1), t_end)
    return rng.integers(1, 50, n).astype(np.uint64), ts.astype(np.uint32), te.astype(np.uint32), int(t_end)


@pytest.mark.parametrize("kind", ["dense", "ties", "mixed", "sparse"])
@pytest.mark.parametrize("n", [63, 64, 65, 257, 4097, 20011])
def test_near_pairs_match_all_pairs(oracle, n, kind):
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(n)
    size, ts, te, t_end = _trace(rng, n, kind)
    P = -(-WORK // (n * n)) + 3                               # a count that is no multiple of four, too
    plans = rng.integers(0, 60 * n, (P, n)).astype(np.int64)  # a few conflicts per plan and request
    plans[P // 2] = 0                                         # ... and one in which everything conflicts that can
    dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32), plans)]
    out = S.stalloc_validate(*dev[:3], t_end, dev[3])
    S.check_status(out)
    cnt, pair = out["conflicts"].cpu().numpy(), out["first_pair"].cpu().numpy()
    rows = sorted({0, 1, 2, 3, P // 2, P - 2, P - 1} | set(rng.integers(0, P, 5).tolist()))
    for p in rows if n < 5000 else rows[:2] + [P // 2]:
        want = oracle.validate(size, ts, te, plans[p].view(np.uint64))
        assert (int(cnt[p]), tuple(int(x) & 0xFFFFFFFF for x in pair[p])) == want
    conflicts, first, status = _all_pairs(S, dev[:3], t_end, dev[3])
    assert int(status.item()) == 0
    assert torch.equal(out["conflicts"], conflicts) and torch.equal(out["first_pair"], first)


def test_near_pairs_report_a_range_that_would_wrap(oracle):
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(3)
    n = 20011
    size, ts, te, t_end = _trace(rng, n, "mixed")
    plan = rng.integers(0, 1 << 40, (1, n)).astype(np.int64)
    size[n // 2] = 1
    for P in (4, 1):                                          # (four plans: one form or the other, by how many are alive together)
        for bad, start, status in ((0, -1, 3), (n // 2, -1, 3), (n - 1, -1, 3),       # 2^64 - 1: any size wraps, 1 as well
                                   (n // 2, -2, 0), (7, -1 - int(size[7]), 0)):       # ... and these end at 2^64 - 1
            bent = np.repeat(plan, P, axis=0)
            bent[P - 1, bad] = start
            dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32), bent)]
            out = S.stalloc_validate(*dev[:3], t_end, dev[3])
            assert int(out["status"].item()) == status, (P, bad, start)
            assert int(_all_pairs(S, dev[:3], t_end, dev[3])[2].item()) == status, (P, bad, start)


def _all_pairs(S, dev, t_end, plans):
    """The call with no more workspace than the all-pairs form needs, which a call always accepts."""
    import torch
    n, P = plans.shape[1], plans.shape[0]
    out = [torch.empty(P, dtype=torch.int64, device="cuda"), torch.empty((P, 2), dtype=torch.int32, device="cuda"),
           torch.empty(1, dtype=torch.int32, device="cuda")]
    need = ctypes.c_size_t(0)
    few = S._trace(*[t[:2] for t in dev], t_end)
    assert S.lib.stalloc_validate(ctypes.byref(few), plans.data_ptr(), P, *[o.data_ptr() for o in out], None, ctypes.byref(need), None) == 0
    ws = torch.empty(need.value, dtype=torch.uint8, device="cuda")
    tr = S._trace(*dev, t_end)
    stream = torch.cuda.current_stream().cuda_stream
    assert S.lib.stalloc_validate(ctypes.byref(tr), plans.data_ptr(), P, *[o.data_ptr() for o in out], ws.data_ptr(),
                                  ctypes.byref(need), stream) == 0
    need.value -= 1
    assert S.lib.stalloc_validate(ctypes.byref(tr), plans.data_ptr(), P, *[o.data_ptr() for o in out], ws.data_ptr(),
                                  ctypes.byref(need), stream) == 1
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("P", [1, 3, 4, 6])
@pytest.mark.parametrize("kind", ["dense", "crowded", "ties", "mixed", "sparse", "far end"])
def test_both_forms_agree_on_few_plans(kind, P):
    """Beyond the lengths at which plans are gone through four at a time; in crowded traces all requests count as long-lived."""
    import torch
    import paper_2507_16274_amd as S
    n = 40011
    rng = np.random.default_rng(n + P)
    if kind == "crowded":
        ts, te = np.sort(rng.permutation(2 * n).reshape(n, 2), axis=1).T
        size, t_end = rng.integers(1, 50, n).astype(np.uint64), 2 * n
        ts, te = np.ascontiguousarray(ts).astype(np.uint32), np.ascontiguousarray(te).astype(np.uint32)
    else:
        size, ts, te, t_end = _trace(rng, n, "mixed" if kind == "far end" else kind)
        t_end = 1 << 30 if kind == "far end" else t_end
    dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32))]
    plans = torch.from_numpy(rng.integers(0, 60 * n, (P, n)).astype(np.int64)).cuda()
    out = S.stalloc_validate(*dev, t_end, plans)
    S.check_status(out)
    conflicts, first, status = _all_pairs(S, dev, t_end, plans)
    assert int(status.item()) == 0 and (conflicts > 0).all()
    assert torch.equal(out["conflicts"], conflicts) and torch.equal(out["first_pair"], first)


def _alive(rng, n, alive):
    """About `alive` requests at a time."""
    ts = np.arange(n) * 2
    te = ts + 2 * rng.integers(1, max(2, 2 * alive), n)
    return rng.integers(1, 50, n).astype(np.uint64), ts.astype(np.uint32), te.astype(np.uint32), int(te.max())


@pytest.mark.parametrize("alive", [4, 50, 150])
@pytest.mark.parametrize("n", [5, 63, 64, 65, 128, 129, 223, 224, 225, 257, 2048, 2049, 8192, 8193])
def test_four_plans_a_wave(n, alive):
    """Lengths around one, two and four tiles and around those at which plans are gone through four at a time, always or if few requests
    are alive together; a number of plans that is no multiple of four; requests numbered by time and not."""
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng([n, alive])
    size, ts, te, t_end = _alive(rng, n, alive)
    if n % 2:
        mixed = rng.permutation(n)
        size, ts, te = size[mixed], ts[mixed], te[mixed]
    P = max(300_000_000 // (n * n), 4_000_000 // n) + 3
    dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32))]
    gen = torch.Generator(device="cuda").manual_seed(n)
    plans = torch.randint(0, 25 * min(n, 2 * alive) * 4 + 1, (P, n), device="cuda", generator=gen)
    plans[::3] *= 1000                                        # (mostly without conflicts)
    out = S.stalloc_validate(*dev, t_end, plans)
    S.check_status(out)
    conflicts, first, status = _all_pairs(S, dev, t_end, plans)
    assert int(status.item()) == 0
    assert torch.equal(out["conflicts"], conflicts) and torch.equal(out["first_pair"], first)
    plans[P - 2, n // 2] = -1
    assert int(S.stalloc_validate(*dev, t_end, plans)["status"].item()) == 3


def test_short_traces_with_few_alive_take_half_of_all_pairs():
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(11)
    n, P = 200, 60000
    size, ts, te, t_end = _alive(rng, n, 20)
    te[::70] += 300                                           # (spans of time reach far)
    t_end = int(te.max())
    dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32))]
    plans = torch.from_numpy((np.cumsum(size) - size).astype(np.int64) % 1000).cuda().expand(P, n).contiguous()     # (addresses are used anew)
    need = ctypes.c_size_t(0)
    few, tr = S._trace(*[t[:2] for t in dev], t_end), S._trace(*dev, t_end)
    out = [torch.empty(P, dtype=torch.int64, device="cuda"), torch.empty((P, 2), dtype=torch.int32, device="cuda"),
           torch.empty(1, dtype=torch.int32, device="cuda")]
    took = []
    for asked in (few, tr):
        args = (plans.data_ptr(), P, *[o.data_ptr() for o in out])
        assert S.lib.stalloc_validate(ctypes.byref(asked), *args, None, ctypes.byref(need), None) == 0
        ws = torch.empty(need.value, dtype=torch.uint8, device="cuda")
        best = 1e9
        for _ in range(10):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            assert S.lib.stalloc_validate(ctypes.byref(tr), *args, ws.data_ptr(), ctypes.byref(need), torch.cuda.current_stream().cuda_stream) == 0
            end.record()
            end.synchronize()
            best = min(best, begin.elapsed_time(end))
        took.append(best)
    assert took[1] < 0.55 * took[0], took                     # ms; 1.01 and 0.69 with a plan a wave, 0.44 with four
