"""The forms of the trace check, the lower bound, the time-memory products and the choice of the best plan for
short traces and few plans, around the sizes where the other forms take over, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t_end", [3, 1023, 16383, 16384])
@pytest.mark.parametrize("n", [1, 1023, 8192, 8193, 16384, 16385])
def test_checks_bounds_and_products(oracle, n, t_end):
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(n + t_end)
    ts = rng.integers(0, t_end, n)
    te = np.minimum(ts + rng.integers(1, 40, n), t_end)
    size = rng.integers(1, 1 << 41, n).astype(np.uint64)
    dev = lambda x, t: torch.from_numpy(np.ascontiguousarray(x).view(t)).cuda()
    for broken in (None, "size", "life", "end", "sum"):
        s, a, f = size.copy(), ts.astype(np.uint32), te.astype(np.uint32)
        k = n - 1
        if broken == "size":
            s[k] = 0
        elif broken == "life":
            f[k] = a[k]
        elif broken == "end":
            f[k] = t_end + 1
        elif broken == "sum":
            s[k] = (1 << 63) - 1 if n > 1 else 1 << 63
        args = (dev(s, np.int64), dev(a, np.int32), dev(f, np.int32), t_end)
        lb = S.stalloc_lower_bound(*args)
        ext = rng.integers(1 << 41, 1 << 50, 7 if n % 2 else 8193)
        tmp = S.stalloc_tmp(*args, dev(ext, np.int64))
        want = {None: 0, "sum": 3}.get(broken, 2)
        assert int(lb["status"].item()) == want and int(tmp["status"].item()) == want
        if broken is None:
            assert (int(lb["lower_bound"].item()), int(lb["t_at_max"].item())) == oracle.lower_bound(s, a, f, t_end)
            used = sum(int(x) * int(y) for x, y in zip(s, f.astype(np.int64) - a))
            span = int(f.max()) - int(a.min())
            exact = np.asarray([used / (int(e) * span) for e in ext])
            assert np.all(np.abs(tmp["tmp"].cpu().numpy() - exact) <= 10 * 2.0 ** -53 * exact)    # eight roundings at most


@pytest.mark.parametrize("P", [1, 255, 4096, 4097])
def test_best_plan_and_its_addresses(P):
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(P)
    n = 40
    ts = np.sort(rng.integers(0, 60, n))
    te = ts + rng.integers(1, 30, n)
    dev = lambda x, t: torch.from_numpy(np.ascontiguousarray(x).astype(t)).cuda()
    orders = dev(np.stack([rng.permutation(n) for _ in range(P)]), np.int32)
    args = (dev(rng.integers(1, 20, n) * 512, np.int64), dev(ts, np.int32), dev(te, np.int32), int(te.max()))
    plan = S.stalloc_plan(*args, orders)
    S.check_status(plan)
    best = int(plan["best_plan"].item())
    assert best == int(np.argmin(plan["peaks"].cpu().numpy()))
    assert torch.equal(plan["best_offsets"], plan["offsets"][best])
    assert int(S.stalloc_plan(*args, orders, want_best_offsets=False)["best_plan"].item()) == best
