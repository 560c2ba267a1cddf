"""stalloc_make_orders around the edges of its buckets (one bucket up to 2048 requests, 1536 a bucket beyond),
for windows of rows that begin and end at every kind of row, against the oracle; and the way around a bucket that
holds more numbers than it has room for, in a library of its own whose buckets are meant for 2040 of 2048."""
import ctypes
import os

import numpy as np
import pytest

from helpers import random_trace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[4096], [512, 1024, 8192, 1 << 33], None])
@pytest.mark.parametrize("n", [2047, 2048, 2049, 3072, 4080, 6120, 16385])
def test_edges_of_buckets_and_windows(oracle, n, sizes):
    import torch
    import paper_2507_16274_amd as S
    rng = np.random.default_rng(n)
    size, ts, te, t_end = random_trace(rng, n, t_max=n)
    size = rng.choice(np.asarray(sizes), n).astype(np.uint64) if sizes else rng.permutation(n).astype(np.uint64) + np.uint64(1)
    dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32))]
    for first, P in ((0, 9), (0, 1), (0, 4), (1, 4), (2, 1), (3, 1), (3, 6), (4, 5), (777, 8)):
        out = S.stalloc_make_orders(*dev, t_end, P, seed=n, first_plan=first)
        S.check_status(out)
        want = oracle.make_orders(size, ts, te, P, seed=n, first_plan=first)
        assert np.array_equal(out["orders"].cpu().numpy().view(np.uint32), want), (first, P)


@pytest.mark.parametrize("n, P", [(4080, 8), (6120, 8), (20400, 8), (20400, 200)])
def test_full_buckets_are_sorted_all_the_same(oracle, n, P):
    """(20400, 200): enough numbers for those that are stored in runs."""
    import torch
    import paper_2507_16274_amd as S
    from paper_2507_16274_amd import build
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libfullbuckets.so")
    lib = ctypes.CDLL(path if os.path.exists(path) else build.build_full_buckets())
    vp, u32 = ctypes.c_void_p, ctypes.c_uint32
    lib.stalloc_make_orders.argtypes = [ctypes.POINTER(S._Trace), u32, u32, ctypes.c_uint64, vp, vp, vp, ctypes.POINTER(ctypes.c_size_t), vp]
    rng = np.random.default_rng(n)
    size, ts, te, t_end = random_trace(rng, n, t_max=n)
    size = rng.choice([512, 1024, 8192, 1 << 33], n).astype(np.uint64)
    dev = [torch.from_numpy(x).cuda() for x in (size.view(np.int64), ts.view(np.int32), te.view(np.int32))]
    tr, first = S._trace(*dev, t_end), 3
    orders = torch.empty((P, n), dtype=torch.int32, device="cuda")
    status = torch.empty(1, dtype=torch.int32, device="cuda")
    need = ctypes.c_size_t(0)
    args = (ctypes.byref(tr), first, P, n, orders.data_ptr(), status.data_ptr())
    assert lib.stalloc_make_orders(*args, None, ctypes.byref(need), None) == 0
    ws = torch.empty(need.value, dtype=torch.uint8, device="cuda")
    assert lib.stalloc_make_orders(*args, ws.data_ptr(), ctypes.byref(need), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    # numbers per bucket: [rows][buckets] words in front of the buckets themselves, the last two pieces of the workspace
    buckets = n // 2040
    pieces = [-(-P * buckets * 4 // 256) * 256, P * buckets * 2048 * 4]
    at = need.value - sum(pieces)
    filled = ws[at:at + P * buckets * 4].view(torch.int32).view(P, buckets).cpu()
    assert (filled.sum(1) == n).all() and (filled > 2048).any(1).sum() >= 4, "buckets that hold more than they have room for"
    want = oracle.make_orders(size, ts, te, P, seed=n, first_plan=first)
    assert np.array_equal(orders.cpu().numpy().view(np.uint32), want)
