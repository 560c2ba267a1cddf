"""stalloc_make_orders around the edges of its buckets (one bucket up to 2048 requests, 1536 a bucket beyond),
for windows of rows that begin and end at every kind of row, against the oracle.  A build with
-DSTALLOC_OR_BUCKET_MEAN=2040 overfills buckets at 4080 and 6120 requests (the same results, slowly)."""
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
