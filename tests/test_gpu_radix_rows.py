"""The radix sort where its scan of the digit counts changes: just above the 32 tiles that need no scan, digits of 8 to
11 bits, and on both sides of the 2,048 tiles that one round of the scan's loop takes.  The order is exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,max_deg", [(65_536, 200), (65_537, 200), (66_000, 1_000), (300_001, 2_000), (700_000, 90_000), (2_097_153, 300),
                                       (4_194_304, 300), (4_194_305, 300_000), (8_390_000, 5)])
def test_nodes_ranked_by_degree(n, max_deg):
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(n)
    deg = rng.integers(0, 4, n)
    high = rng.integers(0, n, 50)
    deg[high] = rng.integers(0, max_deg + 1, 50)
    deg[high[0]] = max_deg
    row_ptr = torch.zeros(n + 1, dtype=torch.int64)
    row_ptr[1:] = torch.from_numpy(np.cumsum(deg))
    g = mqg.Graph(row_ptr.cuda(), torch.zeros(int(row_ptr[-1]), dtype=torch.int32, device="cuda"))
    ctx = mqg.Context(g, 1, [1])
    cache = mqg.Cache(g, torch.zeros((n, 2), device="cuda"), n)
    mqg.mqg_build_cache(ctx, g, cache)
    torch.cuda.synchronize()
    want = torch.from_numpy(np.argsort(-deg, kind="stable").astype(np.int32))      # equal degrees: smaller id first
    assert torch.equal(cache.cached_ids.cpu(), want)
    ctx.close()
