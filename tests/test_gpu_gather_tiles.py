"""The split of the ids into hits and misses at the edges of its tiles (1,024 ids, 4,096 above 512 k) and of its
workgroups' loop, with ids outside the graph among them.  Bytes and counts are exact."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("num_ids,cap,idx", [(1, 1, torch.int64), (1023, 1024, torch.int32), (1025, 1025, torch.int64), (5000, 524_288, torch.int32),
                                             (524_288, 524_288, torch.int64), (4097, 524_289, torch.int64), (700_001, 700_001, torch.int32)])
def test_tiles_of_ids(num_ids, cap, idx):
    from paper_2601_04707_amd import mqg
    gen = torch.Generator(device="cuda").manual_seed(num_ids)
    n, dim = 50_000, 8
    deg = torch.randint(0, 9, (n,), generator=gen, device="cuda")
    row_ptr = torch.zeros(n + 1, dtype=idx, device="cuda")
    row_ptr[1:] = torch.cumsum(deg, 0).to(idx)
    g = mqg.Graph(row_ptr, torch.zeros(int(row_ptr[-1]), dtype=idx, device="cuda"))
    feats = torch.randn((n, dim), generator=gen, device="cuda")
    host = feats.cpu().pin_memory()
    ctx = mqg.Context(g, 1 << 17, [6])
    ids = torch.randint(0, n, (cap,), generator=gen, device="cuda")
    bad = torch.rand(cap, generator=gen, device="cuda") < 0.01
    bad[0] = False
    ids[bad] = torch.where(torch.rand(int(bad.sum()), generator=gen, device="cuda") < 0.5, -1 - ids[bad], n + ids[bad])
    out = torch.full((cap, dim), 9.0, device="cuda")
    stats = torch.zeros(2, dtype=torch.int64, device="cuda")
    count = torch.tensor([num_ids], device="cuda")
    cache = mqg.Cache(g, host, n // 3)
    mqg.mqg_build_cache(ctx, g, cache)
    used = torch.arange(cap, device="cuda") < num_ids
    valid = used & ~bad
    want = torch.full((cap, dim), 9.0, device="cuda")
    want[valid] = feats[ids[valid]]
    hits = int((cache.slot_of[ids[valid]] >= 0).sum())
    for _ in range(2):                                     # the counters are clear for the second call
        out.fill_(9.0)
        mqg.mqg_gather_features_static(cache, ids.to(idx), count, out, stats)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert stats.tolist() == [hits, int(valid.sum()) - hits]
