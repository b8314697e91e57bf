"""The gather's hits and misses in one launch: sides of different vector widths and strides, only hits, only misses, no rows; a
second half on its own; and the statistics of a gather without a cache."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def setup(n, dim, dtype, feat_pad, cached, cache_pad, seed=0):
    from paper_2601_04707_amd import mqg
    gen = torch.Generator(device="cuda").manual_seed(seed)
    g = mqg.Graph(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")[:0])
    feats = torch.randn((n, dim + feat_pad), generator=gen, device="cuda").to(dtype).cpu().pin_memory()[:, :dim]
    ctx = mqg.Context(g, 50_000, [1])
    cache = mqg.Cache(g, feats, cached, cache_stride=dim + cache_pad)
    mqg.mqg_build_cache(ctx, g, cache)
    return mqg, ctx, cache, feats.cuda(), gen


@pytest.mark.parametrize("dim,dtype,feat_pad,cache_pad", [(64, torch.float32, 0, 0), (100, torch.float32, 0, 0), (602, torch.float32, 6, 6),
                                                          (30, torch.float16, 0, 2), (30, torch.float16, 2, 0), (7, torch.float16, 0, 1),
                                                          (33, torch.float32, 0, 3), (1, torch.float16, 0, 0)])
def test_both_sides(dim, dtype, feat_pad, cache_pad):
    n = 3000
    mqg, ctx, cache, feats, gen = setup(n, dim, dtype, feat_pad, n // 3, cache_pad)
    slot = cache.slot_of
    hit, miss = torch.nonzero(slot >= 0).flatten(), torch.nonzero(slot < 0).flatten()
    mixed = torch.randint(-20, n + 20, (4000,), generator=gen, device="cuda")
    for ids in (mixed, hit, miss, mixed[:0], mixed[:1], hit[:1], miss[:1]):
        valid = (ids >= 0) & (ids < n)
        buf = torch.full((len(ids) + 1, dim + 8), 3.0, dtype=dtype, device="cuda")
        out = buf[:, :dim]
        stats = torch.zeros(2, dtype=torch.int64, device="cuda")
        num = torch.tensor([len(ids)], device="cuda")
        padded = torch.cat([ids, ids[:1] if len(ids) else torch.zeros(1, dtype=ids.dtype, device="cuda")])
        mqg.mqg_gather_features(ctx, cache, padded, num, out, stats)
        # a second half after the rows are copied copies nothing
        other = torch.full((len(ids) + 1, dim), 5.0, dtype=dtype, device="cuda")
        mqg.mqg_gather_features_missed(ctx, cache, padded, num, other)
        torch.cuda.synchronize()
        want = torch.full_like(out, 3.0)
        want[:-1][valid] = feats[ids[valid]]
        assert torch.equal(out, want) and torch.all(buf[:, dim + 7:] == 3.0)
        assert torch.all(other == 5.0)
        hits = int((slot[ids[valid]] >= 0).sum())
        assert stats.tolist() == [hits, int(valid.sum()) - hits]


@pytest.mark.parametrize("dim,dtype,feat_pad,cache_pad", [(64, torch.float32, 0, 0), (602, torch.float32, 6, 6), (602, torch.float32, 0, 14),
                                                          (30, torch.float16, 2, 2), (7, torch.float16, 1, 1), (7, torch.float16, 0, 1)])
@pytest.mark.parametrize("idx", [torch.int32, torch.int64])
def test_every_node_cached(dim, dtype, feat_pad, cache_pad, idx):
    """Also where the table of slots says otherwise for some nodes: their rows come from the feature matrix."""
    n = 3000
    mqg, ctx, cache, feats, gen = setup(n, dim, dtype, feat_pad, n, cache_pad)
    for gone in (0, 700, n):
        cache.slot_of[torch.randperm(n, generator=gen, device="cuda")[:gone]] = -1
        for count in (0, 1, 255, 4000, 45_000):
            ids = torch.randint(-20, n + 20, (max(count, 1) + 9,), generator=gen, device="cuda")
            valid = (ids >= 0) & (ids < n)
            valid[count:] = False
            buf = torch.full((len(ids), dim + 8), 3.0, dtype=dtype, device="cuda")
            stats = torch.full((2,), -1, dtype=torch.int64, device="cuda")
            for _ in range(2):
                mqg.mqg_gather_features(ctx, cache, ids.to(idx), torch.tensor([count], device="cuda"), buf[:, :dim], stats)
            torch.cuda.synchronize()
            want = torch.full((len(ids), dim), 3.0, dtype=dtype, device="cuda")
            want[valid] = feats[ids[valid]]
            assert torch.equal(buf[:, :dim], want) and torch.all(buf[:, dim + 7:] == 3.0)
            hits = int((cache.slot_of[ids[valid]] >= 0).sum())
            assert stats.tolist() == [hits, int(valid.sum()) - hits]


@pytest.mark.parametrize("rows", [1, 2000, 2047, 2048, 2049, 12_287, 12_288, 12_289, 40_000, 600_001])
@pytest.mark.parametrize("dim", [64, 602])
def test_statistics_without_a_cache(rows, dim):
    """A counting workgroup per 2,048 ids, 256 at most."""
    from paper_2601_04707_amd import mqg
    n = 5000
    gen = torch.Generator(device="cuda").manual_seed(rows)
    g = mqg.Graph(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")[:0])
    feats = torch.randn((n, dim), generator=gen, device="cuda")
    ctx = mqg.Context(g, 50_000, [1])
    cache = mqg.Cache(g, feats, None)
    for bad in (0, 1, rows):
        ids = torch.randint(0, n, (rows,), generator=gen, device="cuda")
        ids[torch.randperm(rows, generator=gen, device="cuda")[:bad]] = n + 3
        valid = ids < n
        want = torch.full((rows, dim), 2.0, device="cuda")
        want[valid] = feats[ids[valid]]
        for fewer in (0, rows // 2):
            out = torch.full((rows, dim), 2.0, device="cuda")
            stats = torch.zeros(2, dtype=torch.int64, device="cuda")
            mqg.mqg_gather_features(ctx, cache, ids, torch.tensor([rows - fewer], device="cuda"), out, stats)
            torch.cuda.synchronize()
            assert torch.equal(out[: rows - fewer], want[: rows - fewer]) and torch.all(out[rows - fewer:] == 2.0)
            assert stats.tolist() == [0, int(valid[: rows - fewer].sum())]


@pytest.mark.parametrize("dim,dtype,cap", [(16, torch.float32, 1 << 19), (16, torch.float32, (1 << 19) + 1), (32, torch.float32, (1 << 19) + 1),
                                           (45, torch.float16, 1 << 17), (45, torch.float16, (1 << 17) + 1), (6, torch.float32, (1 << 17) + 1)])
def test_every_node_cached_with_and_without_lists(dim, dtype, cap):
    """On both sides of the numbers of ids from which narrow rows go through the lists again."""
    from paper_2601_04707_amd import mqg
    n = 40_000
    gen = torch.Generator(device="cuda").manual_seed(dim)
    g = mqg.Graph(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(0, dtype=torch.int64, device="cuda"))
    feats = torch.randn((n, dim), generator=gen, device="cuda").to(dtype)
    ctx = mqg.Context(g, cap, [1])
    cache = mqg.Cache(g, feats.cpu().pin_memory(), n, cache_stride=dim)
    mqg.mqg_build_cache(ctx, g, cache)
    ids = torch.randint(-20, n + 20, (cap,), generator=gen, device="cuda")
    for num in (cap, 5000):
        valid = (ids >= 0) & (ids < n) & (torch.arange(cap, device="cuda") < num)
        out = torch.full((cap, dim), 3.0, dtype=dtype, device="cuda")
        stats = torch.zeros(2, dtype=torch.int64, device="cuda")
        mqg.mqg_gather_features(ctx, cache, ids, torch.tensor([num], device="cuda"), out, stats)
        want = torch.full_like(out, 3.0)
        want[valid] = feats[ids[valid]]
        assert torch.equal(out, want)
        assert stats.tolist() == [int(valid.sum()), 0]


def test_many_narrow_rows_with_every_node_cached():
    """1 M rows of 300 bytes, 4-byte vectors: as fast from a cache that holds every node as from one that lacks a single one (1.35
    times as long with a slot lookup per vector)."""
    from paper_2601_04707_amd import mqg
    n, num, dim = 2_000_000, 1_000_000, 150
    gen = torch.Generator(device="cuda").manual_seed(8)
    g = mqg.Graph(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(0, dtype=torch.int64, device="cuda"))
    feats = torch.zeros((n, dim), dtype=torch.float16, device="cuda")
    ctx = mqg.Context(g, num, [1])
    out = torch.empty((num, dim), dtype=torch.float16, device="cuda")
    count = torch.tensor([num], device="cuda")
    caches = [mqg.Cache(g, feats, k, cache_stride=dim) for k in (n, n - 1)]
    for cache in caches:
        mqg.mqg_build_cache(ctx, g, cache)
    cached = torch.nonzero(caches[1].slot_of >= 0).flatten()
    ids = cached[torch.randint(0, len(cached), (num,), generator=gen, device="cuda")]
    best = [float("inf")] * 2
    for _ in range(8):
        for k, cache in enumerate(caches):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                mqg.mqg_gather_features(ctx, cache, ids, count, out, None)
            b.record()
            torch.cuda.synchronize()
            best[k] = min(best[k], a.elapsed_time(b))
    assert best[0] < 1.15 * best[1], best
