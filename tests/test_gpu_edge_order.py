"""The order of a block's edges by source: the way through buckets gives the same bits as the radix sort that blocks of more
than 2^22 sources take (capacity decides), at the edges of its buckets, ranges and chunks."""
import numpy as np
import pytest
import torch

from gpu_util import to_dev
from test_gpu_backward import bare_blocks

pytestmark = pytest.mark.gpu


def backward(mqg, ctx, blocks, cap_src, ns, g, w):
    nd, nnz = blocks.bounds[0][0], blocks.bounds[0][2]
    ip, ix, sizes, _ = blocks._keep
    blocks.c[0] = mqg.CBlock(nd, cap_src, max(nnz, 1), None, ip.data_ptr(), ix.data_ptr(), sizes.data_ptr())
    gx = torch.full((cap_src, g.shape[1]), 7.0, dtype=g.dtype, device="cuda")
    if w is None:
        mqg.mqg_sage_mean_aggregate_backward(ctx, blocks, 0, g, gx)
    else:
        mqg.mqg_weighted_aggregate_backward(ctx, blocks, 0, w, None, g, gx)
    torch.cuda.synchronize()
    assert torch.all(gx[ns:] == 7.0)
    return gx[:ns]


# (sources, edges, how the edges choose them): one source up to several ranges a bucket, all edges in one bucket or
# one source (several chunks), a launch per number of tiles
CASES = [(1, 700, "all"), (255, 9000, "all"), (256, 9000, "all"), (257, 9000, "all"), (2047 * 256, 70_000, "all"),
         (1 << 19, 300_000, "all"), ((1 << 19) + 1, 300_000, "all"), (3_000_000, 900_000, "all"), (1 << 22, 200_000, "ends"),
         (600_000, 200_000, "one"), (600_000, 16_384, "one"), (600_000, 16_385, "one"), (2, 5000, "all"), (513, 5000, "all"), (1025, 90_000, "all"), (2049, 90_000, "all"), (600_000, 150_000, "bucket"),
         (1_200_000, 400_000, "bucket"), (300, 65_536, "one"), (5000, 0, "all")]


@pytest.mark.parametrize("ns,nnz,how", CASES)
@pytest.mark.parametrize("weighted", [False, True])
def test_same_bits_as_the_radix_sort(ns, nnz, how, weighted):
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(ns + nnz)
    nd = max(1, nnz // 7)
    lens = rng.multinomial(nnz, np.full(nd, 1 / nd))
    indptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    if how == "all":
        cols = rng.integers(0, ns, nnz)
        cols[: min(nnz, 1)] = ns - 1
    elif how == "ends":
        cols = rng.choice([0, 1, ns // 2, ns - 1], nnz)
    elif how == "one":
        cols = np.full(nnz, ns // 3)
    else:
        cols = ns // 2 + rng.integers(0, 3000, nnz)
    ctx, blocks = bare_blocks(mqg, indptr, cols, nd, ns)
    g = torch.from_numpy(rng.standard_normal((nd, 3)).astype(np.float32)).cuda()
    w = to_dev(torch.from_numpy(rng.random(max(nnz, 1), dtype=np.float32))) if weighted else None
    got = backward(mqg, ctx, blocks, ns, ns, g, w)
    want = backward(mqg, ctx, blocks, (1 << 22) + 1, ns, g, w)
    assert torch.equal(got, want)
    again = backward(mqg, ctx, blocks, min(1 << 22, 8 * ns + 5), ns, g, w)       # more ranges than the sources need
    assert torch.equal(again, want)
    # the sums in 64 bits, on the CPU
    rows = np.repeat(np.arange(nd), lens)
    coeff = w[:nnz].double().cpu().numpy() if weighted else 1.0 / np.maximum(lens, 1)[rows]
    gh, terms = g.double().cpu().numpy()[rows], np.bincount(cols, minlength=ns)
    for c in range(3):
        ref = np.bincount(cols, weights=coeff * gh[:, c], minlength=ns)
        mag = np.bincount(cols, weights=coeff * np.abs(gh[:, c]), minlength=ns)
        assert np.all(np.abs(got[:, c].double().cpu().numpy() - ref) <= (terms + 4) * 2.0 ** -24 * mag)


def crowded(nnz, ns, how, rng):
    if how == "one":
        return np.full(nnz, ns // 3)
    if how == "bucket":
        return np.minimum(ns // 2 + rng.integers(0, 700, nnz), ns - 1)
    if how == "hub":
        cols = rng.integers(0, ns, nnz)
        cols[rng.random(nnz) < 0.6] = ns // 5
        return cols
    p = 1 / (np.arange(ns) + 3.0)
    return rng.choice(ns, nnz, p=p / p.sum())


# buckets around one chunk (4,096 edges; 8,192 and more where a bucket has as many sources), around the 131,072 edges from
# which chunks are counted in a launch of their own, in blocks on both sides of 2^20 and 2^23 edges, of 1 to 8,192 sources
@pytest.mark.parametrize("ns,nnz,how", [(400, 4096, "one"), (400, 4097, "one"), (2, 40_000, "zipf"), (4000, 131_072, "one"), (4000, 131_073, "one"),
                                        (400, 200_000, "one"), (3, 300_000, "zipf"), (20_000, 300_000, "zipf"), (700_000, 300_000, "hub"),
                                        (2_000_000, 400_000, "bucket"), ((1 << 22) - 3, 400_000, "hub"), (5000, 1 << 20, "zipf"),
                                        (600_000, (1 << 20) + 1, "hub"), (1_100_000, 1_500_000, "bucket"), (1 << 22, 2_000_001, "one"),
                                        (60_000, (1 << 23) + 5, "zipf"), (1 << 22, (1 << 23) + 70_001, "hub")])
@pytest.mark.parametrize("weighted", [False, True])
def test_crowded_buckets(ns, nnz, how, weighted):
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(ns + nnz)
    cols = crowded(nnz, ns, how, rng)
    nd = max(1, nnz // 9)
    indptr = np.minimum(np.arange(nd + 1) * 9, nnz)
    indptr[-1] = nnz
    ctx, blocks = bare_blocks(mqg, indptr, cols, nd, ns)
    g = torch.from_numpy(rng.standard_normal((nd, 2)).astype(np.float32)).cuda()
    w = to_dev(torch.from_numpy(rng.random(nnz, dtype=np.float32))) if weighted else None
    got = backward(mqg, ctx, blocks, ns, ns, g, w)
    want = backward(mqg, ctx, blocks, (1 << 22) + 1, ns, g, w)
    assert torch.equal(got, want)
    again = backward(mqg, ctx, blocks, ns, ns, g, w)       # after another block's order on the same scratch
    assert torch.equal(again, want)


@pytest.mark.parametrize("how", ["one", "bucket", "hub"])
def test_crowded_buckets_take_no_more_than_a_few_times_as_long(how):
    """The order of 2 M edges of which most share a source or a bucket, against 2 M spread evenly (at most twice;
    11 to 63 times with every chunk counting the whole bucket)."""
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(1)
    ns, nnz = 600_000, 2_000_000
    indptr = np.arange(nnz // 10 + 1) * 10
    g = torch.zeros((nnz // 10, 2), device="cuda")
    took = []
    for cols in (rng.integers(0, ns, nnz), crowded(nnz, ns, how, rng)):
        ctx, blocks = bare_blocks(mqg, indptr, cols, nnz // 10, ns)
        gx = torch.empty((ns, 2), device="cuda")
        ctx.set_option(mqg.MQG_OPT_PROFILE, 1)
        mqg.mqg_sage_mean_aggregate_backward(ctx, blocks, 0, g, gx)
        best = float("inf")
        for _ in range(5):
            ctx.reset_profile()
            mqg.mqg_sage_mean_aggregate_backward(ctx, blocks, 0, g, gx)
            torch.cuda.synchronize()
            best = min(best, sum(ctx.kernel_time(k)[0] for k in ctx.kernel_names() if k.startswith("k_order") or k.startswith("k_radix")))
        took.append(best)
    assert took[1] < 5 * took[0], took
