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
