"""The segmented reduction where its runs of rows begin, end and are cut: row counts around the number of
wavefronts of a launch (32,768) and its multiples, rows without entries, rows of more than the 64
entries that are fetched at a time, rows narrower and wider than a wavefront, diagonal terms of zero.

Against float64 sums.  Bound per element: a sum of n fp32 products has an error of at most (n + 2) 2^-24
times the sum of its terms' magnitudes; a result stored as fp16 is rounded once more, by 2^-11 of itself.
"""
import numpy as np
import pytest
import scipy.sparse
import torch

from test_gpu_backward import bare_blocks

pytestmark = pytest.mark.gpu


def spmm(rows, cols, w, x, n):
    """out[rows[e]] += w[e] x[cols[e]] in float64, on the CPU."""
    m = scipy.sparse.csr_matrix((w.cpu().numpy(), (rows.cpu().numpy(), cols.cpu().numpy())), shape=(n, x.shape[0]))
    return torch.from_numpy(m @ x.cpu().numpy()).cuda()


@pytest.mark.parametrize("num_dst,dim,dtype", [(1, 5, torch.float32), (17, 70, torch.float16), (32_768, 3, torch.float32), (32_769, 64, torch.float16),
                                               (70_001, 33, torch.float32), (70_001, 130, torch.float16), (40_000, 260, torch.float32),
                                               (3_000, 1030, torch.float32), (530_000, 16, torch.float16), (600_000, 9, torch.float32)])
def test_runs_of_rows(num_dst, dim, dtype):
    check_runs(num_dst, dim, dtype, dim)


# several vectors of 16 bytes per lane: two to four forward, up to six backward; slabs
@pytest.mark.parametrize("dim,dtype", [(390, torch.float32), (516, torch.float32), (602, torch.float32), (780, torch.float32), (1150, torch.float32),
                                       (1500, torch.float32), (600, torch.float16), (1100, torch.float16), (1570, torch.float16),
                                       (2100, torch.float16), (2900, torch.float16), (3100, torch.float16)])
def test_runs_of_wide_padded_rows(dim, dtype):
    check_runs(2_100, dim, dtype, -(-dim // 8) * 8)


def check_runs(num_dst, dim, dtype, stride):
    from paper_2601_04707_amd import mqg
    gen = torch.Generator(device="cuda").manual_seed(num_dst + dim)
    lens = torch.randint(0, 7, (num_dst,), generator=gen, device="cuda")
    lens[torch.randint(0, num_dst, (max(1, num_dst // 50),), generator=gen, device="cuda")] = 0
    lens[num_dst // 2] = 300
    num_src = num_dst + 500
    indptr = torch.zeros(num_dst + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=indptr[1:])
    nnz = int(indptr[-1])
    rows = torch.repeat_interleave(torch.arange(num_dst, device="cuda"), lens)
    cols = torch.randint(0, num_src, (nnz,), generator=gen, device="cuda")
    cols[: nnz // 4] = num_src // 3                        # one source that a quarter of the edges point to
    ctx, blocks = bare_blocks(mqg, indptr.cpu().numpy(), cols.cpu().numpy(), num_dst, num_src)
    x = torch.randn((num_src, stride), generator=gen, device="cuda").to(dtype)[:, :dim]
    g = torch.randn((num_dst, stride), generator=gen, device="cuda").to(dtype)[:, :dim]
    ew = torch.randn(max(nnz, 1), generator=gen, device="cuda")
    sw = torch.randn(num_dst, generator=gen, device="cuda")
    sw[::3] = 0                                            # a diagonal term of zero is no term:
    xi = torch.empty((num_src, stride), dtype=dtype, device="cuda")[:, :dim].copy_(x)
    xi[:num_dst:3] = float("inf")                          # its input row may hold anything, as long as no edge reads it
    keep = ~((cols < num_dst) & (cols % 3 == 0))
    out = torch.full((num_dst + 1, stride), 7.0, dtype=dtype, device="cuda")[:, :dim]
    gx = torch.full((num_src + 1, stride), 7.0, dtype=dtype, device="cuda")[:, :dim]

    def check(got, rows, cols, w, x, n, scale=None, diag=None):
        ref, mag = spmm(rows, cols, w, x.double(), n), spmm(rows, cols, w.abs(), x.double().abs(), n)
        terms = torch.from_numpy(np.bincount(rows.cpu().numpy(), minlength=n)).double().cuda()
        if diag is not None:
            ref[: len(diag)] += diag[:, None] * x.double()[: len(diag)]
            mag[: len(diag)] += diag.abs()[:, None] * x.double()[: len(diag)].abs()
        if scale is not None:
            ref, mag = ref * scale[:, None], mag * scale[:, None]
        bound = (terms + 4)[:, None] * 2.0 ** -24 * mag + (2.0 ** -11 * ref.abs() + 2.0 ** -24 if dtype == torch.float16 else 0)
        assert torch.all((got[:n].double() - ref).abs() <= bound)
        assert torch.all(got[n:] == 7.0)

    one = torch.ones(nnz, dtype=torch.float64, device="cuda")
    inv = 1 / lens.clamp(min=1).double()
    mqg.mqg_sage_mean_aggregate(ctx, blocks, 0, x, out)
    check(out, rows, cols, one, x, num_dst, scale=inv)
    mqg.mqg_sage_mean_aggregate_backward(ctx, blocks, 0, g, gx)
    check(gx, cols, rows, inv[rows], g, num_src)
    w = ew[:nnz].double()
    mqg.mqg_weighted_aggregate(ctx, blocks, 0, ew, sw, x, out)
    check(out, rows, cols, w, x, num_dst, diag=sw.double())
    mqg.mqg_weighted_aggregate_backward(ctx, blocks, 0, ew, sw, g, gx)
    check(gx, cols, rows, w, g, num_src, diag=sw.double())
    # rows that only see finite inputs stay finite next to a zero-weight diagonal over an infinite row
    mqg.mqg_weighted_aggregate(ctx, blocks, 0, ew, sw, xi, out)
    dirty = torch.zeros(num_dst, dtype=torch.bool, device="cuda")
    dirty[rows[~keep]] = True
    assert torch.all(torch.isfinite(out[:num_dst][~dirty & (sw == 0)]))


@pytest.mark.parametrize("scale", [1, 60, 80])
@pytest.mark.parametrize("cap_src", [3000, (1 << 22) + 1])
def test_edges_find_their_rows(scale, cap_src):
    """The backward's order of edges where rows are empty in long stretches, hold one edge each, or thousands: through buckets, and
    with room for more than 2^22 sources through a radix sort (scale 80: enough edges for its weighted form to write all
    rows down first)."""
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(scale)
    lens = np.concatenate([np.zeros(70), [3], np.zeros(5000), np.ones(700), [9000, 0, 0, 64, 1], np.zeros(64), np.full(300, 2),
                           np.zeros(20_000), [513, 511], rng.integers(0, 40, 500), np.zeros(130)]).astype(np.int64)
    lens = np.tile(lens, scale)
    indptr = np.concatenate([[0], np.cumsum(lens)])
    nd, nnz, ns = len(lens), int(indptr[-1]), 3000
    assert (nnz > 3 << 19) == (scale == 80)
    cols = rng.integers(0, ns, nnz)
    cols[cols == 17] = 18                                  # a source without edges
    ctx, blocks = bare_blocks(mqg, indptr, cols, nd, ns)
    blocks.c[0].cap_src = cap_src
    rows = torch.from_numpy(np.repeat(np.arange(nd), lens))
    g = torch.randn((nd, 2), device="cuda")
    w = torch.rand(nnz, device="cuda")
    gx = torch.full((cap_src, 2), 7.0, device="cuda")
    for weights in (None, w):
        coeff = w.double() if weights is not None else (1.0 / torch.from_numpy(np.maximum(lens, 1)).double())[rows].cuda()
        ref = spmm(torch.from_numpy(cols), rows, coeff, g.double(), ns)
        mag = spmm(torch.from_numpy(cols), rows, coeff, g.double().abs(), ns)
        terms = torch.from_numpy(np.bincount(cols, minlength=ns)).double().cuda()
        if weights is None:
            mqg.mqg_sage_mean_aggregate_backward(ctx, blocks, 0, g, gx)
        else:
            mqg.mqg_weighted_aggregate_backward(ctx, blocks, 0, w, None, g, gx)
        assert torch.all((gx[:ns].double() - ref).abs() <= (terms + 4)[:, None] * 2.0 ** -24 * mag)


@pytest.mark.parametrize("nd,per_row,extra", [(1, 3, 700), (64, 2, 5), (65, 1, 130), (1300, 2, 700), (20_001, 80, 3000)])
@pytest.mark.parametrize("cap_src", [500, (1 << 22) + 1])
def test_edges_past_the_last_offset(nd, per_row, extra, cap_src):
    """A block whose edge count is larger than its last offset: the edges past it are the last row's, in the order through
    buckets and in the radix sort of blocks with room for more than 2^22 sources."""
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(nd)
    lens = np.full(nd, per_row)
    indptr = np.concatenate([[0], np.cumsum(lens)])
    nnz, ns = int(indptr[-1]) + extra, 500
    cols = rng.integers(0, ns, nnz)
    offsets = indptr.copy()
    offsets[-1] = nnz                                      # the buffers' size; the block's own last offset follows
    ctx, blocks = bare_blocks(mqg, offsets, cols, nd, ns)
    blocks._keep[0][nd] = int(indptr[-1])
    blocks.c[0].cap_src = cap_src
    rows = torch.from_numpy(np.concatenate([np.repeat(np.arange(nd), lens), np.full(extra, nd - 1)]))
    g = torch.randn((nd, 2), device="cuda")
    w = torch.rand(nnz, device="cuda")
    gx = torch.zeros((cap_src, 2), device="cuda")
    for weights in (None, w):
        coeff = w.double() if weights is not None else torch.full((nnz,), 1.0 / per_row, dtype=torch.float64, device="cuda")
        ref = spmm(torch.from_numpy(cols), rows, coeff, g.double(), ns)
        mag = spmm(torch.from_numpy(cols), rows, coeff, g.double().abs(), ns)
        terms = torch.from_numpy(np.bincount(cols, minlength=ns)).double().cuda()
        if weights is None:
            mqg.mqg_sage_mean_aggregate_backward(ctx, blocks, 0, g, gx)
        else:
            mqg.mqg_weighted_aggregate_backward(ctx, blocks, 0, w, None, g, gx)
        assert torch.all((gx[:ns].double() - ref).abs() <= (terms + 4)[:, None] * 2.0 ** -24 * mag)


def test_rows_wider_than_one_launch():
    """131,073 fp16 columns (one element per lane) of a block with room for 40,000 rows: more threads than a launch may
    have, so the columns are taken in pieces."""
    from paper_2601_04707_amd import mqg
    nd, cap, dim = 3, 40_000, 131_073
    indptr, cols = np.array([0, 2, 2, 5]), np.array([4, 1, 0, 3, 4])
    ctx, blocks = bare_blocks(mqg, indptr, cols, nd, 5)
    blocks.c[0].cap_dst = cap
    x = torch.randn((5, dim), device="cuda").half()
    out = torch.empty((cap, dim), dtype=torch.float16, device="cuda")
    out[nd] = 7.0
    mqg.mqg_sage_mean_aggregate(ctx, blocks, 0, x, out)
    xd = x.double()
    want = torch.stack([(xd[4] + xd[1]) / 2, torch.zeros(dim, device="cuda", dtype=torch.float64), (xd[0] + xd[3] + xd[4]) / 3])
    mag = torch.stack([(xd[4].abs() + xd[1].abs()) / 2, torch.zeros(dim, device="cuda", dtype=torch.float64),
                       (xd[0].abs() + xd[3].abs() + xd[4].abs()) / 3])
    assert torch.all((out[:nd].double() - want).abs() <= 7 * 2.0 ** -24 * mag + 2.0 ** -11 * want.abs() + 2.0 ** -24)
    assert torch.all(out[nd] == 7.0)


@pytest.mark.parametrize("dim,dtype", [(3, torch.float32), (16, torch.float32), (40, torch.float32), (70, torch.float16), (130, torch.float16),
                                       (255, torch.float32), (256, torch.float32), (300, torch.float32), (602, torch.float32)])
def test_a_row_has_the_same_bits_wherever_it_lies(dim, dtype):
    """Rows with the same entries, between rows of other lengths: the order of a row's additions is its own."""
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(dim)
    kinds, nd, ns = 40, 40_001, 500
    lens = rng.integers(0, 24, kinds)
    first = np.concatenate([[0], np.cumsum(lens)])
    cols = rng.integers(kinds, ns, first[-1])
    kind = rng.integers(0, kinds, nd)
    indptr = np.concatenate([[0], np.cumsum(lens[kind])])
    entry = np.repeat(first[kind] - indptr[:-1], lens[kind]) + np.arange(indptr[-1])
    gen = torch.Generator(device="cuda").manual_seed(dim)
    x = torch.randn((ns, dim), generator=gen, device="cuda").to(dtype)
    w = torch.randn(int(first[-1]), generator=gen, device="cuda")
    small = [bare_blocks(mqg, first, cols, kinds, ns), torch.empty((kinds, dim), dtype=dtype, device="cuda"), w]
    large = [bare_blocks(mqg, indptr, cols[entry], nd, ns), torch.empty((nd, dim), dtype=dtype, device="cuda"), w[torch.from_numpy(entry).cuda()]]
    where = torch.from_numpy(kind).cuda()
    for call in ("mean", "weighted"):
        for (ctx, blocks), out, weights in (small, large):
            if call == "mean":
                mqg.mqg_sage_mean_aggregate(ctx, blocks, 0, x, out)
            else:
                mqg.mqg_weighted_aggregate(ctx, blocks, 0, weights, None, x, out)
        assert torch.equal(large[1], small[1][where])
    # ... and whatever length the block's capacities let expect
    (ctx, blocks), out, _ = small
    mqg.mqg_sage_mean_aggregate(ctx, blocks, 0, x, out)
    again = torch.empty_like(out)
    for cap in (kinds, 60 * kinds):
        blocks.c[0].cap_nnz = cap
        mqg.mqg_sage_mean_aggregate(ctx, blocks, 0, x, again)
        assert torch.equal(again, out)
    # the backward: sources that are neighbours of the same destinations, in the same order
    dst = np.repeat(np.arange(ns), rng.integers(1, 5, ns))                   # 500 destinations, 1 to 4 kinds of sources each
    pairs = np.stack([dst, rng.integers(0, kinds, len(dst))], 1)
    pairs = np.unique(pairs, axis=0)
    members = [np.flatnonzero(kind == k) for k in range(kinds)]
    big_cols = np.concatenate([members[k] for _, k in pairs])
    big_ptr = np.concatenate([[0], np.cumsum(np.bincount(pairs[:, 0], weights=[len(members[k]) for _, k in pairs], minlength=ns))]).astype(np.int64)
    small_ptr = np.concatenate([[0], np.cumsum(np.bincount(pairs[:, 0], minlength=ns))])
    ew = torch.rand(len(pairs), generator=gen, device="cuda")
    ew_big = ew[torch.from_numpy(np.repeat(np.arange(len(pairs)), [len(members[k]) for _, k in pairs])).cuda()]
    got = []
    for ptr, c, n_src, weights in ((small_ptr, pairs[:, 1], kinds, ew), (big_ptr, big_cols, nd, ew_big)):
        ctx, blocks = bare_blocks(mqg, ptr, c, ns, n_src)
        gx = torch.empty((n_src, dim), dtype=dtype, device="cuda")
        mqg.mqg_weighted_aggregate_backward(ctx, blocks, 0, weights, None, x, gx)
        got.append(gx)
    assert torch.equal(got[1], got[0][where])


@pytest.mark.parametrize("dim,entries", [(4, 2000), (8, 300), (8, 2000), (16, 300), (16, 2000)])
def test_error_of_long_narrow_rows(dim, entries):
    """Rows of `entries` normal terms in fp32: G = 64 / (dim / 4) partial sums, then log2 G additions and a division.  The
    sum so far of m terms has a variance of m, and an addition is off by at most 2^-24 of it, uniformly at worst (a
    standard deviation of 2^-24 / sqrt(3)): the error is at most that times sqrt(entries / 2G + log2 G + 1) of the
    result.  With four partial sums it was 1.3 to 2.4 times this bound."""
    from paper_2601_04707_amd import mqg
    nd, ns = 1500, 40_000
    gen = torch.Generator(device="cuda").manual_seed(dim + entries)
    cols = torch.randint(0, ns, (nd * entries,), generator=gen, device="cuda")
    ctx, blocks = bare_blocks(mqg, np.arange(nd + 1) * entries, cols.cpu().numpy(), nd, ns)
    x = torch.randn((ns, dim), generator=gen, device="cuda")
    w = torch.randn(nd * entries, generator=gen, device="cuda")
    out = torch.empty((nd, dim), device="cuda")
    groups = 64 // (dim // 4)
    bound = 2.0 ** -24 / 3 ** 0.5 * (entries / (2 * groups) + np.log2(groups) + 1) ** 0.5
    for weights in (None, w):
        terms = x.double()[cols].view(nd, entries, dim)
        if weights is None:
            mqg.mqg_sage_mean_aggregate(ctx, blocks, 0, x, out)
            want = terms.mean(1)
        else:
            mqg.mqg_weighted_aggregate(ctx, blocks, 0, weights, None, x, out)
            want = (terms * weights.double().view(nd, entries, 1)).sum(1)
        error = float((out.double() - want).pow(2).mean().sqrt() / want.pow(2).mean().sqrt())
        assert error <= bound, (error, bound)
