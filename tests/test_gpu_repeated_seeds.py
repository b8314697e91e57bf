"""Seeds that repeat so often that the call's bounds, which count distinct ones, leave no room for all new sources: nothing is
written past them, the last sources are left out, edges to these point at position 0, and the flags say that the sample is
not valid.  A small graph, and one for each way of listing new sources; further calls on the context are as ever."""
import pytest
import torch

pytestmark = pytest.mark.gpu

GUARD = 4096


def expected(rp, ci, dst, most, degree):
    """Rows are taken whole.  (src, indptr, indices, number of sources without the bound)"""
    n = rp.numel() - 1
    pos = torch.full((n,), -1, dtype=torch.int64, device=rp.device)
    pos.scatter_reduce_(0, dst, torch.arange(dst.numel(), device=rp.device), "amax")
    nbr = ci.view(n, degree)[dst].reshape(-1).long()
    marked = torch.zeros(n, dtype=torch.bool, device=rp.device)
    marked[nbr] = True
    new = torch.nonzero(marked & (pos < 0)).view(-1)
    wanted = dst.numel() + new.numel()
    new = new[:most - dst.numel()]
    pos[new] = dst.numel() + torch.arange(new.numel(), device=rp.device)
    indptr = torch.arange(dst.numel() + 1, device=rp.device) * degree
    return torch.cat((dst, new)), indptr, pos[nbr].clamp_(min=0), wanted


# 33.6 M nodes: bitmaps of more than 2^20 words; 3.2 M: rows recorded by launches of their own; 530,000: tiles counted in a launch before
@pytest.mark.parametrize("n,seeds,ids,degree,layers", [(600, 500, 40, 12, 2), (600, 900, 300, 12, 3), (530_000, 540_000, 260_000, 2, 2),
                                                       (3_200_000, 3_210_000, 1_000_000, 2, 2), (33_600_000, 33_610_000, 9_000_000, 2, 1)])
@pytest.mark.parametrize("dedup_hash", [False, True])
def test_more_sources_than_the_bounds_hold(n, seeds, ids, degree, layers, dedup_hash):
    from paper_2601_04707_amd import mqg
    dev = "cuda"
    rp = torch.arange(n + 1, device=dev) * degree
    ci = ((torch.arange(n, device=dev).view(-1, 1) * 3 + 1 + torch.arange(degree, device=dev) * 7) % n).to(torch.int32).reshape(-1)
    g = mqg.Graph(rp, ci)
    fanouts = [degree] * layers
    ctx = mqg.Context(g, seeds, fanouts)
    if dedup_hash:
        ctx.set_option(mqg.MQG_OPT_DEDUP_HASH, 1)
    blocks = mqg.Blocks(g, seeds, fanouts)
    for l, (_, cap_src, _) in enumerate(blocks.bounds):
        blocks.src_ids[l] = torch.empty(cap_src + GUARD, dtype=torch.int32, device=dev)
        blocks.c[l].src_ids = blocks.src_ids[l].data_ptr()
    gen = torch.Generator(device=dev).manual_seed(n + seeds)
    repeated = torch.randint(0, ids, (seeds,), generator=gen, device=dev)
    distinct = torch.randperm(n, generator=gen, device=dev)[:37]
    over = 0
    for call, (ask, flag) in enumerate(((repeated, 2), (distinct, 0), (repeated, 2), (distinct, 0))):
        for t in blocks.src_ids:
            t.fill_(-7)
        mqg.mqg_sample_blocks(ctx, g, ask.to(torch.int32), fanouts, call, blocks)
        torch.cuda.synchronize()
        sizes = blocks.host_sizes()
        need = mqg.block_bounds(n, ask.numel(), fanouts)
        dst = ask
        for l in range(layers - 1, -1, -1):
            most = need[l][1] if l > 0 else blocks.bounds[l][1]
            src, indptr, indices, wanted = expected(rp, ci, dst, most, degree)
            over += wanted > most
            nd, ns, nnz, flags = sizes[l]
            assert (nd, ns, nnz, flags) == (dst.numel(), src.numel(), indices.numel(), flag if l == layers - 1 else 0), (call, l)
            assert torch.equal(blocks.src_ids[l][:ns].long(), src), (call, l)
            assert (blocks.src_ids[l][ns:] == -7).all(), (call, l)
            assert torch.equal(blocks.indptr[l][:nd + 1].long(), indptr), (call, l)
            got = blocks.indices[l][:nnz].long()
            if dedup_hash:                                 # any of a repeated seed's positions
                left_out = indices == 0
                assert ((got >= 0) & (got < ns)).all() and torch.equal(src[got][~left_out], src[indices][~left_out]), (call, l)
            else:
                assert torch.equal(got, indices), (call, l)
            dst = src
    assert over >= 2
