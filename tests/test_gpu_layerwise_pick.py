"""Layer-wise sampling around the line between its two ways of picking a layer's nodes, with a crowded bin of keys at the
threshold, with more rows than fill a launch's own sums, and with hubs in several chunks."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_04707_amd import synth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


def check(mqg, rp, ci, seeds, sizes, seed, method=0, candidates=0):
    """Drawn nodes and edges as the oracle has them; weights: computed in double on both sides, rounded once."""
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    ctx = mqg.Context(g, len(seeds), [2] * len(sizes))
    ctx.set_option(mqg.MQG_OPT_LAYERWISE_CANDIDATES, candidates)
    blocks = mqg.LayerwiseBlocks(g, len(seeds), sizes)
    flags = dict(fastgcn=bool(method & mqg.MQG_LAYERWISE_FASTGCN), debias=bool(method & mqg.MQG_LAYERWISE_DEBIAS), flat=bool(method & mqg.MQG_LAYERWISE_FLAT))
    want = oracle.ladies_blocks(rp.numpy(), ci.numpy(), seeds, sizes, seed, **flags)
    for _ in range(2):                                     # the second call finds what the first one left
        mqg.mqg_sample_layerwise(ctx, g, to_dev(torch.from_numpy(seeds).to(g.idx_dtype)), sizes, seed, blocks, method=method)
        torch.cuda.synchronize()
        for l, (nd, ns, nnz, fl) in enumerate(blocks.host_sizes()):
            w = want[l]
            assert (nd, ns, nnz, fl) == (w.num_dst, w.num_src, w.nnz, 0), l
            assert np.array_equal(blocks.src_ids[l][:ns].cpu().numpy(), w.src_ids), l
            assert np.array_equal(blocks.indptr[l][:nd + 1].cpu().numpy(), w.indptr), l
            assert np.array_equal(blocks.indices[l][:nnz].cpu().numpy(), w.indices), l
            assert np.allclose(blocks.edge_w[l][:nnz].cpu().numpy(), w.edge_w, rtol=1e-6, atol=0), l
    return want


@pytest.mark.parametrize("sizes", [[1, 2], [255, 257], [2047, 2048], [2049, 64], [5000, 2048]])
@pytest.mark.parametrize("candidates", [0, 1, 2, 3])
def test_layer_sizes_around_the_line(sizes, candidates):
    from paper_2601_04707_amd import mqg
    rp, ci = synth.chung_lu_graph(20000, 300_000, max_degree=6000, seed=2)      # hubs of many chunks
    rng = np.random.default_rng(1)
    seeds = rng.permutation(20000)[:150].astype(np.int64)
    method = [0, mqg.MQG_LAYERWISE_FLAT, mqg.MQG_LAYERWISE_DEBIAS, mqg.MQG_LAYERWISE_FASTGCN][(sizes[0] + candidates) % 4]
    check(mqg, rp, ci, seeds, sizes, 31 + candidates, method, candidates)


@pytest.mark.parametrize("size", [1, 700, 1000, 1500])
def test_crowded_bin(size):
    """Degrees chosen so that the race keys of 3,000 nodes lie within a few per cent: more of them in the threshold's bin
    than are compared with one another."""
    from paper_2601_04707_amd import mqg
    n, seed = 3001, 77
    ctx0 = mqg.Context(mqg.Graph(torch.zeros(2, dtype=torch.int64, device="cuda"), torch.zeros(0, dtype=torch.int64, device="cuda")), 1, [1])
    ticket = mqg.mqg_exp_tickets(ctx0, seed, 64, 0, n).cpu().numpy().astype(np.float64)
    deg = np.clip(np.round(3e11 / ticket), 2, n - 1).astype(np.int64) - 1
    deg[0] = n - 1                                         # the seed: its row holds every other node, once
    key = ticket[1:] * (deg[1:] + 1)
    near = np.abs(key / 3e11 - 1) < 0.03
    assert near.sum() > 2000
    row_ptr = np.concatenate([[0], np.cumsum(deg)])
    col = np.arange(row_ptr[-1]) - np.repeat(row_ptr[:-1], deg)
    col += col >= np.repeat(np.arange(n), deg)             # no self loops
    check(mqg, torch.from_numpy(row_ptr), torch.from_numpy(col), np.array([0], dtype=np.int64), [size], seed)


@pytest.mark.parametrize("num_seeds,sizes", [(8191, [100]), (8193, [300]), (20, [40, 9000]), (100, [12000, 64])])
def test_many_rows(num_seeds, sizes):
    from paper_2601_04707_amd import mqg
    rp, ci = synth.chung_lu_graph(20000, 200_000, max_degree=900, seed=4)
    seeds = np.random.default_rng(3).permutation(20000)[:num_seeds].astype(np.int64)
    check(mqg, rp, ci, seeds, sizes, 5)


@pytest.mark.parametrize("n", [262_144, 262_145])
@pytest.mark.parametrize("candidates", [0, 2, 3])
def test_large_layers_around_32_tiles(n, candidates):
    """Up to 32 tiles of the node bitmap several workgroups share a tile's drawn nodes, and the bitmap is cleared by a later launch;
    the node-wise sampler finds it clear."""
    from paper_2601_04707_amd import mqg
    rp, ci = synth.chung_lu_graph(n, 1_200_000, max_degree=2000, seed=6)
    seeds = np.random.default_rng(4).permutation(n)[:1200].astype(np.int64)
    sizes = [3000, 2500]
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    dev_seeds = to_dev(torch.from_numpy(seeds).to(g.idx_dtype))
    ctx, fresh = mqg.Context(g, len(seeds), [5, 5]), mqg.Context(g, len(seeds), [5, 5])
    ctx.set_option(mqg.MQG_OPT_LAYERWISE_CANDIDATES, candidates)
    out = mqg.LayerwiseBlocks(g, len(seeds), sizes)
    want = oracle.ladies_blocks(rp.numpy(), ci.numpy(), seeds, sizes, 9, fastgcn=False, debias=False, flat=False)
    got, ref = mqg.Blocks(g, len(seeds), [5, 5]), mqg.Blocks(g, len(seeds), [5, 5])
    for _ in range(2):
        mqg.mqg_sample_layerwise(ctx, g, dev_seeds, sizes, 9, out)
        for l, (nd, ns, nnz, flags) in enumerate(out.host_sizes()):
            assert (nd, ns, nnz, flags) == (want[l].num_dst, want[l].num_src, want[l].nnz, 0), l
            assert np.array_equal(out.src_ids[l][:ns].cpu().numpy(), want[l].src_ids), l
            assert np.array_equal(out.indices[l][:nnz].cpu().numpy(), want[l].indices), l
            assert np.allclose(out.edge_w[l][:nnz].cpu().numpy(), want[l].edge_w, rtol=1e-6, atol=0), l
        for c, b in ((ctx, got), (fresh, ref)):
            mqg.mqg_sample_blocks(c, g, dev_seeds, [5, 5], 3, b)
        assert got.host_sizes() == ref.host_sizes()
        for l, (nd, ns, nnz, _) in enumerate(ref.host_sizes()):
            assert torch.equal(got.src_ids[l][:ns], ref.src_ids[l][:ns]) and torch.equal(got.indices[l][:nnz], ref.indices[l][:nnz])
