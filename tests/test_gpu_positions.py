"""Positions of nodes in the source lists carry an offset that grows from call to call: what earlier calls left in the
table must not be taken for this call's, across the clearing of the table when the offsets run out, between the two
samplers, and between recorded calls (which use one range again and again) and others on the same context."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_04707_amd import synth
from gpu_util import assert_blocks_equal, hip_sample, to_dev

pytestmark = pytest.mark.gpu


def read_blocks(blocks):
    out = []
    for l, (nd, ns, nnz, flags) in enumerate(blocks.host_sizes()):
        assert flags == 0
        out.append((blocks.src_ids[l][:ns].cpu().numpy(), blocks.indptr[l][:nd + 1].cpu().numpy(), blocks.indices[l][:nnz].cpu().numpy()))
    return out


def assert_same(got, want):
    for (src, indptr, indices), w in zip(got, want):
        assert np.array_equal(src, w.src_ids) and np.array_equal(indptr, w.indptr) and np.array_equal(indices, w.indices)


@pytest.mark.parametrize("max_seeds", [1 << 28, 300])
def test_offsets_run_out_and_recorded_calls(max_seeds):
    """2^28 seeds at most: a call takes 2^28 offsets, and the ninth call finds none left (one range is the recorded calls')."""
    from paper_2601_04707_amd import mqg
    rp, ci = synth.chung_lu_graph(3000, 60_000, max_degree=800, seed=3)
    n, fanouts, batch = rp.numel() - 1, [4], 300
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    ctx = mqg.Context(g, max_seeds, fanouts)
    blocks, recorded = mqg.Blocks(g, batch, fanouts), mqg.Blocks(g, batch, fanouts)
    layers = mqg.LayerwiseBlocks(g, batch, [64])
    rp_np, ci_np = rp.numpy(), ci.numpy()
    batches = synth.seed_batches(n, batch, 9, seed=5)
    seeds_buf, rng_seed = to_dev(batches[0].clone()), torch.tensor([7], dtype=torch.int64, device="cuda")

    def eager(i):
        got = hip_sample(mqg, ctx, g, blocks, batches[i % 9], fanouts, 100 + i)
        assert_blocks_equal(got, oracle.sample_blocks(rp_np, ci_np, batches[i % 9].numpy(), fanouts, 100 + i))

    eager(0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mqg.mqg_sample_blocks_seed_dev(ctx, g, seeds_buf, fanouts, rng_seed, recorded)
    for i in range(1, 12):
        eager(i)
        if i % 3 == 1:
            seeds_buf.copy_(batches[(i + 4) % 9].cuda())
            rng_seed.fill_(1000 + i)
            graph.replay()
            torch.cuda.synchronize()
            assert_same(read_blocks(recorded), oracle.sample_blocks(rp_np, ci_np, batches[(i + 4) % 9].numpy(), fanouts, 1000 + i))
        if i % 3 == 2:                                     # the other sampler, through the same table
            mqg.mqg_sample_layerwise(ctx, g, to_dev(batches[i % 9]), [64], 50 + i, layers)
            torch.cuda.synchronize()
            assert_same(read_blocks(layers), oracle.ladies_blocks(rp_np, ci_np, batches[i % 9].numpy(), [64], 50 + i))


def test_recorded_layerwise_calls():
    """Both layers of a recorded call use the same range of offsets."""
    from paper_2601_04707_amd import mqg
    rp, ci = synth.chung_lu_graph(3000, 60_000, max_degree=800, seed=3)
    n, sizes, batch = rp.numel() - 1, [128, 64], 200
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    ctx = mqg.Context(g, batch, [2, 2])
    ctx.reserve(mqg.MQG_RESERVE_LAYERWISE, 200)
    blocks, eager_blocks = mqg.LayerwiseBlocks(g, batch, sizes), mqg.LayerwiseBlocks(g, batch, sizes)
    batches = synth.seed_batches(n, batch, 4, seed=5)
    seeds_buf = to_dev(batches[0].clone())
    mqg.mqg_sample_layerwise(ctx, g, seeds_buf, sizes, 11, eager_blocks)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mqg.mqg_sample_layerwise(ctx, g, seeds_buf, sizes, 11, blocks)
    for i in range(4):
        seeds_buf.copy_(batches[i].cuda())
        graph.replay()
        torch.cuda.synchronize()
        assert_same(read_blocks(blocks), oracle.ladies_blocks(rp.numpy(), ci.numpy(), batches[i].numpy(), sizes, 11))
        mqg.mqg_sample_layerwise(ctx, g, to_dev(batches[3 - i]), sizes, 20 + i, eager_blocks)
        torch.cuda.synchronize()
        assert_same(read_blocks(eager_blocks), oracle.ladies_blocks(rp.numpy(), ci.numpy(), batches[3 - i].numpy(), sizes, 20 + i))
