"""The innermost block's rows: below 16,384 seeds of a call with several blocks, on graphs of few bitmap tiles, the first sampling launch takes
them from the seeds themselves, finds the hubs among them and marks the seeds in a bitmap of their own; else a launch before does.
Seed counts around a tile, the hubs' workgroups and the line, seeds that are each other's neighbours, hubs, repeated ids and
ids outside the graph, and further calls on the same context, whose seeds' bitmap has to be empty again."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_04707_amd import synth
from gpu_util import assert_blocks_equal, hip_sample, to_dev

pytestmark = pytest.mark.gpu


def rows(n, width):
    """Neighbours close by, so that seeds are neighbours of seeds; every 40th row is a hub of 100 or, every 4,000th, 3,000 slots."""
    ids = np.arange(n, dtype=np.int64)
    deg = np.where(ids % 4000 == 0, min(3000, n // 2), np.where(ids % 40 == 0, 100, width))
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    row = np.repeat(ids, deg)
    return torch.from_numpy(rp), torch.from_numpy((row + 1 + np.arange(rp[-1], dtype=np.int64) - rp[row]) % n)


@pytest.mark.parametrize("n", [30_000, 530_000])
@pytest.mark.parametrize("batch", [0, 1, 255, 256, 257, 2049, 16_383, 16_384])
@pytest.mark.parametrize("cached_first", [False, True])
def test_seeds_that_are_neighbours_of_seeds(n, batch, cached_first):
    from paper_2601_04707_amd import mqg
    rp, ci = rows(n, 9)
    fanouts = [4, 3]
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    ctx = mqg.Context(g, max(batch, 300), fanouts)
    ctx.set_option(mqg.MQG_OPT_HEAVY_DEGREE, 64)
    blocks = mqg.Blocks(g, max(batch, 300), fanouts)
    prio = None
    if cached_first:
        cache = mqg.Cache(g, synth.node_features(n, 4, seed=2).pin_memory(), n // 5)
        mqg.mqg_build_cache(ctx, g, cache)
        ctx.set_sampling_priority(cache)
        torch.cuda.synchronize()
        prio = cache.slot_of.cpu().numpy()
    rng = np.random.default_rng(batch)
    near = rng.permutation(np.arange(39, 39 + batch, dtype=np.int64))          # all of them neighbours of others, hubs among them
    for call, seeds in enumerate((near, rng.choice(n, min(batch, 300), replace=False).astype(np.int64), near)):
        got = hip_sample(mqg, ctx, g, blocks, torch.from_numpy(seeds), fanouts, 7 + call)
        assert_blocks_equal(got, oracle.sample_blocks(rp.numpy(), ci.numpy(), seeds, fanouts, 7 + call, prio_slot_of=prio))


@pytest.mark.parametrize("n", [30_000, 530_000])
def test_repeated_ids_and_ids_outside_the_graph(n):
    """Their rows are kept, an id outside the graph is node 0, and the flags tell; a neighbour's position is that of the last seed of its id."""
    from paper_2601_04707_amd import mqg
    rp, ci = rows(n, 3)
    fanouts = [2, 3]
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    ctx = mqg.Context(g, 300, fanouts)
    blocks = mqg.Blocks(g, 300, fanouts)
    for seeds, flags in (([5, 6, 7, 6, 5], 2), ([5, n + 7, 9], 1), ([8, n, 9, -3], 3)):
        mqg.mqg_sample_blocks(ctx, g, to_dev(torch.tensor(seeds)), fanouts, 5, blocks)
        torch.cuda.synchronize()
        (_, sizes) = blocks.host_sizes()
        assert sizes[3] == flags and blocks.host_sizes()[0][3] == 0
        checked = [s if 0 <= s < n else 0 for s in seeds]
        src = blocks.src_ids[1][:sizes[1]].tolist()
        assert src[:len(seeds)] == checked and src[len(seeds):] == sorted(set(src[len(seeds):]) - set(checked))
        indptr, indices = blocks.indptr[1][:len(seeds) + 1].tolist(), blocks.indices[1][:sizes[2]].tolist()
        for r, v in enumerate(checked):
            if v == 0:
                continue                                   # a hub, of which three are drawn
            mine = indices[indptr[r]:indptr[r + 1]]
            assert [src[i] for i in mine] == ci[rp[v]:rp[v + 1]].tolist()      # rows of three slots: all of them
            assert all(i == max(j for j, s in enumerate(checked) if s == src[i]) for i in mine if src[i] in checked)
    seeds = np.arange(1, 200, dtype=np.int64)
    got = hip_sample(mqg, ctx, g, blocks, torch.from_numpy(seeds), fanouts, 6)
    assert_blocks_equal(got, oracle.sample_blocks(rp.numpy(), ci.numpy(), seeds, fanouts, 6))


def ids_of_rows(src, indptr, indices):
    return [src[indices[indptr[r]:indptr[r + 1]]].tolist() for r in range(len(indptr) - 1)]


@pytest.mark.parametrize("n", [30_000, 530_000])
@pytest.mark.parametrize("cached_first", [False, True])
@pytest.mark.parametrize("recorded", [False, True])
def test_hubs_and_ids_that_are_no_valid_sample_with_priority_and_recorded(n, cached_first, recorded):
    """Hubs among the seeds, in other places and numbers each time, also repeated and beside ids outside the graph, eager and in replays of a
    recorded call, between calls of valid seeds.  A node's row is the same wherever and however often it is a seed."""
    from paper_2601_04707_amd import mqg
    rp, ci = rows(n, 9)
    rp_np, ci_np = rp.numpy(), ci.numpy()
    fanouts, batch = [4, 3], 300
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    ctx = mqg.Context(g, batch, fanouts)
    ctx.set_option(mqg.MQG_OPT_HEAVY_DEGREE, 64)
    blocks = mqg.Blocks(g, batch, fanouts)
    prio = None
    if cached_first:
        cache = mqg.Cache(g, synth.node_features(n, 4, seed=2).pin_memory(), n // 5)
        mqg.mqg_build_cache(ctx, g, cache)
        ctx.set_sampling_priority(cache)
        torch.cuda.synchronize()
        prio = cache.slot_of.cpu().numpy()
    rng = np.random.default_rng(n)
    hubs = np.arange(0, n, 40)
    few = rng.choice(n, batch, replace=False)
    many = rng.permutation(np.concatenate([rng.choice(hubs, 200, replace=False), rng.choice(n, 100) // 40 * 40 + 7]))
    many = many[np.sort(np.unique(many, return_index=True)[1])]
    many = np.concatenate([many, np.setdiff1d(np.arange(9, n, 40), many)[:batch - len(many)]])
    repeated = rng.permutation(np.concatenate([np.repeat(hubs[1:41], 5), np.repeat(np.arange(11, 61), 2)]))
    outside = few.copy()
    outside[[3, 77, 299]] = [n, -1, 2 * n]
    seeds_dev = torch.zeros(batch, dtype=torch.int64, device="cuda")
    seed_dev = torch.zeros(1, dtype=torch.int64, device="cuda")

    def call():
        mqg.mqg_sample_blocks_seed_dev(ctx, g, seeds_dev, fanouts, seed_dev, blocks)

    if recorded:
        seeds_dev.copy_(to_dev(torch.from_numpy(few)))
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call()
        torch.cuda.synchronize()
    for r, seeds in enumerate((many, few, repeated, many, outside, few, repeated, outside, many)):
        assert len(seeds) == batch
        seeds_dev.copy_(to_dev(torch.from_numpy(seeds)))
        seed_dev.fill_(50 + r)
        graph.replay() if recorded else call()
        torch.cuda.synchronize()
        checked = np.where((seeds < 0) | (seeds >= n), 0, seeds)
        flags = (1 if (checked != seeds).any() else 0) | (2 if len(set(checked)) < batch else 0)
        sizes = blocks.host_sizes()
        assert (sizes[1][3], sizes[0][3]) == (flags, 0), r
        want = oracle.sample_blocks(rp_np, ci_np, np.unique(checked), fanouts, 50 + r, prio_slot_of=prio)
        dst = checked
        for l in (1, 0):
            nd, ns, nnz, _ = sizes[l]
            src = blocks.src_ids[l][:ns].cpu().numpy()
            indptr, indices = blocks.indptr[l][:nd + 1].cpu().numpy(), blocks.indices[l][:nnz].cpu().numpy()
            row_of = dict(zip(want[l].src_ids.tolist(), ids_of_rows(want[l].src_ids, want[l].indptr, want[l].indices)))
            assert np.array_equal(src[:nd], dst) and np.array_equal(src[nd:], np.setdiff1d(want[l].src_ids, dst)), (r, l)
            assert ids_of_rows(src, indptr, indices) == [row_of[v] for v in dst.tolist()], (r, l)
            last = {v: i for i, v in enumerate(src.tolist())}
            assert all(last[v] == i for v, i in zip(src[indices].tolist(), indices.tolist())), (r, l)
            dst = src
