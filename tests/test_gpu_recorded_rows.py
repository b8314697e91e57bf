"""Row information, hub lists and source lists of inner blocks: on graphs of few bitmap tiles the launch that lists a block's new
sources records them for the next block and the next sampling launch relabels, on others a launch of their own does
both.  Node counts on both sides of the lines (tiles of 8,192 nodes: 64 and 384), hubs among the new sources of
every block, and several calls on one context, whose two bitmaps and whose list of hubs have to be empty again."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_blocks_equal, hip_sample, to_dev

pytestmark = pytest.mark.gpu


def graph_with_hubs(n, every=50, hub_degree=90):
    """Rows of 4 slots, the first of which points to one of the hubs, whose rows have 90 slots."""
    ids = np.arange(n, dtype=np.int64)
    deg = np.where(ids % every == 0, hub_degree, 4)
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    row = np.repeat(ids, deg)
    j = np.arange(rp[-1], dtype=np.int64) - rp[row]
    ci = (row + 1 + j * 997) % n                           # distinct: 90 * 997 < n
    to_hub = (j == 0) & (row % every != 0)
    hubs = -(-n // every)
    ci[to_hub] = row[to_hub] * 7919 % hubs * every
    slot = np.nonzero((j > 0) & (ci == np.repeat(ci[rp[:-1]], deg)))[0]        # a neighbour that the first slot now names too
    ci[slot] = (ci[slot] + 3) % n
    return torch.from_numpy(rp), torch.from_numpy(ci)


@pytest.mark.parametrize("n", [100_000, 524_288, 524_289, 3_145_728, 3_145_729])
@pytest.mark.parametrize("heavy_degree", [64, 2048])
def test_inner_blocks_on_both_sides_of_the_lines(n, heavy_degree):
    from paper_2601_04707_amd import mqg
    rp, ci = graph_with_hubs(n)
    fanouts = [3, 5, 4]
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    ctx = mqg.Context(g, 700, fanouts)
    ctx.set_option(mqg.MQG_OPT_HEAVY_DEGREE, heavy_degree)
    blocks = mqg.Blocks(g, 700, fanouts)
    rng = np.random.default_rng(n)
    for call, batch in enumerate((700, 3, 257)):
        seeds = torch.from_numpy(rng.choice(n, batch, replace=False).astype(np.int64))
        got = hip_sample(mqg, ctx, g, blocks, seeds, fanouts, 40 + call)
        assert_blocks_equal(got, oracle.sample_blocks(rp.numpy(), ci.numpy(), seeds.numpy(), fanouts, 40 + call))
