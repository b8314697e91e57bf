"""What a context takes of the card's memory: one bitmap and one block's neighbours on graphs of more than 3 M nodes, three
bitmaps and two neighbouring blocks' below, however many layers there are; and blocks at both ends of that room."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_blocks_equal, hip_sample, to_dev

pytestmark = pytest.mark.gpu


def ring(n, degree):
    rp = torch.arange(n + 1) * degree
    return rp, ((torch.arange(n).view(-1, 1) * 5 + 1 + torch.arange(degree) * 11) % n).reshape(-1)


@pytest.mark.parametrize("n,places", [(4_000_000, 1), (3_000_000, 2)])
def test_room_does_not_grow_with_the_layers(n, places):
    from paper_2601_04707_amd import mqg
    rp, ci = ring(n, 1)
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    fanouts = [64] * 5
    _ = mqg.Context(g, 16, [2])                            # the library's own buffers are there
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx = mqg.Context(g, n, fanouts)
    used = before - torch.cuda.mem_get_info()[0]
    bounds = mqg.block_bounds(n, n, fanouts)
    neighbours = places * bounds[0][2] * 4                 # all blocks have the same bound here
    per_node = 4 + 3 / 8 + 8 + 4 + 4 + 2 * 8               # positions, bitmaps, rows' start and degree, hubs, hit and miss lists
    assert neighbours < used < neighbours + per_node * n + (64 << 20), (used, neighbours)
    del ctx


@pytest.mark.parametrize("fanouts", [[7], [3, 9], [9, 3], [2, 11, 1], [1, 2, 12, 1], [4, 1, 3, 1, 5]])
def test_blocks_at_both_ends_of_the_room(fanouts):
    """Neighbouring blocks of any sizes, within the context's bounds and exactly at them."""
    from paper_2601_04707_amd import mqg
    n, batch = 50_000, 61
    rp, ci = ring(n, 13)
    g = mqg.Graph(to_dev(rp), to_dev(ci))
    rng = np.random.default_rng(len(fanouts))
    for room in (fanouts, [f + 5 for f in fanouts]):
        ctx = mqg.Context(g, batch, room)
        blocks = mqg.Blocks(g, batch, room)
        for call, size in enumerate((batch, 7, batch)):
            seeds = rng.choice(n, size, replace=False).astype(np.int64)
            got = hip_sample(mqg, ctx, g, blocks, torch.from_numpy(seeds), fanouts, call)
            assert_blocks_equal(got, oracle.sample_blocks(rp.numpy(), ci.numpy(), seeds, fanouts, call))
