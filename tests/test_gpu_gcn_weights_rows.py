"""mqg_gcn_edge_weights gives a row 8, 16, 32 or 64 lanes by the block's capacities: fanouts on both sides of each line, rows
shorter and without neighbours, blocks of larger capacities than the call needs, and blocks with room for more rows than edges, whose
rows take their lanes several rounds; against the formula in float64."""
import numpy as np
import pytest
import torch

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


N, BATCH = 2000, 301


def graph(mqg, rng, deg):
    rp = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    row = np.repeat(np.arange(N), deg)
    ci = (row + 1 + np.arange(rp[-1]) - rp[row]) % N
    return mqg.Graph(to_dev(torch.from_numpy(rp)), to_dev(torch.from_numpy(ci)))


@pytest.mark.parametrize("fanout", [1, 8, 9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("room", [1, 700])
def test_weights_of_rows_of_every_length(fanout, room):
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(fanout)
    deg = rng.integers(0, 100, N)
    g = graph(mqg, rng, deg)
    check(mqg, rng, g, deg, fanout, mqg.Context(g, BATCH * room, [fanout]), mqg.Blocks(g, BATCH * room, [fanout]))


@pytest.mark.parametrize("lanes", [8, 16, 32, 64])
def test_rows_of_several_rounds(lanes):
    """Rows of 0 to 64 edges, on both sides of the lanes' multiples."""
    from paper_2601_04707_amd import mqg
    rng = np.random.default_rng(lanes)
    lengths = [0, 1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 90]
    deg = rng.permutation(np.resize(lengths, N))
    g = graph(mqg, rng, deg)
    blocks = mqg.Blocks(g, BATCH * 64 // lanes, [64])
    blocks.c[0].cap_nnz = BATCH * 64                       # all that the call needs, of a buffer of lanes times as much
    assert blocks.c[0].cap_nnz // blocks.c[0].cap_dst == lanes
    count = check(mqg, rng, g, deg, 64, mqg.Context(g, BATCH, [64]), blocks)
    assert set(lengths[:-1]) == set(count.tolist())


def check(mqg, rng, g, deg, fanout, ctx, blocks):
    seeds = to_dev(torch.from_numpy(rng.choice(N, BATCH, replace=False)))
    mqg.mqg_sample_blocks(ctx, g, seeds, [fanout], 3, blocks)
    edge_w = torch.full((blocks.indices[0].numel(),), -1.0, device="cuda")
    self_w = torch.full((blocks.indptr[0].numel(),), -1.0, device="cuda")
    mqg.mqg_gcn_edge_weights(ctx, g, blocks, 0, edge_w, self_w)
    torch.cuda.synchronize()
    nd, ns, nnz, _ = blocks.host_sizes()[0]
    src, indptr = blocks.src_ids[0][:ns].cpu().numpy(), blocks.indptr[0][:nd + 1].cpu().numpy()
    to = src[blocks.indices[0][:nnz].cpu().numpy()]
    d, count = deg[src[:nd]].astype(np.float64), np.diff(indptr)
    per_edge = np.repeat(np.arange(nd), count)
    want = d[per_edge] / count[per_edge] / np.sqrt((d[per_edge] + 1) * (deg[to] + 1.0))
    # float32 rounding of a value that float64 gives to a few units in 2^-53
    np.testing.assert_allclose(edge_w[:nnz].cpu().numpy(), want, rtol=2.0 ** -24 * 1.01, atol=0)
    np.testing.assert_allclose(self_w[:nd].cpu().numpy(), 1 / (d + 1), rtol=2.0 ** -24 * 1.01, atol=0)
    assert (edge_w[nnz:] == -1).all() and (self_w[nd:] == -1).all()
    return count
