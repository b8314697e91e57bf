"""mqg_gcn_edge_weights gives a row 8, 16, 32 or 64 lanes by the block's capacities: fanouts on both sides of each line, rows
shorter and without neighbours, and blocks of larger capacities than the call needs; against the formula in float64."""
import numpy as np
import pytest
import torch

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fanout", [1, 8, 9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("room", [1, 700])
def test_weights_of_rows_of_every_length(fanout, room):
    from paper_2601_04707_amd import mqg
    n, batch = 2000, 301
    rng = np.random.default_rng(fanout)
    deg = rng.integers(0, 100, n)
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    row = np.repeat(np.arange(n), deg)
    ci = (row + 1 + np.arange(rp[-1]) - rp[row]) % n
    g = mqg.Graph(to_dev(torch.from_numpy(rp)), to_dev(torch.from_numpy(ci)))
    ctx = mqg.Context(g, batch * room if room > 1 else batch, [fanout])
    blocks = mqg.Blocks(g, batch * room if room > 1 else batch, [fanout])
    seeds = to_dev(torch.from_numpy(rng.choice(n, batch, replace=False)))
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
