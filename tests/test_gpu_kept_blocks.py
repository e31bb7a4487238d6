"""Device blocks that a context keeps for its next allocations: graphs made in used memory are the same, the memory is bounded by what was
in use, is given back with the context and under a byte budget, and a graph may outlive its context."""
import numpy as np
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


def _graph(V, E, seed):
    src, dst = inputs.rmat_edges(V, E, seed)
    return src.cuda(), dst.cuda()


def _layer(ctx, g, V, d_in, d_out, seed):
    gen = torch.Generator().manual_seed(seed)
    H, W = B.to_matrix(torch.randn(V, d_in, generator=gen)), torch.randn(d_in, d_out, generator=gen).cuda()
    out = B.alloc_matrix(V, d_out)
    B.ht_layer_fwd(ctx, g, d_in, d_out, B.HT_ACT_RELU, H, W, out)
    B.ht_sync(ctx)
    return out[:, :d_out].cpu()


def test_graphs_made_in_used_memory():
    sizes = [(5_003, 60_000, 3), (20_011, 300_007, 4), (4_999, 61_000, 2), (20_000, 299_000, 5), (30_000, 30_000, 1), (5_003, 60_000, 3)]
    def run(keep):
        ctx = B.ht_ctx_create(0)
        outs = []
        for k in range(2):
            for i, (V, E, n) in enumerate(sizes):
                if not keep:
                    B.ht_ctx_destroy(ctx)
                    ctx = B.ht_ctx_create(0)
                g = B.ht_partition(ctx, V, *_graph(V, E, i), n)
                chunks = [B.ht_graph_export_chunk(g, j) for j in range(n)]
                outs.append((_layer(ctx, g, V, 33, 20, i), chunks))
                B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
        return outs
    for (a, ca), (b, cb) in zip(run(True), run(False)):
        assert torch.equal(a, b)
        for x, y in zip(ca, cb):
            assert all(np.array_equal(x[k], y[k]) for k in x)


def test_memory_is_bounded_and_given_back():
    torch.cuda.synchronize()
    ctx = B.ht_ctx_create(0)
    src, dst = _graph(200_000, 3_000_000, 1)
    before, low = torch.cuda.mem_get_info()[0], []
    for _ in range(6):
        g = B.ht_partition(ctx, 200_000, src, dst, 4)
        B.ht_graph_destroy(g)
        low.append(torch.cuda.mem_get_info()[0])
    assert low[-1] == low[1], "the same graph again takes no more"
    assert before - low[-1] < 1 << 30
    B.ht_ctx_set_hbm_budget(ctx, 1 << 40)
    assert torch.cuda.mem_get_info()[0] > low[-1]
    B.ht_ctx_destroy(ctx)
    assert torch.cuda.mem_get_info()[0] >= before


def test_graph_outlives_its_context():
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, 5_003, *_graph(5_003, 60_000, 1), 3)
    _layer(ctx, g, 5_003, 8, 8, 1)
    B.ht_ctx_destroy(ctx)
    others = [B.ht_ctx_create(0) for _ in range(2)]
    B.ht_graph_destroy(g)
    for c in others:
        h = B.ht_partition(c, 5_003, *_graph(5_003, 60_000, 1), 3)
        assert torch.isfinite(_layer(c, h, 5_003, 8, 8, 1)).all()
        B.ht_graph_destroy(h)
        B.ht_ctx_destroy(c)
