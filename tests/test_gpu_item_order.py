"""Work items in row order and in dispatch order: the same sums either way, to the last bit, and dispatch order is what every graph gets, however small."""
import statistics

import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


# one item; few items over few rows; enough of them that the sort is the one for long inputs (262,144 keys); more rows
@pytest.mark.parametrize("V,E,seg", [(1, 0, 256), (16_384, 100_000, 256), (16_385, 100_000, 256), (12_000, 20_000_000, 64), (300_001, 600_000, 256)])
def test_order_changes_no_bit(V, E, seg, monkeypatch):
    src, dst = inputs.rmat_edges(V, E, 7, device="cuda") if E else (torch.empty(0, dtype=torch.int32, device="cuda"),) * 2
    gen = torch.Generator().manual_seed(1)
    X, dH, W = torch.randn(V, 40, generator=gen), torch.randn(V, 24, generator=gen), torch.randn(40, 24, generator=gen).cuda()
    monkeypatch.setenv("HT_SEG_FWD", str(seg))
    monkeypatch.setenv("HT_SEG_BWD", str(seg))
    monkeypatch.setenv("HT_MERGE_DUPS", "0")
    if E > 262_144 * seg:
        assert (E + V) // seg > 262_144
    got = []
    for order in ("1", "0"):
        monkeypatch.setenv("HT_ITEM_ORDER", order)
        ctx = B.ht_ctx_create(0)
        g = B.ht_partition(ctx, V, src, dst, 3)
        H, A, dX, dW = B.alloc_matrix(V, 24), B.alloc_matrix(V, 40), B.alloc_matrix(V, 40), torch.empty(40, 24, device="cuda")
        dX.zero_()
        B.ht_layer_fwd(ctx, g, 40, 24, B.HT_ACT_RELU, B.to_matrix(X), W, H, A)
        B.ht_layer_bwd(ctx, g, 40, 24, B.HT_ACT_RELU, A, W, B.to_matrix(dH), dW, dH_in=dX, H_out=H)
        B.ht_sync(ctx)
        got.append([H[:, :24].clone(), A[:, :40].clone(), dX[:, :40].clone(), dW.clone()])
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("V,deg,d", [(8_000, 40, 256), (8_000, 10, 128)])
def test_small_graphs_are_ordered(V, deg, d, monkeypatch):
    """Small graphs whose rows' lengths follow their numbers: an aggregation takes 0.73 and 0.81 of its time in row order, more than 0.9 of it where the order is left as it is."""
    src, dst = inputs.rmat_edges(V, V * deg, 3, device="cuda")
    stream = torch.cuda.Stream()
    ctx, graphs, times = B.ht_ctx_create(0, stream.cuda_stream), [], [[], []]
    try:
        for order in ("1", "0"):
            monkeypatch.setenv("HT_ITEM_ORDER", order)
            graphs.append(B.ht_partition(ctx, V, src, dst, 3))
        X, A, H, W = B.alloc_matrix(V, d).normal_(), B.alloc_matrix(V, d), B.alloc_matrix(V, 16), torch.randn(d, 16, device="cuda")
        torch.cuda.synchronize()
        for _ in range(9):
            for g, t in zip(graphs, times):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                with torch.cuda.stream(stream):
                    a.record()
                    for _ in range(20):
                        B.ht_layer_fwd_static(ctx, g, d, 16, B.HT_ACT_NONE, X, W, H, A)
                    b.record()
                b.synchronize()
                t.append(a.elapsed_time(b))
        assert statistics.median(times[0]) < 0.9 * statistics.median(times[1]), [statistics.median(t) for t in times]
    finally:
        for g in graphs:
            B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
