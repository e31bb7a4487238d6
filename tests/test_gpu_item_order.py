"""Work items stay in row order where they read few rows, and go into dispatch order beyond it: the same sums either way, to the last bit."""
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,E", [(1, 0), (16_384, 100_000), (16_385, 100_000), (12_000, 2_000_000)])
def test_order_changes_no_bit(V, E, monkeypatch):
    src, dst = inputs.rmat_edges(V, E, 7) if E else (torch.empty(0, dtype=torch.int32),) * 2
    gen = torch.Generator().manual_seed(1)
    X, dH, W = torch.randn(V, 40, generator=gen), torch.randn(V, 24, generator=gen), torch.randn(40, 24, generator=gen).cuda()
    got = []
    for order in ("1", "0"):
        monkeypatch.setenv("HT_ITEM_ORDER", order)
        ctx = B.ht_ctx_create(0)
        g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), 3)
        H, A, dX, dW = B.alloc_matrix(V, 24), B.alloc_matrix(V, 40), B.alloc_matrix(V, 40), torch.empty(40, 24, device="cuda")
        dX.zero_()
        B.ht_layer_fwd(ctx, g, 40, 24, B.HT_ACT_RELU, B.to_matrix(X), W, H, A)
        B.ht_layer_bwd(ctx, g, 40, 24, B.HT_ACT_RELU, A, W, B.to_matrix(dH), dW, dH_in=dX, H_out=H)
        B.ht_sync(ctx)
        got.append([H[:, :24].clone(), A[:, :40].clone(), dX[:, :40].clone(), dW.clone()])
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
    assert all(torch.equal(a, b) for a, b in zip(*got))
