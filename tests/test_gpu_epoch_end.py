"""The last launch of an epoch (sums of the products' slices, update, loss) against the same steps made one by one, and products that read W
in place at the sizes around where they pack it."""
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,E,dims,n,order", [
    (3_001, 30_000, [33, 17, 5], 3, B.HT_ORDER_AGG_FIRST),
    (3_001, 30_000, [64, 32, 8], 2, B.HT_ORDER_UPDATE_FIRST),
    (70_003, 300_000, [40, 65, 12], 5, B.HT_ORDER_AGG_FIRST),      # several row groups
    (500, 3_000, [5], 1, None),
])
def test_update_and_loss(V, E, dims, n, order):
    if order is None:
        dims, order = [5, 3], B.HT_ORDER_AGG_FIRST
    src, dst = inputs.rmat_edges(V, E, 5)
    gen = torch.Generator().manual_seed(1)
    X, y = B.to_matrix(torch.randn(V, dims[0], generator=gen)), torch.randint(0, dims[-1], (V,), generator=gen).to(torch.int32)
    y[torch.rand(V, generator=gen) < 0.3] = -1
    W0 = inputs.glorot_weights(dims, seed=4)
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), n)
    try:
        lr = 0.37
        for _ in range(2):
            W = [w.clone().cuda() for w in W0]
            loss, _ = B.ht_epoch(ctx, g, dims, W, lr, X, y.cuda(), order=order)
            for l, w in enumerate(W):
                dW = B.ht_epoch_buffer(ctx, B.HT_BUF_DW, l).cpu()
                assert float(dW.abs().sum()) > 0
                step = torch.tensor(lr, dtype=torch.float32).double() * dW.double()
                want = W0[l].double() - step
                # at most one rounding of the product (none where it is fused) and one of the difference
                assert ((w.cpu().double() - want).abs() <= 1.01 * 2.0 ** -24 * (step.abs() + want.abs())).all()
            L = len(W)
            logits = B.ht_epoch_buffer(ctx, B.HT_BUF_H, L).cpu().double()
            want = torch.nn.functional.cross_entropy(logits, y.long().clamp(min=0), reduction="none")[y >= 0].mean()
            assert abs(loss - float(want)) <= 1e-6 * abs(float(want))
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_weights_that_share_memory():
    """Two layers with one weight matrix: both updates reach it, one after the other."""
    V, d = 2_000, 24
    src, dst = inputs.rmat_edges(V, 20_000, 5)
    gen = torch.Generator().manual_seed(1)
    X, y = B.to_matrix(torch.randn(V, d, generator=gen)), torch.randint(0, d, (V,), generator=gen).to(torch.int32).cuda()
    w0 = inputs.glorot_weights([d, d], seed=4)[0]
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), 2)
    try:
        w = w0.clone().cuda()
        B.ht_epoch(ctx, g, [d, d, d], [w, w], 0.5, X, y)
        dW = [B.ht_epoch_buffer(ctx, B.HT_BUF_DW, l).cpu() for l in (0, 1)]
        want = w0 - 0.5 * dW[0] - 0.5 * dW[1]
        assert ((w.cpu() - want).abs() <= 1e-6 * want.abs() + 1e-9).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("V", [1, 127, 129, 32_768, 32_769])
@pytest.mark.parametrize("K,N", [(1, 1), (15, 63), (16, 64), (17, 65), (33, 130), (130, 7)])
def test_products_with_w_in_place(V, K, N):
    """No edges but the self-loops: the layer is H W forward and dz W^T backward."""
    gen = torch.Generator().manual_seed(K + N)
    H, W, dz = torch.randn(V, K, generator=gen), torch.randn(K, N, generator=gen), torch.randn(V, N, generator=gen)
    ctx = B.ht_ctx_create(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, 1)
    try:
        out, A, dX, dW = B.alloc_matrix(V, N), B.alloc_matrix(V, K), B.alloc_matrix(V, K), torch.empty(K, N, device="cuda")
        Wd = torch.cat([torch.full((3,), float("nan")), W.reshape(-1), torch.full((5,), float("nan"))]).cuda()[3:3 + K * N].view(K, N)
        dX.zero_()
        B.ht_layer_fwd(ctx, g, K, N, B.HT_ACT_NONE, B.to_matrix(H), Wd, out, A)
        B.ht_layer_bwd(ctx, g, K, N, B.HT_ACT_NONE, A, Wd, B.to_matrix(dz), dW, dH_in=dX)
        B.ht_sync(ctx)
        # n fp32 products and sums: off by at most (n + 2) 2^-24 of the sum of absolute values
        for got, a, b in ((out[:, :N], H, W), (dX[:, :K], dz, W.t())):
            want, mag = a.double() @ b.double(), a.abs().double() @ b.abs().double()
            assert ((got.cpu().double() - want).abs() <= (b.shape[0] + 4) * 2.0 ** -24 * mag).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
