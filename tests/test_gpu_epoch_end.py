"""Products that read W in place, at the sizes around where they pack it."""
import pytest
import torch

from paper_2311_14898_amd import binding as B

pytestmark = pytest.mark.gpu


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
