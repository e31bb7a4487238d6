"""grad W out of many slices: tiles of few and of many elements, as many slices as a stage takes and some more, in one group of rows and in several."""
import pytest
import torch

from paper_2311_14898_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,K,N", [(65_536, 20, 24), (65_537, 3, 5), (200_003, 64, 64), (20_003, 520, 64), (60_001, 300, 130), (70_003, 1000, 20)])
@pytest.mark.parametrize("n", [1, 5])
def test_sums_of_slices(V, K, N, n):
    ctx = B.ht_ctx_create(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, n)
    try:
        gen = torch.Generator(device="cuda").manual_seed(V)
        A, dz, dX = B.alloc_matrix(V, K), B.alloc_matrix(V, N), B.alloc_matrix(V, K)
        A.normal_(generator=gen)
        dz.normal_(generator=gen)
        dX.zero_()
        W, got = torch.randn(K, N, generator=gen, device="cuda"), []
        for _ in range(2):
            dW = torch.full((K, N), 7.0, device="cuda")
            B.ht_layer_bwd(ctx, g, K, N, B.HT_ACT_NONE, A, W, dz, dW, dH_in=dX)
            B.ht_sync(ctx)
            got.append(dW)
        assert torch.equal(*got)
        a, b = A[:, :K].double(), dz[:, :N].double()
        want, mag = a.t().contiguous() @ b, a.abs().t().contiguous() @ b.abs()
        # V fp32 products and sums, in random order of size and sign: 64 of the roundings are well above sqrt(V) of them over V terms
        assert ((got[0].double() - want).abs() <= 64 * 2.0 ** -24 * mag).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
