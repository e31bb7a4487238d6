"""grad W out of many slices: tiles of few and of many elements, as many slices as a stage takes and some more, in one group of rows and in several;
and dz written by the product on its way."""
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


@pytest.mark.parametrize("V,K,N", [(1, 3, 5), (17, 33, 7), (3_000, 128, 64), (3_001, 40, 130), (3_002, 129, 64), (70_003, 64, 41), (70_003, 100, 67)])
@pytest.mark.parametrize("n", [1, 5])
def test_dz_written_by_the_product(V, K, N, n):
    """A layer whose grad W masks dz for the other product too: the bits of the call whose dz was masked before, whether the activation is
    given or made again into the memory that dz takes."""
    ctx = B.ht_ctx_create(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, n)
    try:
        gen = torch.Generator(device="cuda").manual_seed(V + K)
        A, dH, H, W = B.alloc_matrix(V, K), B.alloc_matrix(V, N), B.alloc_matrix(V, N), torch.randn(K, N, generator=gen, device="cuda")
        A.normal_(generator=gen)
        dH.normal_(generator=gen)
        A[:, K:], dH[:, N:] = float("nan"), float("inf")
        B.ht_layer_fwd(ctx, g, K, N, B.HT_ACT_RELU, A, W, H)     # (no edges but the self-loops: the aggregate is A)
        B.ht_sync(ctx)
        H[:, N:] = float("nan")
        dz = dH.clone()
        dz[:, :N] *= (H[:, :N] > 0)
        got = []
        for act, grad, h in ((B.HT_ACT_NONE, dz, None), (B.HT_ACT_RELU, dH, H), (B.HT_ACT_RELU, dH, None)):
            dW, dX = torch.full((K, N), 7.0, device="cuda"), B.alloc_matrix(V, K).zero_()
            B.ht_layer_bwd(ctx, g, K, N, act, A, W, grad, dW, dH_in=dX, H_out=h)
            B.ht_sync(ctx)
            got.append((dW, dX[:, :K].clone()))
        for dW, dX in got[1:]:
            assert torch.equal(dW, got[0][0]) and torch.equal(dX, got[0][1])
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("given,first,takes", [(True, True, False), (False, True, True), (True, False, True)])
def test_dz_is_held_where_it_is_used(given, first, takes):
    """A first layer (no input gradient) whose activations are given masks dz inside grad W: no memory for dz of all vertices."""
    V, K, N = 400_000, 20, 256
    ctx = B.ht_ctx_create(0)
    B.ht_ctx_set_hbm_budget(ctx, 1 << 40)      # (nothing is kept of what is given back)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, 1)
    try:
        gen = torch.Generator(device="cuda").manual_seed(1)
        A, dH, H, dX, W, dW = B.alloc_matrix(V, K), B.alloc_matrix(V, N), B.alloc_matrix(V, N), B.alloc_matrix(V, K), torch.zeros(K, N, device="cuda"), torch.empty(K, N, device="cuda")
        A.normal_(generator=gen)
        dH.normal_(generator=gen)
        H.normal_(generator=gen)
        mask = H > 0 if given else torch.zeros_like(H, dtype=torch.bool)       # (W is 0: made again, no activation is positive)
        want, mag = A[:, :K].double().t().contiguous() @ (dH * mask).double(), A[:, :K].double().abs().t().contiguous() @ (dH * mask).double().abs()
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        B.ht_layer_bwd(ctx, g, K, N, B.HT_ACT_RELU, A, W, dH, dW, dH_in=None if first else dX, H_out=H if given else None)
        B.ht_sync(ctx)
        taken = free - torch.cuda.mem_get_info()[0]
        assert (taken >= V * N * 4) == takes, taken
        # (as above)
        assert ((dW.double() - want).abs() <= 64 * 2.0 ** -24 * mag).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
