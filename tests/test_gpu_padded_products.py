"""Products whose widths fill tiles of 32 columns better than blocks of 64 or 128, at the edges of tiles, steps of the reduction, strips of
rows and of what of W fits into a CU's memory, against fp64."""
import ctypes
import threading

import pytest
import torch

from paper_2311_14898_amd import binding as B

pytestmark = pytest.mark.gpu


# (rows that leave a wave for every SIMD only with narrower tiles: one tile of 32 columns at a time up to some 10,000 rows, two or four of five at 12,000 and 20,000, two of three at 20,000)
@pytest.mark.parametrize("V", [1, 33, 3_000, 12_000, 20_000, 40_001])
@pytest.mark.parametrize("K,N", [(1, 1), (31, 32), (33, 8), (64, 65), (67, 129), (129, 96), (301, 160), (300, 161), (96, 257), (416, 66), (424, 66), (1216, 20), (1217, 20)])
def test_layer_without_edges(V, K, N):
    """No edges but the self-loops: the layer is H W forward and dz W^T backward; the widths are taken both ways."""
    if V > 20_000 and K > 500:
        pytest.skip("the rows' rule is tested at the narrower widths")
    ctx = B.ht_ctx_create(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, 1)
    try:
        for di, dn in ((K, N), (N, K)):
            gen = torch.Generator().manual_seed(di)
            H, W, dz = torch.randn(V, di, generator=gen), torch.randn(di, dn, generator=gen), torch.randn(V, dn, generator=gen)
            out, A, dX, dW = B.alloc_matrix(V, dn), B.alloc_matrix(V, di), B.alloc_matrix(V, di), torch.empty(di, dn, device="cuda")
            Hd, dzd = B.to_matrix(H), B.to_matrix(dz)
            for m, cols in ((Hd, di), (dzd, dn), (A, di)):
                m[:, cols:] = float("nan")     # what lies behind a row's last value is nobody's business
            out.fill_(-3.0)
            dX.zero_()
            Wd = torch.cat([torch.full((3,), float("nan")), W.reshape(-1), torch.full((5,), float("nan"))]).cuda()[3:3 + di * dn].view(di, dn)
            B.ht_layer_fwd(ctx, g, di, dn, B.HT_ACT_RELU, Hd, Wd, out, A)
            B.ht_layer_bwd(ctx, g, di, dn, B.HT_ACT_NONE, A, Wd, dzd, dW, dH_in=dX)
            B.ht_sync(ctx)
            assert bool((out[:, dn:] == -3.0).all())
            # n fp32 products and sums: off by at most (n + 4) 2^-24 of the sum of absolute values
            for got, a, b, relu in ((out[:, :dn], H, W, True), (dX[:, :di], dz, W.t(), False)):
                want, mag = a.double() @ b.double(), a.abs().double() @ b.abs().double()
                if relu:
                    want = want.clamp(min=0)
                assert ((got.cpu().double() - want).abs() <= (b.shape[0] + 4) * 2.0 ** -24 * mag).all(), (di, dn)
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("K,N,sizes", [(67, 129, (100, 5_000, 200_000)), (129, 67, (100, 12_000, 20_000, 200_000)), (50, 20, (100, 5_000, 200_000)),
                                       (424, 70, (100, 400_000, 400_001)), (417, 96, (20_000, 400_001))])
def test_rows_do_not_depend_on_their_number(K, N, sizes):
    """The same bits however many rows are multiplied, in tiles of any number of columns and, beyond 400,000 rows of three tiles, in blocks."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    H, W = torch.randn(max(sizes), K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    rows = []
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    for V in sizes:
        ctx = B.ht_ctx_create(0)
        g = B.ht_partition(ctx, V, none, none, 1)
        Hd, out = B.alloc_matrix(V, K), B.alloc_matrix(V, N)
        Hd[:, :K] = H[:V]
        B.ht_layer_fwd(ctx, g, K, N, B.HT_ACT_NONE, Hd, W, out)
        B.ht_sync(ctx)
        rows.append(out[:, :N].clone())
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
    for less, more in zip(rows, rows[1:]):
        assert torch.equal(less, more[:less.shape[0]])


def test_threads_with_unlike_lds():
    """Two threads, each with its context, through one kernel with 68 and 161 KB of LDS: neither is refused its launch, and both get their product."""
    V, N, calls = 64, 96, 3_000
    none, out = torch.empty(0, dtype=torch.int32, device="cuda"), {}

    def run(K):
        try:
            stream = torch.cuda.Stream()
            ctx = B.ht_ctx_create(0, stream.cuda_stream)
            g = B.ht_partition(ctx, V, none, none, 1)
            gen = torch.Generator().manual_seed(K)
            H, W, got = torch.randn(V, K, generator=gen), torch.randn(K, N, generator=gen), B.alloc_matrix(V, N)
            Hd, Wd = B.to_matrix(H), W.cuda()
            torch.cuda.synchronize()
            desc, views = B.ht_layer_desc(K, N, B.HT_ACT_NONE, B.HT_GATHER_AUTO, 0, B.HT_ORDER_AGG_FIRST), (B.tensor_view(Hd, K), B.tensor_view(got, N))
            for _ in range(calls):
                rc = B.load().ht_layer_fwd(ctx, g, ctypes.byref(desc), ctypes.byref(views[0]), ctypes.c_void_p(Wd.data_ptr()), ctypes.byref(views[1]), None, None)
                assert rc == 0, rc
            B.ht_sync(ctx)
            want, mag = H.double() @ W.double(), H.abs().double() @ W.abs().double()
            assert ((got[:, :N].cpu().double() - want).abs() <= (K + 4) * 2.0 ** -24 * mag).all()
            B.ht_graph_destroy(g)
            B.ht_ctx_destroy(ctx)
            out[K] = "done"
        except BaseException as e:      # (a thread's failure is the test's)
            out[K] = repr(e)

    threads = [threading.Thread(target=run, args=(K,)) for K in (416, 176)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert out == {416: "done", 176: "done"}


@pytest.mark.parametrize("K", [1, 7, 17, 50, 67, 130])
@pytest.mark.parametrize("N", [3, 32, 65, 129])
def test_columns_do_not_depend_on_the_width(K, N):
    """The same bits whether a column is among those of a padded width or of one that fills its blocks."""
    V, wide = 5_000, 64 if N <= 32 else 256
    gen = torch.Generator().manual_seed(K)
    H, W = torch.randn(V, K, generator=gen), torch.randn(K, wide, generator=gen)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, none, none, 1)
    try:
        got = []
        for n in (N, wide):
            out = B.alloc_matrix(V, n)
            B.ht_layer_fwd(ctx, g, K, n, B.HT_ACT_NONE, B.to_matrix(H), W[:, :n].contiguous().cuda(), out)
            B.ht_sync(ctx)
            got.append(out[:, :N].cpu())
        assert torch.equal(*got)
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("V", [1, 15, 17, 33, 49, 1_000, 20_011])
@pytest.mark.parametrize("K,N", [(1, 1), (5, 4), (33, 7), (129, 64), (128, 61), (130, 66), (40, 130)])
def test_weight_gradients_by_steps_of_rows(V, K, N):
    """grad W = H^T dz over slices of rows that end anywhere in a step, with anything behind the rows' last values."""
    ctx = B.ht_ctx_create(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, 1)
    try:
        gen = torch.Generator().manual_seed(V)
        A, dz = torch.randn(V, K, generator=gen), torch.randn(V, N, generator=gen)
        Ad, dzd, dW = B.to_matrix(A), B.to_matrix(dz), torch.full((K, N), 7.0, device="cuda")
        Ad[:, K:], dzd[:, N:] = float("nan"), float("inf")
        B.ht_layer_bwd(ctx, g, K, N, B.HT_ACT_NONE, Ad, torch.randn(K, N, generator=gen).cuda(), dzd, dW)
        B.ht_sync(ctx)
        want, mag = A.double().t() @ dz.double(), A.double().abs().t() @ dz.double().abs()
        # V fp32 products and sums: off by at most (V + 4) 2^-24 of the sum of absolute values
        assert ((dW.cpu().double() - want).abs() <= (V + 4) * 2.0 ** -24 * mag).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def _same(a, b):
    return bool(((a == b) | (a.isnan() & b.isnan())).all())


@pytest.mark.parametrize("V,K,N", [(1, 3, 5), (17, 33, 7), (3_000, 129, 64), (3_001, 40, 130), (40_003, 70, 66)])
@pytest.mark.parametrize("odd", [None, "A", "masked", "unmasked", "large"])
def test_masked_weight_gradients(V, K, N, odd):
    """grad W masks dz on the way, alone or for the product behind it too: the bits of the call without an activation whose dz was masked before, also where values are not finite
    or too large to be split into bf16, on either side of the mask (40,003 x 70 x 66 goes through the split product)."""
    ctx = B.ht_ctx_create(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, 3)
    try:
        gen = torch.Generator().manual_seed(V)
        A, dH, H, W = B.to_matrix(torch.randn(V, K, generator=gen)), B.to_matrix(torch.randn(V, N, generator=gen)), torch.randn(V, N, generator=gen), torch.randn(K, N, generator=gen).cuda()
        H[::3] = 0.0
        H[::7] = float("nan")                        # (not positive: the derivative is 0)
        H[V // 2, 0] = 1.0
        Hd = B.to_matrix(H)
        if odd == "A":
            A[V // 2, K // 2], A[0, 0] = float("inf"), 3.4e38
        elif odd == "masked":
            dH[0, 0], dH[0, N - 1], dH[3 % V, 1] = float("inf"), float("nan"), 3.4e38
            if V <= 3:
                Hd[0] = -1.0
        elif odd == "unmasked":
            dH[V // 2, 0] = float("inf")
        elif odd == "large":
            dH[V // 2, 0] = 3.4e38
        Hc = Hd[:, :N].cpu()
        dz = B.to_matrix(torch.where(Hc > 0, dH[:, :N].cpu(), torch.zeros(())))
        A[:, K:], dH[:, N:], Hd[:, N:], dz[:, N:] = float("nan"), float("inf"), float("nan"), float("nan")
        got = []
        for act, grad, h, dX in ((B.HT_ACT_NONE, dz, None, None), (B.HT_ACT_RELU, dH, Hd, None), (B.HT_ACT_RELU, dH, Hd, B.alloc_matrix(V, K).zero_())):
            dW = torch.full((K, N), 7.0, device="cuda")
            B.ht_layer_bwd(ctx, g, K, N, act, A, W, grad, dW, dH_in=dX, H_out=h)
            B.ht_sync(ctx)
            got.append(dW)
        assert _same(got[1], got[0]) and _same(got[2], got[0])
        if odd is None or odd == "masked":
            a, b = A[:, :K].cpu().double(), dz[:, :N].cpu().double()
            assert ((got[0].cpu().double() - a.t() @ b).abs() <= (V + 4) * 2.0 ** -24 * (a.abs().t() @ b.abs())).all()
        else:
            assert not (got[0].abs() < 1e30).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
