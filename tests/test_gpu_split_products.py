"""grad W on the bf16 matrix cores, its operands as three-way splits, and the fp32 products beside it: against fp64 at the edges of
their tiles and of the rule that takes a call to the split kernel, single products as exact as fp32 rounds them (every partial
product counts there), sums no further off than those of the fp32 kernels, and infinities and NaN where fp32 products have them."""
import pytest
import torch

from paper_2311_14898_amd import binding as B

gpu = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.ht_ctx_create(0)
    yield c
    B.ht_ctx_destroy(c)


def _run(ctx, X, W, dH):
    """H = X W, dW = X^T dH, dX = dH W^T through a layer over a graph of self-loops alone, whose aggregation is the identity."""
    V, di, dn = X.shape[0], X.shape[1], W.shape[1]
    own = torch.arange(V, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, own, own, 3, add_self_loops=False)
    Xd, dHd = B.to_matrix(X), B.to_matrix(dH)
    H, dX, dW = B.alloc_matrix(V, dn), B.alloc_matrix(V, di), torch.empty(di, dn, device="cuda")
    A = B.alloc_matrix(V, di)
    B.ht_layer_fwd(ctx, g, di, dn, B.HT_ACT_NONE, Xd, W.cuda(), H, A)
    B.ht_layer_bwd(ctx, g, di, dn, B.HT_ACT_NONE, A, W.cuda(), dHd, dW, dH_in=dX, ckpt_kind=B.HT_CKPT_AGG)
    B.ht_sync(ctx)
    B.ht_graph_destroy(g)
    return H[:, :dn].cpu(), dW.cpu(), dX[:, :di].cpu()


@gpu
@pytest.mark.parametrize("V,di,dn", [(8192, 32, 65), (8193, 33, 128), (9001, 129, 127), (8320, 256, 129), (8191, 96, 96), (12_345, 65, 66),
                                     (32_768, 65, 65), (32_769, 66, 128), (33_001, 129, 127), (32_767, 96, 96), (32_800, 64, 65),
                                     (15_201, 256, 257), (1500, 1000, 700)])
@pytest.mark.parametrize("lo,hi", [(-30, 30), (0, 0)])
def test_split_products_match_fp64(ctx, V, di, dn, lo, hi):
    gen = torch.Generator().manual_seed(V)
    X = torch.randn(V, di, generator=gen) * torch.pow(2.0, torch.randint(lo, hi + 1, (V, 1), generator=gen))     # rows of many sizes
    W = torch.randn(di, dn, generator=gen) / di ** 0.5
    dH = torch.randn(V, dn, generator=gen) / torch.pow(2.0, torch.randint(lo, hi + 1, (V, 1), generator=gen))
    for got, a, b in zip(_run(ctx, X, W, dH), (X, X.t(), dH), (W, dH, W.t())):
        want, size = a.double() @ b.double(), a.double().abs() @ b.double().abs()
        # n fp32 additions and products in any order are off by at most n 2^-24 of the sum of absolute values, typically by
        # sqrt(n) of it; 8 sqrt(n) 2^-24 leaves room for the largest of a million elements
        assert ((got.double() - want).abs() <= 8 * a.shape[1] ** 0.5 * 2.0 ** -24 * size).all()


@gpu
@pytest.mark.parametrize("V", [8500, 33_000])
def test_split_products_not_finite(ctx, V):
    di, dn = 70, 100
    gen = torch.Generator().manual_seed(1)
    X, W, dH = torch.randn(V, di, generator=gen), torch.randn(di, dn, generator=gen), torch.randn(V, dn, generator=gen)
    X[200, 69], X[8499, 0], X[400, 7] = 3.4e38, float("nan"), -3.4e38       # (3.4e38 rounds to infinity as bf16)
    X[300, 5], dH[300, 6] = 2.0 ** 60, 2.0 ** 30                            # (finite in fp32, not in the splits' scale)
    W[7], W[69] = W[7] * 1e-3, W[69] * 1e-3                                 # (and its products stay finite)
    dH[130, 99], dH[131, 98] = float("inf"), float("-inf")
    H, dW, dX = _run(ctx, X, W, dH)
    keep = torch.ones(V, dtype=torch.bool)
    keep[[130, 131]] = False                                                # (the aggregation behind dX turns infinities into NaN)
    for got, a, b in ((H, X, W), (dW, X.t(), dH), (dX[keep], dH[keep], W.t())):
        exact, size = a.double() @ b.double(), a.double().abs() @ b.double().abs()
        want = a @ b                                                        # (fp32: infinities and NaN where its partial sums leave the range)
        nan, ok = torch.isnan(want), torch.isfinite(want)
        assert torch.equal(torch.isnan(got), nan) and torch.equal(torch.isfinite(got), ok)
        assert torch.equal(got[~ok & ~nan], want[~ok & ~nan])
        # the bound of the finite sums above, for every element
        assert ((got.double() - exact).abs()[ok] <= (8 * a.shape[1] ** 0.5 * 2.0 ** -24 * size)[ok]).all()


# One product per output element: an fp32 product is off by at most 2^-24 of it, and so is the split one up to what its smaller
# partial sums round (seven times 2^-24 of 2^-8) and x2 y2 (2^-33): together below 2^-29.
SINGLE = 2.0 ** -24 * (1 + 2.0 ** -5)


def _mantissas(shape, gen):
    """In [1, 2), a quarter of them near 1 + 2^-8 - 2^-17, where the second and third parts of the split are largest."""
    m = 1 + torch.randint(0, 1 << 23, shape, generator=gen).double() / (1 << 23)
    near = 1 + 2.0 ** -8 - 2.0 ** -17 + torch.randint(-32, 33, shape, generator=gen).double() / (1 << 23)
    return torch.where(torch.rand(shape, generator=gen) < 0.25, near, m).float()


def test_single_products_show_every_partial_product():
    """The kernels' arithmetic on the CPU: with all eight partial products the bound holds, without any one of them it does not."""
    gen = torch.Generator().manual_seed(2)
    x, y = _mantissas((200_000,), gen), _mantissas((200_000,), gen)

    def parts(v):
        p0 = v.bfloat16().float()
        p1 = (v - p0).bfloat16().float()
        return p0, p1, (v - p0 - p1).bfloat16().float()
    a, b = parts(x), parts(y)
    order = [(2, 1), (1, 2), (2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]

    def error(pairs):
        s = torch.zeros_like(x)
        for i, j in pairs:
            s = s + a[i] * b[j]
        return float(((s.double() - x.double() * y.double()) / (x.double() * y.double())).abs().max())
    assert error(order) <= SINGLE
    for drop in order:
        assert error([p for p in order if p != drop]) > SINGLE * 1.2, drop


@gpu
@pytest.mark.parametrize("lo,hi", [(-40, 40), (-126, -100), (-126, -126), (90, 100)])
def test_split_single_products(ctx, lo, hi):
    V, di, dn = 33_000, 160, 144
    gen = torch.Generator().manual_seed(hi)
    def scale(shape):
        return torch.ldexp(torch.ones(shape), torch.randint(lo, hi + 1, shape, generator=gen).float())
    r = torch.arange(V)
    X, dH, W = torch.zeros(V, di), torch.zeros(V, dn), _mantissas((di, dn), gen)
    X[r, r % di] = _mantissas((V,), gen) * scale((V,))
    dH[r, r % dn] = _mantissas((V,), gen) * scale((V,))
    H, _, dX = _run(ctx, X, W, dH)
    for got, want in ((H, X[r, r % di].double()[:, None] * W.double()[r % di]), (dX, dH[r, r % dn].double()[:, None] * W.double().t()[r % dn])):
        assert ((got.double() - want).abs() <= SINGLE * want.abs()).all()
    X[di:] = 0
    dH = torch.zeros(V, dn)
    dH[:di] = _mantissas((di, dn), gen)
    _, dW, _ = _run(ctx, X, W, dH)
    want = X[r[:di], r[:di]].double()[:, None] * dH[:di].double()
    assert ((dW.double() - want).abs() <= SINGLE * want.abs()).all()


@gpu
@pytest.mark.parametrize("V,di,dn,masked,fp32", [(60_013, 256, 128, False, 4.0e-7), (60_013, 256, 128, True, 3.4e-7),
                                                 (116_483, 301, 129, False, 5.2e-7), (200_000, 602, 256, True, 5.7e-7)])
def test_split_sums_are_no_further_off_than_fp32_sums(ctx, V, di, dn, masked, fp32):
    """2-norm error of grad W for N(0, 1) operands, half of X masked by a ReLU; fp32: what the fp32 kernel showed at these sizes."""
    X, dH = torch.randn(V, di, device="cuda"), torch.randn(V, dn, device="cuda")
    X = X.relu() if masked else X
    _, dW, _ = _run(ctx, X, torch.ones(di, dn), dH)
    want = X.double().t().contiguous() @ dH.double()
    err = float((dW.cuda().double() - want).norm() / want.norm())
    assert err <= fp32, (err, fp32)
