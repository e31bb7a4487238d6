"""The dense products that run on the bf16 matrix cores as three-way splits: against fp64 at the edges of their tiles (128 x 128,
32 along the reduction) and of the rule that takes a call to them, with an error no larger than fp32 sums have, and with
infinities and NaN where fp32 products have them."""
import pytest
import torch

from paper_2311_14898_amd import binding as B

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("V,di,dn", [(8192, 32, 65), (8193, 33, 128), (9001, 129, 127), (8320, 256, 129), (8191, 96, 96), (12_345, 65, 66)])
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


def test_split_products_not_finite(ctx):
    V, di, dn = 8500, 70, 100
    gen = torch.Generator().manual_seed(1)
    X, W, dH = torch.randn(V, di, generator=gen), torch.randn(di, dn, generator=gen), torch.randn(V, dn, generator=gen)
    X[200, 69], X[8499, 0], X[400, 7] = 3.4e38, float("nan"), -3.4e38       # (3.4e38 rounds to infinity as bf16)
    W[7], W[69] = W[7] * 1e-3, W[69] * 1e-3                                 # (and its products stay finite)
    dH[130, 99], dH[131, 98] = float("inf"), float("-inf")
    H, dW, dX = _run(ctx, X, W, dH)
    keep = torch.ones(V, dtype=torch.bool)
    keep[[130, 131]] = False                                                # (the aggregation behind dX turns infinities into NaN)
    for got, want in ((H, X @ W), (dW, X.t() @ dH), (dX[keep], (dH @ W.t())[keep])):
        nan, ok = torch.isnan(want), torch.isfinite(want)
        assert torch.equal(torch.isnan(got), nan) and torch.equal(torch.isfinite(got), ok)
        assert torch.equal(got[~ok & ~nan], want[~ok & ~nan])
        assert ((got[ok] - want[ok]).abs() <= 1e-4 * want[ok].abs() + 1e-3).float().mean() > 0.999
