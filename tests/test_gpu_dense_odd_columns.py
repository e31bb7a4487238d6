"""Values that the products over dense tiles cannot take (beyond 2^64, or not finite) are added entry by entry beside them: each sum is as exact as any
other, and a pass does not slow down for a few of them."""
import time

import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


def _graph(V, E, seed):
    src, dst = inputs.rmat_edges(V, E, seed)
    loop = torch.arange(V)
    u, v = torch.cat([src.long(), loop]), torch.cat([dst.long(), loop])
    s = torch.bincount(v, minlength=V).double().rsqrt()
    return src, dst, u, v, s[u] * s[v]


@pytest.mark.parametrize("d", [40, 64, 65, 130, 200])
@pytest.mark.parametrize("share", [1, 7, 600])
def test_sums_beside_the_products(d, share, monkeypatch):
    """`share` vertices have one value of about 2^70 each, in one block of 64 features: rows and features without them keep their precision."""
    V = 600
    src, dst, u, v, w = _graph(V, 40 * V, 3)
    gen = torch.Generator().manual_seed(d)
    X = torch.randn(V, d, generator=gen)
    at = torch.randperm(V, generator=gen)[:share]
    X[at, torch.randint(0, d, (1,), generator=gen)] *= 2.0 ** 70
    want, mag = (torch.zeros(V, d, dtype=torch.float64).index_add_(0, v, w[:, None] * Z.double()[u]) for Z in (X, X.abs()))
    monkeypatch.setenv("HT_DENSE_WORK", "1")
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), 2)
    try:
        H, A = B.alloc_matrix(V, d), B.alloc_matrix(V, d)
        base = B.ht_graph_info_get(g).hbm_bytes
        B.ht_layer_fwd(ctx, g, d, d, B.HT_ACT_NONE, B.to_matrix(X), torch.eye(d, device="cuda"), H, A)
        B.ht_sync(ctx)
        assert B.ht_graph_info_get(g).hbm_bytes > base, "the pass was meant to plan"
        # (the bound of the other tests over tiles: the factors' roundings and the few dozen additions on the longest path)
        assert ((A[:, :d].cpu().double() - want).abs() <= 16 * 2.0 ** -24 * mag).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_a_few_do_not_slow_a_pass_down():
    """One value out of range in the heaviest column: nearly every segment of tiles holds that column."""
    V, E, d = 60_000, 20_000_000, 256
    src, dst = inputs.rmat_edges(V, E, 3, device="cuda")
    hub = int(torch.bincount(src, minlength=V).argmax())
    X = B.alloc_matrix(V, d)
    X.normal_()
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src, dst, 2)
    try:
        H, A, W = B.alloc_matrix(V, 8), B.alloc_matrix(V, d), torch.zeros(d, 8, device="cuda")
        base = B.ht_graph_info_get(g).hbm_bytes

        def best():
            times = []
            for _ in range(12):
                torch.cuda.synchronize()
                t = time.perf_counter()
                B.ht_layer_fwd(ctx, g, d, 8, B.HT_ACT_NONE, X, W, H, A)
                B.ht_sync(ctx)
                times.append(time.perf_counter() - t)
            return min(times[2:])

        plain = best()
        assert B.ht_graph_info_get(g).hbm_bytes > base, "the pass was meant to plan"
        X[hub, 5] = 1e25
        # (11 times as long when such segments went entry by entry; the added column is one of thousands)
        assert best() <= 1.5 * plain
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
