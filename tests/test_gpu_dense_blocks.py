"""The products over dense tiles in blocks of 128 features (what tiles leave behind the last 128 in blocks of 64) and in blocks of 64 alone,
with values that the products take and with some that they do not; and what tiles leave, in the longer and the shorter work items."""
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


def _forward(V, d, src, dst, X):
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), 2)
    try:
        H, A = B.alloc_matrix(V, d), B.alloc_matrix(V, d)
        base = B.ht_graph_info_get(g).hbm_bytes
        B.ht_layer_fwd(ctx, g, d, d, B.HT_ACT_NONE, B.to_matrix(X), torch.eye(d, device="cuda"), H, A)
        B.ht_sync(ctx)
        assert B.ht_graph_info_get(g).hbm_bytes > base, "the pass was meant to plan"
        return A[:, :d].cpu()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def _check(V, d, src, dst, X):
    loop = torch.arange(V)
    u, v = torch.cat([src.long(), loop]), torch.cat([dst.long(), loop])
    s = torch.bincount(v, minlength=V).double().rsqrt()
    w = (s[u] * s[v])[:, None]
    want, mag = (torch.zeros(V, d, dtype=torch.float64).index_add_(0, v, w * Z.double()[u]) for Z in (X, X.abs()))
    # (the bound of the other tests over tiles: the factors' roundings and the few dozen additions on the longest path)
    assert ((_forward(V, d, src, dst, X).double() - want).abs() <= 16 * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("wide", ["1", str(1 << 40)])
@pytest.mark.parametrize("d", [3, 64, 65, 128, 129, 192, 193, 256, 300])
@pytest.mark.parametrize("odd", [0, 9])
def test_block_widths(monkeypatch, wide, d, odd):
    V = 700
    src, dst = inputs.rmat_edges(V, 60 * V, 3)
    gen = torch.Generator().manual_seed(d)
    X = torch.randn(V, d, generator=gen)
    at = torch.randperm(V, generator=gen)[:odd]
    X[at, torch.randint(0, d, (odd,), generator=gen)] *= 2.0 ** 70
    monkeypatch.setenv("HT_DENSE_WORK", "1")
    monkeypatch.setenv("HT_DENSE_WIDE", wide)
    _check(V, d, src, dst, X)


@pytest.mark.parametrize("others", [1, 47, 49, 50, 51, 130])
def test_items_of_what_tiles_leave(monkeypatch, others):
    """1,024 vertices with 400 edges each among themselves (tiles), the others with `others` edges from anywhere: the rows of the others
    are left, on either side of the line between the two lengths of items."""
    V, hubs, d = 20_000, 1024, 36
    gen = torch.Generator().manual_seed(others)
    dst = torch.cat([torch.arange(hubs).repeat_interleave(400), torch.arange(hubs, V).repeat_interleave(others)])
    src = torch.cat([torch.randint(0, hubs, (hubs * 400,), generator=gen), torch.randint(0, V, ((V - hubs) * others,), generator=gen)])
    monkeypatch.setenv("HT_DENSE_WORK", "1")
    _check(V, d, src.to(torch.int32), dst.to(torch.int32), torch.randn(V, d, generator=gen))
