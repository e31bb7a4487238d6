"""Making a graph's plan: both directions share the order of the vertices, whichever is made first and whichever way the sources' entries were
counted, and a pass whose tiles cannot hold enough takes none."""
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


def _passes(V, src, dst, d, order, chunks=3, d_first=None):
    """(aggregate, backward aggregate, bytes that the plans hold), the passes made in that order."""
    gen = torch.Generator().manual_seed(d)
    X, dz = B.to_matrix(torch.randn(V, d, generator=gen)), B.to_matrix(torch.randn(V, d, generator=gen))
    I = torch.eye(d, device="cuda")
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), chunks)
    try:
        H, A, dX, dW = B.alloc_matrix(V, d), B.alloc_matrix(V, d), B.alloc_matrix(V, d), torch.empty(d, d, device="cuda")
        held = [B.ht_graph_info_get(g).hbm_bytes]
        for what in order:
            if what == "fwd":
                B.ht_layer_fwd(ctx, g, d, d, B.HT_ACT_NONE, X, I, H, A)
            else:
                dX.zero_()
                B.ht_layer_bwd(ctx, g, d, d, B.HT_ACT_NONE, A, I, dz, dW, dH_in=dX)
            B.ht_sync(ctx)
            held.append(B.ht_graph_info_get(g).hbm_bytes)
        return A[:, :d].cpu(), dX[:, :d].cpu(), held
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("merge", ["1", "0"])
@pytest.mark.parametrize("V,E", [(300, 60_000), (3_001, 200_000), (40_000, 900_000)])
def test_either_direction_first(V, E, merge, monkeypatch):
    monkeypatch.setenv("HT_DENSE_WORK", "1")
    monkeypatch.setenv("HT_MERGE_DUPS", merge)
    src, dst = inputs.rmat_edges(V // 2, E, 5)      # (half of the vertices have their self-loop alone)
    A, dX, held = _passes(V, src, dst, 24, ["fwd", "bwd"])
    A2, dX2, held2 = _passes(V, src, dst, 24, ["bwd", "fwd"])
    assert torch.equal(A, A2) and torch.equal(dX, dX2)
    assert held[1] > held[0] and held[2] > held[1]
    assert held[2] == held2[2], "what the two directions share goes with the second"
    loop = torch.arange(V)
    u, v = torch.cat([src.long(), loop]), torch.cat([dst.long(), loop])
    s = torch.bincount(v, minlength=V).double().rsqrt()
    X = torch.randn(V, 24, generator=torch.Generator().manual_seed(24))
    w = (s[u] * s[v])[:, None]
    want, mag = (torch.zeros(V, 24, dtype=torch.float64).index_add_(0, v, w * Z.double()[u]) for Z in (X, X.abs()))
    assert ((A.double() - want).abs() <= 16 * 2.0 ** -24 * mag).all()


def test_no_tiles_where_they_cannot_hold_enough(monkeypatch):
    """Uniform edges: tiles of 1 % at most.  With the bound at a tenth of all entries x columns nothing is made."""
    V, E, d = 20_000, 400_000, 32
    gen = torch.Generator().manual_seed(1)
    src, dst = (torch.randint(0, V, (E,), generator=gen).to(torch.int32) for _ in range(2))
    monkeypatch.setenv("HT_DENSE_WORK", str(E * d // 10))
    monkeypatch.setenv("HT_FINE", "0")
    _, _, held = _passes(V, src, dst, d, ["fwd", "fwd"])
    assert held[1] == held[0] and held[2] == held[0]
    monkeypatch.setenv("HT_DENSE_WORK", str(E * d // 10))
    src, dst = inputs.rmat_edges(V, E, 5)           # the same sizes, a third of the entries in tiles
    _, _, held = _passes(V, src, dst, d, ["fwd", "fwd"])
    assert held[1] > held[0] and held[2] == held[1]
