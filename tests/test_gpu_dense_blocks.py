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


HUBS = 1024


def _hubs_and(V, lengths, seed, each=400):
    """1,024 vertices with `each` edges each among themselves (tiles); lengths[i] edges from anywhere for each vertex i behind them."""
    gen = torch.Generator().manual_seed(seed)
    dst = torch.cat([torch.arange(HUBS).repeat_interleave(each), torch.arange(HUBS, V).repeat_interleave(lengths)])
    src = torch.cat([torch.randint(0, HUBS, (HUBS * each,), generator=gen), torch.randint(0, V, (int(lengths.sum()),), generator=gen)])
    return src.to(torch.int32), dst.to(torch.int32)


@pytest.mark.parametrize("others", [1, 31, 32, 47, 49, 50, 51, 130])
def test_items_of_what_tiles_leave(monkeypatch, others):
    """The rows of the others are left, on either side of the lines between the two lengths of items; half of them have 20 edges fewer or more."""
    V, d = 20_000, 36
    lengths = torch.full((V - HUBS,), others)
    if others > 31:
        lengths[::4], lengths[1::4] = others - 20, others + 20
    monkeypatch.setenv("HT_DENSE_WORK", "1")
    _check(V, d, *_hubs_and(V, lengths, others), torch.randn(V, d, generator=torch.Generator().manual_seed(others)))


# stored entries a row: (of one row of `every`, of the others); rows that items of the rest cut
@pytest.mark.parametrize("every,long,short,cut", [(1, 40, 40, False), (1, 48, 48, False), (1, 60, 60, True), (33, 40, 8, True), (31, 40, 8, False), (33, 48, 8, True), (33, 33, 8, True), (33, 32, 8, False)])
def test_length_of_items_of_what_tiles_leave(monkeypatch, every, long, short, cut):
    """Items of 32 entries for sparse rests, but not where that cuts many rows that items of 48 leave whole: by the memory of the partial sums."""
    V, wide = 300_000, 512
    lengths = torch.full((V - HUBS,), short - 1)
    lengths[::every] = long - 1
    src, dst = _hubs_and(V, lengths, 1, 1000)
    monkeypatch.setenv("HT_DENSE_WORK", "1")
    monkeypatch.setenv("HT_MERGE_DUPS", "0")
    ctx = B.ht_ctx_create(0)
    B.ht_ctx_set_hbm_budget(ctx, 1 << 40)      # (nothing is kept of what the partition gives back)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), 1)
    try:
        H, W, held, free = B.alloc_matrix(V, 16), torch.zeros(wide, 16, device="cuda"), B.ht_graph_info_get(g).hbm_bytes, []
        layers = [(d, B.alloc_matrix(V, d), B.alloc_matrix(V, d)) for d in (4, wide)]      # the plan and its making; partial sums alone
        for d, X, A in layers:
            B.ht_layer_fwd(ctx, g, d, 16, B.HT_ACT_NONE, X, W[:d], H, A)
            B.ht_sync(ctx)
            free.append(torch.cuda.mem_get_info()[0])
        assert B.ht_graph_info_get(g).hbm_bytes > held + 8 * int(lengths.sum()), "the pass was meant to go over tiles"
        sums = int((lengths == long - 1).sum()) * 2 * wide * 4      # two of each row that is cut, beside those of the tiles (some 19 MB)
        assert (free[0] - free[1] > 0.9 * sums) == cut, (free[0] - free[1], sums)
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_shorter_items_refuse_no_plan(monkeypatch):
    """Every other row has 85 entries: two rows of sums in items of 48, 7.2 GB of them, three in items of 32, 10.8 GB, over which the pass plans all the same."""
    V, d = 100_000, 18_000
    lengths = torch.ones(V - HUBS, dtype=torch.int64)
    lengths[::2] = 84
    src, dst = _hubs_and(V, lengths, 1, 1000)
    monkeypatch.setenv("HT_DENSE_WORK", "1")
    monkeypatch.setenv("HT_MERGE_DUPS", "0")
    ctx = B.ht_ctx_create(0)
    B.ht_ctx_set_hbm_budget(ctx, 1 << 40)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), 1)
    try:
        X, A, H, W = B.alloc_matrix(V, d), B.alloc_matrix(V, d), B.alloc_matrix(V, 16), torch.zeros(d, 16, device="cuda")
        at = [0, 1, 9_000, d - 1]
        X[:, at] = torch.randn(V, len(at), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        B.ht_layer_fwd(ctx, g, d, 16, B.HT_ACT_NONE, X, W, H, A)
        B.ht_sync(ctx)
        assert free - torch.cuda.mem_get_info()[0] >= 3 * ((V - HUBS) // 2) * d * 4
        loop = torch.arange(V)
        u, v = torch.cat([src.long(), loop]).cuda(), torch.cat([dst.long(), loop]).cuda()
        s = torch.bincount(v, minlength=V).double().rsqrt()
        want, mag = (torch.zeros(V, len(at), dtype=torch.float64, device="cuda").index_add_(0, v, (s[u] * s[v])[:, None] * Z[u]) for Z in (X[:, at].double(), X[:, at].double().abs()))
        assert ((A[:, at].double() - want).abs() <= 16 * 2.0 ** -24 * mag).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
        del X, A
        torch.cuda.empty_cache()
