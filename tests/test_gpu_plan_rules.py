"""Both sides of the rules that small graphs do not reach by themselves: products that read W in place, rows wider than a column block over dense tiles, rows that column units
address in 64 bits, the least rows for short items, and the end of a GAT epoch whose attention vectors share memory."""
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


def _passes(V, src, dst, d, n=2, passes=("fwd", "bwd")):
    """(aggregate, backward aggregate, bytes that the graph holds before and after)"""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    X, dz = B.alloc_matrix(V, d), B.alloc_matrix(V, d)
    X[:, :d], dz[:, :d] = (torch.randn(V, d, generator=gen, device="cuda") for _ in range(2))
    W = torch.eye(d, device="cuda")
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), n)
    try:
        H, A, dX, dW = B.alloc_matrix(V, d), B.alloc_matrix(V, d), B.alloc_matrix(V, d), torch.empty(d, d, device="cuda")
        held = [B.ht_graph_info_get(g).hbm_bytes]
        B.ht_layer_fwd(ctx, g, d, d, B.HT_ACT_NONE, X, W, H, A)
        B.ht_sync(ctx)
        held.append(B.ht_graph_info_get(g).hbm_bytes)
        if "bwd" in passes:
            dX.zero_()
            B.ht_layer_bwd(ctx, g, d, d, B.HT_ACT_NONE, A, W, dz, dW, dH_in=dX)
            B.ht_sync(ctx)
        return X[:, :d], dz[:, :d], A[:, :d], dX[:, :d], held
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("d", [1024, 1030, 1100, 2050])
def test_rows_wider_than_a_column_block(d, monkeypatch):
    monkeypatch.setenv("HT_DENSE_WORK", "1")
    V = 700
    src, dst = inputs.rmat_edges(V, 40 * V, 3)
    X, dz, A, dX, held = _passes(V, src, dst, d)
    assert held[1] > held[0], "the pass was meant to plan"
    loop = torch.arange(V)
    u, v = torch.cat([src.long(), loop]).cuda(), torch.cat([dst.long(), loop]).cuda()
    s = torch.bincount(v, minlength=V).double().rsqrt()
    w = (s[u] * s[v])[:, None]
    for got, a, b, Z in ((A, u, v, X), (dX, v, u, dz)):
        want, mag = (torch.zeros(V, d, dtype=torch.float64, device="cuda").index_add_(0, b, w * Y.double()[a]) for Y in (Z, Z.abs()))
        # (dX goes through a product with the unit matrix, exact)
        assert ((got.double() - want).abs() <= 16 * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("V,E,d", [(300_007, 3_000_000, 64), (600_011, 3_000_000, 32), (140_003, 2_000_000, 128)])
def test_rows_addressed_in_64_bits(V, E, d, monkeypatch):
    """The same sums at either width of the offsets; rows of 4 GiB and more need the wider ones."""
    monkeypatch.setenv("HT_DENSE", "0")
    monkeypatch.setenv("HT_FINE_WORK", "1")
    src, dst = inputs.rmat_edges(V, E, 3, device="cuda")
    _, _, A, dX, held = _passes(V, src, dst, d)
    assert held[1] > held[0]
    monkeypatch.setenv("HT_UNIT_SMALL", "0")
    _, _, A2, dX2, _ = _passes(V, src, dst, d)
    assert torch.equal(A, A2) and torch.equal(dX, dX2)
    assert A.isfinite().all() and float(A.abs().sum()) > 0


@pytest.mark.parametrize("entries,cut", [(64, False), (65, True)])
def test_length_of_short_items(entries, cut, monkeypatch):
    """Rows of up to 64 entries are one work item: no partial sums, two rows of them for each row beyond."""
    monkeypatch.setenv("HT_DENSE", "0")
    monkeypatch.setenv("HT_MERGE_DUPS", "0")
    V, d = 400_000, 64
    gen = torch.Generator(device="cuda").manual_seed(1)
    dst = torch.arange(V, dtype=torch.int32, device="cuda").repeat_interleave(entries - 1)
    src = torch.randint(0, V, (dst.numel(),), generator=gen, dtype=torch.int32, device="cuda")
    ctx = B.ht_ctx_create(0)
    B.ht_ctx_set_hbm_budget(ctx, 1 << 40)      # (nothing is kept of what the partition gives back)
    g = B.ht_partition(ctx, V, src, dst, 1)
    try:
        X, A, H, W = B.alloc_matrix(V, d).zero_(), B.alloc_matrix(V, d), B.alloc_matrix(V, 16), torch.zeros(d, 16, device="cuda")
        held = B.ht_graph_info_get(g).hbm_bytes
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        B.ht_layer_fwd(ctx, g, d, 16, B.HT_ACT_NONE, X, W, H, A)
        B.ht_sync(ctx)
        assert B.ht_graph_info_get(g).hbm_bytes > held, "the pass was meant to plan"
        taken = free - torch.cuda.mem_get_info()[0]
        assert (taken >= 2 * V * d * 4) == cut, taken
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_rows_beyond_four_gib():
    """... and rows that really are that large, against the sums of an equal graph's passes that do not plan."""
    V, E, d = 8_600_000, 9_000_000, 128
    src, dst = inputs.rmat_edges(V, E, 3, device="cuda")
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src, dst, 4)
    try:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(1)
        X, A, H, H2 = B.alloc_matrix(V, d), B.alloc_matrix(V, d), B.alloc_matrix(V, 4), B.alloc_matrix(V, 4)
        X.normal_(generator=gen)
        W = torch.randn(d, 4, generator=gen, device="cuda")
        base = B.ht_graph_info_get(g).hbm_bytes
        B.ht_layer_fwd(ctx, g, d, 4, B.HT_ACT_NONE, X, W, H, A)
        B.ht_layer_fwd(ctx, g, d, 4, B.HT_ACT_NONE, X, W, H2)
        B.ht_sync(ctx)
        assert B.ht_graph_info_get(g).hbm_bytes > base, "the pass was meant to plan"
        # (rows of up to a few thousand terms, then a product over 128: orders of the same fp32 sums)
        assert float((H - H2).norm() / H2.norm()) <= 1e-6
        assert float((H - H2).abs().max()) <= 1e-5 * float(H2.abs().max())
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def _held(V, src, dst, d, fine, monkeypatch):
    """Bytes that the graph holds before any pass, after a forward and after a backward pass; the aggregates."""
    monkeypatch.setenv("HT_DENSE", "0")
    monkeypatch.setenv("HT_FINE", fine)
    X, W, dh = B.alloc_matrix(V, d), torch.ones(d, 4, device="cuda") / d, B.alloc_matrix(V, 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    X.normal_(generator=gen)
    dh.normal_(generator=gen)
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src, dst, 3)
    try:
        H, A, dX, dW = B.alloc_matrix(V, 4), B.alloc_matrix(V, d), B.alloc_matrix(V, d), torch.empty(d, 4, device="cuda")
        held = [B.ht_graph_info_get(g).hbm_bytes]
        B.ht_layer_fwd(ctx, g, d, 4, B.HT_ACT_NONE, X, W, H, A)
        B.ht_sync(ctx)
        held.append(B.ht_graph_info_get(g).hbm_bytes)
        dX.zero_()
        B.ht_layer_bwd(ctx, g, d, 4, B.HT_ACT_NONE, A, W, dh, dW, dH_in=dX)
        B.ht_sync(ctx)
        held.append(B.ht_graph_info_get(g).hbm_bytes)
        return held, A[:, :d].clone(), dX[:, :d].clone()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("V,E,d,fwd,bwd", [
    (100_000, 2_500_000, 96, True, False),      # the slab kernel: forward from 64 columns and 16 entries a row on
    (100_000, 1_300_000, 160, False, True),     # ... fewer entries a row; backward between 129 and 256 columns
    (220_000, 9_000_000, 32, False, False),     # ... narrow
    (70_000, 3_000_000, 80, False, False),      # ... rows of less than 24 MiB
    (70_000, 5_000_000, 130, True, False),      # ... long rows
    (20_000, 400_000, 602, True, True),         # ... wide
    (20_000, 800_000, 602, True, False),        # ... wide and long
    (300_000, 4_000_000, 64, True, True),       # one column unit
    (300_000, 24_000_000, 64, True, False),     # ... long rows
    (300_000, 4_000_000, 96, True, False),      # one and a half
    (300_000, 4_000_000, 128, True, True),      # two
    (300_000, 4_000_000, 192, True, False),     # three, few entries a row
    (300_000, 6_000_000, 192, True, True),      # three
    (100_000, 1_300_000, 256, True, True),      # four
])
def test_which_passes_take_short_items(V, E, d, fwd, bwd, monkeypatch):
    src, dst = inputs.rmat_edges(V, E, 3, device="cuda")
    plain, A, dX = _held(V, src, dst, d, "0", monkeypatch)
    held, A2, dX2 = _held(V, src, dst, d, "1", monkeypatch)
    extra = [h - p for h, p in zip(held, plain)]
    assert extra[0] == 0
    assert (extra[1] > 0) == fwd and (extra[2] > extra[1]) == bwd
    for x, y, planned in ((A, A2, fwd), (dX, dX2, bwd)):
        assert float((x - y).norm() / x.norm()) <= (1e-6 if planned else 0.0)


@pytest.mark.parametrize("V", [200, 20_000])
@pytest.mark.parametrize("K,N", [(192, 100), (193, 100), (120, 256), (512, 64), (513, 64), (100, 192), (100, 193), (602, 256)])
def test_products_around_the_packing_rule(V, K, N):
    """No edges but the self-loops: the layer is H W forward and dz W^T backward, the same whether W is read in place or packed."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K + N)
    rand = lambda a, b: torch.randn(a, b, generator=gen, device="cuda")
    H, W, dz = rand(V, K), rand(K, N), rand(V, N)
    ctx = B.ht_ctx_create(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, 1)
    more = B.ht_partition(ctx, 40_000, none, none, 1)      # (beyond the rows that read W in place)
    try:
        def both(graph, H, dz):
            v = H.shape[0]
            out, A, dX, dW = B.alloc_matrix(v, N), B.alloc_matrix(v, K), B.alloc_matrix(v, K), torch.empty(K, N, device="cuda")
            dX.zero_()
            B.ht_layer_fwd(ctx, graph, K, N, B.HT_ACT_NONE, B.to_matrix(H), W, out, A)
            B.ht_layer_bwd(ctx, graph, K, N, B.HT_ACT_NONE, A, W, B.to_matrix(dz), dW, dH_in=dX)
            B.ht_sync(ctx)
            return out[:, :N], dX[:, :K]
        got = both(g, H, dz)
        for x, a, b in zip(got, (H, dz), (W, W.t())):
            want, mag = a.double() @ b.double(), a.abs().double() @ b.abs().double()
            # n fp32 products and sums: off by at most (n + 2) 2^-24 of the sum of absolute values
            assert ((x.double() - want).abs() <= (b.shape[0] + 4) * 2.0 ** -24 * mag).all()
        times = 40_000 // V + 1
        packed = both(more, H.repeat(times, 1)[:40_000], dz.repeat(times, 1)[:40_000])
        assert all(torch.equal(x, y[:V]) for x, y in zip(got, packed))
    finally:
        for x in (g, more):
            B.ht_graph_destroy(x)
        B.ht_ctx_destroy(ctx)


def test_gat_parameters_that_share_memory():
    """Two layers with one pair of attention vectors: both layers' steps reach them."""
    V, d = 2_000, 24
    src, dst = inputs.rmat_edges(V, 20_000, 5)
    gen = torch.Generator().manual_seed(1)
    X, y = B.to_matrix(torch.randn(V, d, generator=gen)), torch.randint(0, d, (V,), generator=gen).to(torch.int32).cuda()
    W0 = inputs.glorot_weights([d, d, d], seed=4)
    a0 = [torch.randn(d, generator=gen) / 5 for _ in range(2)]
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), 2)
    try:
        def epoch(a_dst, a_src):
            W = [w.clone().cuda() for w in W0]
            loss, _ = B.ht_gat_epoch(ctx, g, [d, d, d], W, a_dst, a_src, 0.5, X, y)
            return loss, W
        apart = [[a.clone().cuda() for _ in range(2)] for a in a0]
        shared = [a.clone().cuda() for a in a0]
        loss1, W1 = epoch(*apart)
        loss2, W2 = epoch([shared[0]] * 2, [shared[1]] * 2)
        assert loss1 == loss2 and all(torch.equal(a, b) for a, b in zip(W1, W2))
        for a, two, one in zip(a0, apart, shared):
            steps = [t.cpu().double() - a.double() for t in two]
            assert all(float(s.abs().max()) > 0 for s in steps)
            want = a.double() + steps[0] + steps[1]
            # one rounding for each of the three updates that are compared
            assert ((one.cpu().double() - want).abs() <= 4 * 2.0 ** -24 * (a.double().abs() + want.abs())).all()
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
