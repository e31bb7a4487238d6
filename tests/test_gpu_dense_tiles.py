"""Passes over a graph's plan: the products over its dense tiles (256 rows x 64 columns of multiplicities), the work items over the
entries in no tile, and short work items.  Against plain fp64 sums, at the edges of tiles and of column blocks, with multiplicities that a
tile holds and does not hold, with values that are not finite or beyond what the split products take, and twice for the same bits."""
import numpy as np
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu


def _edges(V, kind, gen):
    """Every pair once or more often: one tile after the other is full."""
    if kind == "rmat":
        return inputs.rmat_edges(V, 40 * V, 3)
    u, v = (x.reshape(-1) for x in torch.meshgrid(torch.arange(V), torch.arange(V), indexing="ij"))
    keep = (u != v) & (torch.rand(V * V, generator=gen) < 0.7)
    u, v = u[keep], v[keep]
    if kind == "heavy":      # one in 40 pairs twice, a few of them 254 .. 257 and 1000 times
        more = torch.randint(0, len(u), (len(u) // 40,), generator=gen)
        times = torch.ones_like(more)
        times[:10] = torch.tensor([253, 254, 255, 256, 999, 253, 254, 255, 256, 999])
        u, v = torch.cat([u, u[more].repeat_interleave(times)]), torch.cat([v, v[more].repeat_interleave(times)])
    p = torch.randperm(V, generator=gen)
    return p[u].to(torch.int32), p[v].to(torch.int32)


class Case:
    def __init__(self, V, kind, d, seed=1):
        gen = torch.Generator().manual_seed(seed)
        self.V, self.d = V, d
        self.src, self.dst = _edges(V, kind, gen)
        self.X = torch.randn(V, d, generator=gen)
        self.dz = torch.randn(V, d, generator=gen)
        loop = torch.arange(V)
        self.u, self.v = torch.cat([self.src.long(), loop]), torch.cat([self.dst.long(), loop])
        s = torch.bincount(self.v, minlength=V).double().rsqrt()
        self.w = s[self.u] * s[self.v]

    def ref(self):
        """(A X, A^T dz) and the same of absolute values"""
        def agg(a, b, Z):
            out = torch.zeros(self.V, self.d, dtype=torch.float64)
            for i in range(0, len(a), 1 << 17):
                out.index_add_(0, b[i:i + (1 << 17)], self.w[i:i + (1 << 17), None] * Z.double()[a[i:i + (1 << 17)]])
            return out
        return [(agg(self.u, self.v, x), agg(self.u, self.v, x.abs())) if x is self.X else (agg(self.v, self.u, x), agg(self.v, self.u, x.abs()))
                for x in (self.X, self.dz)]

    def run(self, calls=2):
        """The layer's aggregate and its backward aggregate (identity weights), and whether the graph has a plan."""
        V, d = self.V, self.d
        ctx = B.ht_ctx_create(0)
        g = B.ht_partition(ctx, V, self.src.cuda(), self.dst.cuda(), 2)
        try:
            I = torch.eye(d, device="cuda")
            Xd, dzd = B.to_matrix(self.X), B.to_matrix(self.dz)
            H, A, dX, dW = B.alloc_matrix(V, d), B.alloc_matrix(V, d), B.alloc_matrix(V, d), torch.empty(d, d, device="cuda")
            base = B.ht_graph_info_get(g).hbm_bytes
            outs = []
            for _ in range(calls):
                A.fill_(7.0)
                dX.zero_()
                B.ht_layer_fwd(ctx, g, d, d, B.HT_ACT_NONE, Xd, I, H, A)
                if not outs:
                    assert B.ht_graph_info_get(g).hbm_bytes > base, "the pass was meant to plan"
                B.ht_layer_bwd(ctx, g, d, d, B.HT_ACT_NONE, A, I, dzd, dW, dH_in=dX)
                B.ht_sync(ctx)
                outs.append((A[:, :d].cpu(), dX[:, :d].cpu()))
            for a, b in zip(outs[0], outs[-1]):
                assert torch.equal(a.nan_to_num(nan=3.5), b.nan_to_num(nan=3.5))
            return outs[0]
        finally:
            B.ht_graph_destroy(g)
            B.ht_ctx_destroy(ctx)


def _check(got, ref):
    # A sum of n fp32 terms is off by at most (n + 2) 2^-24 of the sum of their absolute values, and by far less in blocks; 16 x 2^-24
    # covers the factors' roundings and the few dozen additions on the longest path here several times over.
    for g, (r, mag) in zip(got, ref):
        assert ((g.double() - r).abs() <= 16 * 2.0 ** -24 * mag).all(), float(((g.double() - r).abs() / mag).max() * 2 ** 24)


@pytest.fixture
def planned(monkeypatch, request):
    for k, v in getattr(request, "param", {"HT_DENSE_WORK": "1", "HT_FINE_WORK": "1"}).items():
        monkeypatch.setenv(k, v)


@pytest.mark.parametrize("V", [64, 65, 255, 256, 257, 320, 513])
@pytest.mark.parametrize("kind", ["full", "heavy"])
def test_tile_edges(planned, V, kind):
    c = Case(V, kind, 20, seed=V)
    _check(c.run(), c.ref())


@pytest.mark.parametrize("d", [1, 4, 7, 31, 63, 64, 65, 127, 128, 129, 192, 193, 256, 300])
def test_column_blocks(planned, d):
    c = Case(700, "rmat" if d % 2 else "heavy", d, seed=d)
    _check(c.run(), c.ref())


@pytest.mark.parametrize("planned", [{"HT_DENSE": "0", "HT_FINE_WORK": "1"}, {"HT_DENSE_WORK": "1"}], indirect=True)
@pytest.mark.parametrize("V,d", [(3000, 33), (30_011, 130)])
def test_rest_and_short_items(planned, V, d):
    c = Case(V, "rmat", d)
    _check(c.run(), c.ref())


@pytest.mark.parametrize("V,d", [(300_007, 64), (140_003, 128), (300_007, 24), (600_011, 32)])
def test_column_units(planned, V, d):
    """Rows beyond 64 MiB (and one below): a wave works on 4 or 8 short items."""
    c = Case(V, "rmat", d)
    _check(c.run(), c.ref())


@pytest.mark.parametrize("d", [20, 130])
def test_values_out_of_range(planned, d):
    """Infinities and NaN reach exactly the rows that name them; values that the scaled parts cannot hold and subnormal ones are as exact
    as any (the sums, where a subnormal result is kept to its last bit)."""
    V = 520
    c = Case(V, "heavy", d)
    c.X[3] = float("inf")
    c.X[4, d // 2] = float("nan")
    c.X[5] = -float("inf")
    c.X[6, 0] = 3e38
    # (the forward aggregate alone: the product before the backward one spreads 0 x inf over the row)
    g, r32 = c.run()[0], c.ref()[0][0].float()
    assert torch.equal(torch.isnan(g), torch.isnan(r32)) and torch.equal(torch.isinf(g), torch.isinf(r32))
    assert torch.equal(g[torch.isinf(g)], r32[torch.isinf(r32)])
    assert torch.isnan(g).any() and torch.isfinite(g).any()
    for scale in (2.0 ** 63, 2.0 ** 66, 2.0 ** 90, 2.0 ** -100, 2.0 ** -130):
        c = Case(V, "heavy", d, seed=3)
        c.X, c.dz = c.X * scale, c.dz * scale
        for g, (r, mag) in zip(c.run(1), c.ref()):
            assert ((g.double() - r).abs() <= 16 * 2.0 ** -24 * mag + 64 * 2.0 ** -149).all(), scale


def test_accumulates_and_masks(planned):
    """The backward pass adds to dH_in, and an epoch's layers, ReLU masks and stage orders take the same plan."""
    V, d, o = 900, 70, 33
    c = Case(V, "heavy", d)
    gen = torch.Generator().manual_seed(9)
    W, dh, keep = torch.randn(d, o, generator=gen) / 8, torch.randn(V, o, generator=gen), torch.randn(V, o, generator=gen)
    dz = (dh * (keep > 0)).double()
    want = torch.zeros(V, d, dtype=torch.float64).index_add_(0, c.u, c.w[:, None] * (dz @ W.double().t())[c.v])
    for order in (B.HT_ORDER_AGG_FIRST, B.HT_ORDER_UPDATE_FIRST):
        ctx = B.ht_ctx_create(0)
        g = B.ht_partition(ctx, V, c.src.cuda(), c.dst.cuda(), 3)
        try:
            dX, dW = B.alloc_matrix(V, d), torch.empty(d, o, device="cuda")
            dX.fill_(2.0)
            for _ in range(2):
                B.ht_layer_bwd(ctx, g, d, o, B.HT_ACT_RELU, B.to_matrix(c.X), W.cuda(), B.to_matrix(dh), dW, dH_in=dX, H_out=B.to_matrix(keep),
                               ckpt_kind=B.HT_CKPT_INPUT, order=order)
            B.ht_sync(ctx)
            err = (dX[:, :d].cpu().double() - (2 * want + 2.0)).abs().max()
            assert err <= 2e-5 * want.abs().max() + 2.0 ** -20
        finally:
            B.ht_graph_destroy(g)
            B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("planned", [{"HT_DENSE_WORK": "1", "HT_FINE": "0"}], indirect=True)
def test_no_room_for_the_plan(planned):
    """Without memory for it the passes take the graph's own items, call after call, and the plan once there is room."""
    c = Case(2000, "rmat", 40)
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, c.V, c.src.cuda(), c.dst.cuda(), 2)
    try:
        I, Xd = torch.eye(40, device="cuda"), B.to_matrix(c.X)
        H, A = B.alloc_matrix(c.V, 40), B.alloc_matrix(c.V, 40)
        base = B.ht_graph_info_get(g).hbm_bytes
        outs = []
        for room in (1 << 20, 1 << 20, 0):
            B.ht_ctx_set_hbm_budget(ctx, base + room if room else 0)
            B.ht_layer_fwd(ctx, g, 40, 40, B.HT_ACT_NONE, Xd, I, H, A)
            B.ht_sync(ctx)
            assert (B.ht_graph_info_get(g).hbm_bytes > base) == (room == 0)
            outs.append(A[:, :40].cpu())
        assert torch.equal(outs[0], outs[1])
        assert np.allclose(outs[0].numpy(), outs[2].numpy(), rtol=0, atol=1e-6 * float(outs[0].abs().max()))
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("planned", [{"HT_DENSE_WORK": "1"}, {"HT_DENSE": "0", "HT_FINE_WORK": "1"}], indirect=True)
def test_first_pass_inside_a_callers_capture(planned, monkeypatch):
    """A pass that would make its plan while its caller records the stream records the graph's own items instead, with the bits of the
    forward that keeps no aggregate; the plan is made by the next pass outside of a capture."""
    c = Case(2000, "rmat", 40)
    st = torch.cuda.Stream()
    ctx = B.ht_ctx_create(0, st.cuda_stream)
    g = B.ht_partition(ctx, c.V, c.src.cuda(), c.dst.cuda(), 2)
    try:
        I, Xd = torch.eye(40, device="cuda"), B.to_matrix(c.X)
        H, H2, A = (B.alloc_matrix(c.V, 40) for _ in range(3))
        torch.cuda.synchronize()
        B.ht_layer_fwd(ctx, g, 40, 40, B.HT_ACT_NONE, Xd, I, H)
        B.ht_sync(ctx)
        before = B.ht_graph_info_get(g).hbm_bytes
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st), monkeypatch.context() as m:
            m.setattr(torch.cuda, "synchronize", lambda *a: None)     # (the binding's, before every call)
            B.ht_layer_fwd(ctx, g, 40, 40, B.HT_ACT_NONE, Xd, I, H2, A)
        assert B.ht_graph_info_get(g).hbm_bytes == before
        for _ in range(3):
            H2.zero_()
            A.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(H2[:, :40], H[:, :40]) and torch.equal(A[:, :40], H[:, :40])
        B.ht_layer_fwd(ctx, g, 40, 40, B.HT_ACT_NONE, Xd, I, H2, A)
        B.ht_sync(ctx)
        assert B.ht_graph_info_get(g).hbm_bytes > before
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
