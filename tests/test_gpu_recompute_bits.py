"""An aggregate that nothing keeps is the same to the last bit wherever it is made again: the backward pass from the layer input against the
forward pass that returned the activations, and whole epochs in every intermediate-data mode, at sizes where passes run over a graph's plan."""
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

pytestmark = pytest.mark.gpu

PLANS = [{"HT_DENSE_WORK": "1", "HT_FINE_WORK": "1"}, {"HT_DENSE": "0", "HT_FINE_WORK": "1"}]


@pytest.fixture
def planned(monkeypatch, request):
    for k, v in request.param.items():
        monkeypatch.setenv(k, v)


@pytest.mark.parametrize("planned", PLANS, indirect=True, ids=["tiles", "short"])
@pytest.mark.parametrize("forward", ["plain", "static"])
def test_layer_from_its_input(planned, forward):
    """W = I, so H is the aggregate itself; dz has a single 1 per column, so a column of grad W is one row of the aggregate made again."""
    V, d = 3_000, 48
    src, dst = inputs.rmat_edges(V, 150_000, 5)
    gen = torch.Generator().manual_seed(1)
    X, I = B.to_matrix(torch.randn(V, d, generator=gen)), torch.eye(d, device="cuda")
    deg = torch.bincount(dst.long(), minlength=V)
    rows = torch.cat([deg.argsort(descending=True)[:d // 2], torch.randperm(V, generator=gen)])
    rows = torch.tensor(list(dict.fromkeys(rows.tolist()))[:d])         # hubs and others, each once
    dz = torch.zeros(V, d)
    dz[rows, torch.arange(d)] = 1.0
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), 3)
    try:
        H, A, dX, dW = B.alloc_matrix(V, d), B.alloc_matrix(V, d), B.alloc_matrix(V, d), torch.empty(d, d, device="cuda")
        base = B.ht_graph_info_get(g).hbm_bytes
        for _ in range(2):        # the second time there is a plan of both directions
            if forward == "static":
                B.ht_layer_fwd_static(ctx, g, d, d, B.HT_ACT_NONE, X, I, H, A)
            else:
                B.ht_layer_fwd(ctx, g, d, d, B.HT_ACT_NONE, X, I, H)
            dX.zero_()
            B.ht_layer_bwd(ctx, g, d, d, B.HT_ACT_NONE, X, I, B.to_matrix(dz), dW, dH_in=dX, ckpt_kind=B.HT_CKPT_INPUT)
            B.ht_sync(ctx)
            assert torch.equal(dW.t().cpu(), H[:, :d].cpu()[rows])
            B.ht_layer_fwd(ctx, g, d, d, B.HT_ACT_NONE, X, I, B.alloc_matrix(V, d), A)
            B.ht_sync(ctx)
            assert B.ht_graph_info_get(g).hbm_bytes > base, "the passes were meant to plan"
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def _modes(V, E, dims, n, epochs=2):
    src, dst = inputs.rmat_edges(V, E, 5, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    X = B.alloc_matrix(V, dims[0])
    X[:, :dims[0]] = torch.randn(V, dims[0], generator=gen, device="cuda")
    y = torch.randint(0, dims[-1], (V,), generator=gen, device="cuda").to(torch.int32)
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src, dst, n)
    del src, dst
    try:
        base, outs = B.ht_graph_info_get(g).hbm_bytes, []
        for inter in (B.HT_INTER_RECOMPUTE, B.HT_INTER_MASK, B.HT_INTER_HYBRID, B.HT_INTER_RECOMPUTE):
            W = [w.cuda() for w in inputs.glorot_weights(dims, seed=4)]
            losses = [B.ht_epoch(ctx, g, dims, W, 0.5, X, y, inter=inter)[0] for _ in range(epochs)]
            outs.append((losses, [w.cpu() for w in W]))
        assert B.ht_graph_info_get(g).hbm_bytes > base, "the passes were meant to plan"
        for losses, W in outs[1:]:
            assert losses == outs[0][0]
            assert all(torch.equal(a, b) for a, b in zip(W, outs[0][1]))
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


@pytest.mark.parametrize("planned", PLANS, indirect=True, ids=["tiles", "short"])
def test_epochs_of_every_mode(planned):
    _modes(3_000, 150_000, [72, 40, 8], 3)


def test_epochs_with_aggregates_beyond_two_gib():
    _modes(4_300_000, 9_000_000, [128, 16, 4], 4, epochs=1)
