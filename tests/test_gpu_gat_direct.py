"""GAT layers with everything in HBM run over all chunks at once, an epoch keeping what its backward passes need.  Against the
oracle, at sizes with cut rows on both sides, merged and unmerged duplicates and pads, with and without the memory for it (the
chunk-by-chunk passes that recompute)."""
import pytest
import torch

from oracle import oracle as orc
from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs
from tests.util import assert_close_grad, hub_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph,dims,n,loops", [
    ("rmat", [20, 41, 6], 5, True),          # few duplicates; pads in both widths
    ("multi", [24, 300, 72, 5], 4, True),    # merged entries; wider than one slab, lane groups of 32 and 8
    ("hub", [16, 64, 8], 3, True),           # rows and sources cut into several items, no pads
    ("rmat", [20, 33, 6], 2, False),         # rows without an entry on either side
    ("tiny", [5, 3, 2], 2, True),
])
@pytest.mark.parametrize("lean", [False, True])
def test_gat_epoch_all_chunks_at_once(graph, dims, n, loops, lean):
    if graph == "hub":
        V = 15_013
        src, dst = hub_graph(V, 120_000, hub_in=2500, hub_out=2000, seed=2)
    elif graph == "tiny":
        V, src, dst = 3, torch.tensor([0, 1, 2, 2], dtype=torch.int32), torch.tensor([1, 2, 0, 1], dtype=torch.int32)
    else:
        V = 9_001
        src, dst = inputs.rmat_edges(V, 150_000, seed=4)
        if graph == "multi":
            k = torch.arange(0, src.numel(), 3)
            src, dst = torch.cat([src, src[k], src[k]]), torch.cat([dst, dst[k], dst[k]])
    gen = torch.Generator().manual_seed(3)
    X, y = torch.randn(V, dims[0], generator=gen), torch.randint(0, dims[-1], (V,), generator=gen).to(torch.int32)
    W, (a_dst, a_src) = inputs.glorot_weights(dims, seed=1), inputs.attention_vectors(dims, seed=2)
    indptr, col = orc.csc_build(V, src.numpy(), dst.numpy(), loops)
    L, lr = len(dims) - 1, 20.0         # (a large step: the updated parameters expose the gradients)
    Wn, adn, asn = ([t.numpy() for t in ts] for ts in (W, a_dst, a_src))
    h, fwd = [X.numpy()], []
    for l in range(L):
        fwd.append(orc.gat_layer_fwd(indptr, col, h[l], Wn[l], adn[l], asn[l], relu=l < L - 1))
        h.append(fwd[l]["h"])
    ref_loss, grad = orc.softmax_ce(h[L], y.numpy())
    want = [None] * L
    for l in reversed(range(L)):
        b = orc.gat_layer_bwd(indptr, col, h[l], Wn[l], adn[l], asn[l], fwd[l], grad, relu=l < L - 1, want_dH=l > 0)
        want[l], grad = [Wn[l] - lr * b["dW"], adn[l] - lr * b["da_dst"], asn[l] - lr * b["da_src"]], b.get("dH")
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), n, add_self_loops=loops)
    try:
        def epoch():
            p = [[t.clone().cuda() for t in ts] for ts in (W, a_dst, a_src)]
            loss, _ = B.ht_gat_epoch(ctx, g, dims, *p, lr, B.to_matrix(X), y.cuda())
            return loss, p
        if lean:     # the smallest budget that an epoch gets through with
            base, step = B.ht_graph_info_get(g).hbm_bytes, 1 << 18
            for k in range(1, 400):
                B.ht_ctx_set_hbm_budget(ctx, base + k * step)
                try:
                    out = epoch()
                    break
                except B.HongtuError as e:
                    assert e.code == B.HT_ENOMEM
            again = epoch()
            B.ht_ctx_set_hbm_budget(ctx, 0)
        else:
            out, again = epoch(), epoch()
        for loss, p in (out, again):
            assert abs(loss - ref_loss) <= 1e-4 * abs(ref_loss)
            for l in range(L):
                for name, ts, w in zip(("W", "a_dst", "a_src"), p, want[l]):
                    assert_close_grad(ts[l].cpu().numpy(), w, f"{name}[{l}] after the step")
        for a, b in zip(out[1], again[1]):      # the sums' order does not depend on the call
            assert all(torch.equal(s, t) for s, t in zip(a, b))
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_gat_backward_chunk_pass_partial_sums_of_both_directions():
    """The chunk-by-chunk backward pass (host-resident input) keeps the partial sums of cut destinations and of cut sources in one
    slot: here the sources need many times more of it, and destinations are cut in the first and in the last chunk."""
    V, di, dn, n = 4_003, 12, 21, 4
    gen = torch.Generator().manual_seed(8)
    hubs = torch.arange(20).repeat_interleave(1500)                       # sources with about 1500 entries each
    src = torch.cat([torch.randint(0, V, (4 * V,), generator=gen), hubs, torch.randint(0, V, (1600,), generator=gen)])
    dst = torch.cat([torch.randint(0, V, (4 * V + hubs.numel(),), generator=gen), torch.tensor([3, V - 2]).repeat_interleave(800)])
    src, dst = src.to(torch.int32), dst.to(torch.int32)
    X, dH = torch.randn(V, di, generator=gen), torch.randn(V, dn, generator=gen)
    W, a_dst, a_src = torch.randn(di, dn, generator=gen) / di ** 0.5, torch.randn(dn, generator=gen) / 4, torch.randn(dn, generator=gen) / 4
    indptr, col = orc.csc_build(V, src.numpy(), dst.numpy(), True)
    p = (W.numpy(), a_dst.numpy(), a_src.numpy())
    fwd = orc.gat_layer_fwd(indptr, col, X.numpy(), *p, relu=False)
    ref = orc.gat_layer_bwd(indptr, col, X.numpy(), *p, fwd, dH.numpy(), relu=False, want_dH=True)
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src.cuda(), dst.cuda(), n)
    try:
        Xh, H, dHd, dX = B.to_matrix(X, B.HT_LOC_HOST_PINNED), B.to_matrix(torch.from_numpy(fwd["h"]).float()), B.to_matrix(dH), B.alloc_matrix(V, di)
        dW, dad, das = torch.empty(di, dn, device="cuda"), torch.empty(dn, device="cuda"), torch.empty(dn, device="cuda")
        B.ht_gat_layer_bwd(ctx, g, di, dn, B.HT_ACT_NONE, Xh, W.cuda(), a_dst.cuda(), a_src.cuda(), H, dHd, dW, dad, das, dH_in=dX)
        B.ht_sync(ctx)
        for got, name in ((dX[:, :di], "dH"), (dW, "dW"), (dad, "da_dst"), (das, "da_src")):
            assert_close_grad(got.cpu().numpy(), ref[name], name)
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
