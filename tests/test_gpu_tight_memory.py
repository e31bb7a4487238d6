"""Memory that only makes calls faster is not what a call is refused for: every call gets through with the device memory that its
chunk-by-chunk pass needs, on a fresh context and on one that earlier calls have filled, with the same results, and takes the faster
pass again once there is room."""
import pytest
import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs
from tests.util import assert_close, assert_close_grad

pytestmark = pytest.mark.gpu

DI, DN, DIMS = 130, 70, [130, 70, 20]
GRAPHS = {"merged": (40_001, 4_000_000, 3), "sparse": (120_003, 700_001, 9)}
# MiB above what a layer of 4 columns gets through with: the smallest budgets of passes that go chunk by chunk alone (one chunk's
# rows twice, partial sums of one chunk, the tensors of an epoch), measured with a build that had no others.
NEEDS = {
    "fwd": dict(merged=28.41, sparse=41.10),
    "fwd_keep": dict(merged=1.77, sparse=0.22),
    "fwd_update_first": dict(merged=13.33, sparse=37.24),
    "bwd": dict(merged=45.22, sparse=54.96),
    "bwd_recompute": dict(merged=90.54, sparse=115.50),
    "bwd_update_first": dict(merged=27.99, sparse=66.64),
    "epoch": dict(merged=92.49, sparse=219.50),
    "epoch_recompute": dict(merged=106.69, sparse=186.54),
    "gat_bwd": dict(merged=62.77, sparse=126.02),
    "gat_epoch": dict(merged=94.58, sparse=221.35),
}
SLACK = 0.1


class Ctx:
    def __init__(self, data):
        V, src, dst, n = data["V"], data["src"], data["dst"], data["n"]
        self.d, self.ctx = data, B.ht_ctx_create(0)
        self.g = B.ht_partition(self.ctx, V, src, dst, n)
        self.H, self.A, self.dX = B.alloc_matrix(V, DN), B.alloc_matrix(V, DI), B.alloc_matrix(V, DI)
        self.dW, self.dad, self.das = torch.empty(DI, DN, device="cuda"), torch.empty(DN, device="cuda"), torch.empty(DN, device="cuda")

    def close(self):
        B.ht_graph_destroy(self.g)
        B.ht_ctx_destroy(self.ctx)

    def budget(self, mib):
        B.ht_ctx_set_hbm_budget(self.ctx, int(mib * 2 ** 20))

    def tiny(self):
        V, X = self.d["V"], self.d["X4"]
        B.ht_layer_fwd(self.ctx, self.g, 4, 4, B.HT_ACT_RELU, X, self.d["W4"], B.alloc_matrix(V, 4), B.alloc_matrix(V, 4))
        B.ht_sync(self.ctx)

    def run(self, what):
        """The call's outputs, named."""
        c, g, d = self.ctx, self.g, self.d
        X, W = d["X"], d["W"][0]
        order = B.HT_ORDER_UPDATE_FIRST if what.endswith("update_first") else B.HT_ORDER_AGG_FIRST
        if what.startswith("fwd"):
            B.ht_layer_fwd(c, g, DI, DN, B.HT_ACT_RELU, X, W, self.H, self.A if what == "fwd_keep" else None, order=order)
            out = {"H": self.H[:, :DN]}
        elif what.startswith("bwd"):
            self.dX.zero_()
            keeps = what == "bwd"
            B.ht_layer_bwd(c, g, DI, DN, B.HT_ACT_RELU, d["A"] if keeps else X, W, d["dz"], self.dW, dH_in=self.dX, H_out=d["kept"],
                           ckpt_kind=B.HT_CKPT_AGG if keeps else B.HT_CKPT_INPUT, order=order)
            out = {"dW": self.dW, "dX": self.dX[:, :DI]}
        elif what == "gat_bwd":
            self.dX.zero_()
            B.ht_gat_layer_bwd(c, g, DI, DN, B.HT_ACT_RELU, X, W, d["ad"][0], d["as"][0], d["kept"], d["dz"], self.dW, self.dad, self.das,
                               dH_in=self.dX)
            out = {"dW": self.dW, "dX": self.dX[:, :DI], "da_dst": self.dad, "da_src": self.das}
        else:
            Ws, ad, as_ = ([t.clone() for t in d[k]] for k in ("W", "ad", "as"))
            if what == "gat_epoch":
                loss, _ = B.ht_gat_epoch(c, g, DIMS, Ws, ad, as_, 5.0, X, d["y"])
            else:
                inter = B.HT_INTER_RECOMPUTE if what == "epoch_recompute" else B.HT_INTER_AUTO
                loss, _ = B.ht_epoch(c, g, DIMS, Ws, 5.0, X, d["y"], inter=inter)
            out = {"loss": torch.tensor([loss]), "W0": Ws[0], "W1": Ws[1]}
        B.ht_sync(c)
        return {k: v.cpu().numpy().copy() for k, v in out.items()}

    def graph_bytes(self):
        return B.ht_graph_info_get(self.g).hbm_bytes


def _close(got, want, what):
    for k, w in want.items():
        (assert_close if k in ("H", "loss") else assert_close_grad)(got[k], w, f"{what}: {k}")


@pytest.fixture(scope="module", params=list(GRAPHS))
def data(request):
    V, E, n = GRAPHS[request.param]
    src, dst = inputs.rmat_edges(V, E, 7)
    gen = torch.Generator().manual_seed(5)
    rand = lambda d: B.to_matrix(torch.randn(V, d, generator=gen))
    d = dict(name=request.param, V=V, n=n, src=src.cuda(), dst=dst.cuda(), X=rand(DI), A=rand(DI), dz=rand(DN), kept=rand(DN), X4=rand(4),
             W4=torch.randn(4, 4, generator=gen).cuda(), W=[w.cuda() for w in inputs.glorot_weights(DIMS, seed=4)],
             y=torch.randint(0, DIMS[-1], (V,), generator=gen).to(torch.int32).cuda())
    d["ad"], d["as"] = ([a.cuda() for a in x] for x in inputs.attention_vectors(DIMS, seed=5))
    lo, hi = 0.0, 512.0       # the smallest budget of the smallest layer
    while hi - lo > 0.01:
        mid = (lo + hi) / 2
        c = Ctx(d)
        c.budget(mid)
        try:
            c.tiny()
            hi = mid
        except B.HongtuError as e:
            assert e.code == B.HT_ENOMEM
            lo = mid
        c.close()
    d["smallest"] = hi
    return d


@pytest.mark.parametrize("held", [False, True])
@pytest.mark.parametrize("what", list(NEEDS))
def test_smallest_budget(data, what, held):
    c = Ctx(data)
    try:
        base = c.graph_bytes()
        if held:               # scratch memory and a by-source list that wider passes have left
            c.run("bwd_recompute")
            c.run("gat_bwd")
            assert c.graph_bytes() > base
        c.budget(data["smallest"] + NEEDS[what][data["name"]] + SLACK)
        first, again = c.run(what), c.run(what)
        for k in first:        # and the second call takes the same pass
            assert (first[k] == again[k]).all(), k
        c.budget(0)
        roomy = c.run(what)
        if "bwd" in what or "epoch" in what:
            assert c.graph_bytes() > base, "all chunks at once again"
        _close(first, roomy, what)
    finally:
        c.close()


def test_partition_beside_a_filled_context(data):
    """A second graph is partitioned in what two graphs alone need, whatever calls on the first one have left in the context."""
    def second(c):
        return B.ht_partition(c.ctx, data["V"], data["src"], data["dst"], data["n"])
    lo, hi = data["smallest"], 1024.0
    while hi - lo > 0.05:
        mid, c = (lo + hi) / 2, Ctx(data)
        c.budget(mid)
        try:
            B.ht_graph_destroy(second(c))
            hi = mid
        except B.HongtuError as e:
            assert e.code == B.HT_ENOMEM
            lo = mid
        c.close()
    c = Ctx(data)
    try:
        want = c.run("bwd_recompute")
        c.budget(hi + SLACK)
        g = second(c)
        c.budget(0)
        _close(c.run("bwd_recompute"), want, "the first graph afterwards")
        B.ht_graph_destroy(g)
    finally:
        c.close()


def test_graph_capture_under_a_tight_budget(data):
    """Epochs that go chunk by chunk for want of memory settle on their scratch memory, so that they can be captured and replayed."""
    c = Ctx(data)
    try:
        c.budget(data["smallest"] + NEEDS["epoch"][data["name"]] + SLACK)
        Ws, plain = ([t.clone() for t in data["W"]] for _ in range(2))
        losses = [B.ht_epoch(c.ctx, c.g, DIMS, Ws, 0.5, data["X"], data["y"], use_graph=True)[0] for _ in range(6)]
        assert B.ht_ctx_graph_launches(c.ctx) >= 3
        assert losses == [B.ht_epoch(c.ctx, c.g, DIMS, plain, 0.5, data["X"], data["y"])[0] for _ in range(6)]
        assert all(torch.equal(a, b) for a, b in zip(Ws, plain))
    finally:
        c.close()


def test_second_epoch_keeps_its_plan(monkeypatch):
    """The residency planner goes by free memory: what the first epoch's passes keep for the second counts as free."""
    V, dims, n = 500_000, [256, 256, 64], 4
    src, dst = inputs.rmat_edges(V, 1_000_000, 3, device="cuda")
    X = torch.zeros(V, dims[0], device="cuda")
    y = torch.zeros(V, dtype=torch.int32, device="cuda")
    W = [w.cuda() for w in inputs.glorot_weights(dims, seed=4)]
    tensors = V * 4 * (2 * dims[2] + 2 * dims[1] + dims[0] + dims[1])       # logits, h^1 and their gradients; a^0, a^1
    monkeypatch.setenv("HT_DEVICE_BYTES", str(tensors + (2048 + 300) * 2 ** 20))
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src, dst, n)
    try:
        plans = []
        base = B.ht_graph_info_get(g).hbm_bytes
        for _ in range(3):
            _, st = B.ht_epoch(ctx, g, dims, W, 0.1, X, y, want_stats=True)
            plans.append((st.plan_inter, st.plan_res_h, st.plan_res_a, st.plan_res_g))
        assert plans[0][1:] == (B.HT_RES_HBM,) * 3, plans
        assert B.ht_graph_info_get(g).hbm_bytes > base, "the passes were meant to keep more than the tensors"
        assert plans == plans[:1] * 3, plans
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_refused_call_changes_nothing(data):
    """A backward pass that is refused memory has not added to dH_in."""
    c = Ctx(data)
    try:
        c.budget(data["smallest"] + 1)
        c.dX.fill_(7.0)
        with pytest.raises(B.HongtuError) as e:
            B.ht_layer_bwd(c.ctx, c.g, DI, DN, B.HT_ACT_RELU, data["X"], data["W"][0], data["dz"], c.dW, dH_in=c.dX, H_out=data["kept"],
                           ckpt_kind=B.HT_CKPT_INPUT)
        assert e.value.code == B.HT_ENOMEM
        B.ht_sync(c.ctx)
        assert (c.dX == 7.0).all()
        c.budget(0)
        B.ht_layer_bwd(c.ctx, c.g, DI, DN, B.HT_ACT_RELU, data["X"], data["W"][0], data["dz"], c.dW, dH_in=c.dX, H_out=data["kept"],
                       ckpt_kind=B.HT_CKPT_INPUT)
        B.ht_sync(c.ctx)
        got = c.dX[:, :DI].cpu().numpy() - 7.0
        assert_close_grad(got, c.run("bwd_recompute")["dX"], "dX")
    finally:
        c.close()
