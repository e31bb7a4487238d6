"""The work a user of this library has it do, as cases that can be timed and whose outputs can be compared.

Five kinds of pass, each through the public calls of paper_2311_14898_amd.binding:

  gcn        one GCN training epoch (ht_epoch): forward, loss, backward, SGD step
  gat        one GAT training epoch (ht_gat_epoch)
  layer      one GCN layer forward with its checkpoint, then its backward (ht_layer_fwd, ht_layer_bwd): a training loop
             that a program composes by itself
  static     one layer forward through the call that allocates nothing (ht_layer_fwd_static): serving loops
  partition  a graph that is seen once: ht_partition, one layer forward over it, ht_graph_destroy

Graphs are the repository's seeded R-MAT graphs (power-law degrees, duplicate edges kept, one self-loop per vertex added),
features are N(0, 1), labels uniform, weights Glorot-uniform; everything is fp32, as everywhere in the library.
"""
import math

import torch

from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs

LR = 0.01


def listed():
    return [
        # The smallest epoch of the repository's workloads: every kernel is short, launches and host work count.
        dict(name="gcn_epoch_10k", kind="gcn", V=10_000, E=100_000, dims="64-32-8", chunks=4),
        # The headline workload: two layers on a dense power-law graph, everything in HBM, the printed stage order.
        dict(name="gcn_epoch_233k_115M", kind="gcn", V=232_965, E=114_600_000, dims="602-256-41", chunks=8),
        # The same shape at half the size with odd widths, the planner free to transform before it aggregates.
        dict(name="gcn_epoch_auto_order", kind="gcn", V=116_483, E=57_300_000, dims="301-129-47", chunks=7, order="auto"),
        # Three layers on a sparse graph of many vertices, in HBM.
        dict(name="gcn_epoch_2M_62M", kind="gcn", V=2_450_000, E=61_900_000, dims="100-256-256-47", chunks=16),
        # The same graph shape at a quarter of the size, h and grad h in pinned host memory, adjacent-chunk reuse.
        dict(name="gcn_epoch_host", kind="gcn", V=612_500, E=15_475_000, dims="100-256-256-47", chunks=16, host=True),
        # Attention: a small ragged epoch, and the headline graph.
        dict(name="gat_epoch_20k", kind="gat", V=20_011, E=300_007, dims="50-33-7", chunks=3),
        dict(name="gat_epoch_233k_115M", kind="gat", V=232_965, E=114_600_000, dims="602-256-41", chunks=8),
        # A program's own loop over layers: ragged widths with the aggregate kept, and recomputation from the layer input.
        dict(name="layer_60k_ragged", kind="layer", V=60_013, E=3_000_017, dims="129-67", chunks=5, recompute=False),
        dict(name="layer_1M_recompute", kind="layer", V=1_000_003, E=20_000_003, dims="64-64", chunks=16, recompute=True),
        # A serving loop's forward.
        dict(name="static_20k", kind="static", V=20_000, E=400_000, dims="128-64", chunks=4),
        # Graphs that are seen once: a small one, where launches and host work count, and a large one.
        dict(name="partition_10k", kind="partition", V=10_000, E=100_000, dims="64-32", chunks=4),
        dict(name="partition_2M_62M", kind="partition", V=2_450_000, E=61_900_000, dims="100-47", chunks=16),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the same kinds, sizes over the ranges the listed ones span."""
    kind = rng.choice(["gcn", "gcn", "gcn", "gat", "layer", "layer", "static", "partition"])
    host = kind == "gcn" and rng.random() < 0.25
    top_v, top_e = (25_000, 500_000) if kind == "static" else (600_000, 15_000_000) if host else (2_000_000, 60_000_000)
    V = _log_uniform(rng, 3_000, top_v)
    E = max(1_000, min(top_e, int(V * math.exp(rng.uniform(math.log(6), math.log(500))))))
    chunks = rng.randint(1, 4 if V < 30_000 else 16)
    wide = 128 if kind == "static" else 256 if V > 400_000 else 602
    layers = {"gcn": rng.choice([2, 2, 3]), "gat": 2}.get(kind, 1)
    dims = [_log_uniform(rng, 16, wide)] + [_log_uniform(rng, 16, min(wide, 256)) for _ in range(layers - 1)] + [_log_uniform(rng, 5, 128)]
    case = dict(kind=kind, V=V, E=E, dims="-".join(map(str, dims)), chunks=chunks)
    if kind == "gcn":
        case.update(host=host, order="auto" if not host and rng.random() < 0.3 else "printed",
                    labelled_one_in=rng.choice([1, 1, 1, 100]), far=host and rng.random() < 0.5)
    if kind == "layer":
        case.update(recompute=rng.random() < 0.4)
    return case


def _dims(case):
    return [int(x) for x in case["dims"].split("-")]


_serving = []


def _serving_stream():
    """The one stream of the serving loops: calls that allocate nothing share the library's static scratch memory, so they
    must not overlap."""
    if not _serving:
        _serving.append(torch.cuda.Stream())
    return _serving[0].cuda_stream


class State:
    """A context, what the case keeps beside it, and their release."""

    def __init__(self, case):
        self.case = case
        self.dims = _dims(case)
        self.ctx = B.ht_ctx_create(0, _serving_stream() if case["kind"] == "static" else None)
        self.graph = None

    def __del__(self):
        if self.graph is not None:
            B.ht_graph_destroy(self.graph)
        if self.ctx is not None:
            B.ht_ctx_destroy(self.ctx)
        self.graph = self.ctx = None


def _normal(rows, cols, g):
    """[rows x cols] of N(0, 1) in HBM at the library's row pitch."""
    m = B.alloc_matrix(rows, cols)
    m[:, :cols] = torch.randn(rows, cols, generator=g, device="cuda")
    return m


def prepare(case, seed):
    s = State(case)
    V, dims, kind = case["V"], s.dims, case["kind"]
    src, dst = inputs.rmat_edges(V, case["E"], seed=seed + 1, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 2)
    s.X = _normal(V, dims[0], g)
    s.W = [w.cuda() for w in inputs.glorot_weights(dims, seed=seed + 4)]
    if kind == "partition":
        s.src, s.dst = src, dst
        s.H = B.alloc_matrix(V, dims[1])
        return s
    s.graph = B.ht_partition(s.ctx, V, src, dst, case["chunks"],
                             cache_policy=B.HT_CACHE_FARTHEST if case.get("far") else B.HT_CACHE_ADJACENT)
    if kind in ("gcn", "gat"):
        s.y = torch.randint(0, dims[-1], (V,), generator=g, device="cuda").to(torch.int32)
        k = case.get("labelled_one_in", 1)
        if k > 1:
            s.y[torch.randint(0, k, (V,), generator=g, device="cuda") != 0] = -1
            s.y[0] = 0                                     # at least one labelled vertex
    if kind == "gcn":
        s.options = dict(order=B.HT_ORDER_AUTO if case.get("order") == "auto" else B.HT_ORDER_AGG_FIRST)
        if case.get("host"):
            s.options.update(res_h=B.HT_RES_HOST, res_g=B.HT_RES_HOST)
    if kind == "gat":
        a_dst, a_src = inputs.attention_vectors(dims, seed=seed + 5)
        s.a_dst, s.a_src = [a.cuda() for a in a_dst], [a.cuda() for a in a_src]
    if kind in ("layer", "static"):
        s.H, s.A = B.alloc_matrix(V, dims[1]), B.alloc_matrix(V, dims[0])
    if kind == "layer":
        # The backward pass takes ReLU's mask from activations drawn here: about one in 10^7 signs of H hangs on the last bit
        # of an fp32 sum, and each would move a gradient by more than all rounding together.
        s.kept = _normal(V, dims[1], g).clamp_(min=0.0)
        s.dH = _normal(V, dims[1], g)
        s.dX = B.alloc_matrix(V, dims[0])
        s.dW = torch.empty_like(s.W[0])
    return s


def run(s):
    case, dims, kind = s.case, s.dims, s.case["kind"]
    if kind == "gcn":
        loss, _ = B.ht_epoch(s.ctx, s.graph, dims, s.W, LR, s.X, s.y, **s.options)
        return {"loss": loss, "W": s.W}
    if kind == "gat":
        loss, _ = B.ht_gat_epoch(s.ctx, s.graph, dims, s.W, s.a_dst, s.a_src, LR, s.X, s.y)
        return {"loss": loss, "W": s.W, "a_dst": s.a_dst, "a_src": s.a_src}
    if kind == "static":
        B.ht_layer_fwd_static(s.ctx, s.graph, dims[0], dims[1], B.HT_ACT_RELU, s.X, s.W[0], s.H, s.A)
        return {"H": s.H[:, :dims[1]], "A": s.A[:, :dims[0]]}
    if kind == "layer":
        again = case["recompute"]                          # nothing kept: the backward pass aggregates again
        B.ht_layer_fwd(s.ctx, s.graph, dims[0], dims[1], B.HT_ACT_RELU, s.X, s.W[0], s.H, None if again else s.A)
        s.dX.zero_()
        B.ht_layer_bwd(s.ctx, s.graph, dims[0], dims[1], B.HT_ACT_RELU, s.X if again else s.A, s.W[0], s.dH, s.dW, dH_in=s.dX,
                       H_out=s.kept, ckpt_kind=B.HT_CKPT_INPUT if again else B.HT_CKPT_AGG)
        out = {"H": s.H[:, :dims[1]], "dW": s.dW, "dX": s.dX[:, :dims[0]]}
        return out if again else dict(out, A=s.A[:, :dims[0]])
    graph = B.ht_partition(s.ctx, case["V"], s.src, s.dst, case["chunks"])
    info = B.ht_graph_info_get(graph)
    B.ht_layer_fwd(s.ctx, graph, dims[0], dims[1], B.HT_ACT_RELU, s.X, s.W[0], s.H)
    B.ht_sync(s.ctx)
    B.ht_graph_destroy(graph)
    return {"H": s.H[:, :dims[1]], "volumes": [int(info.v_ori), int(info.v_ru), int(info.v_load), int(info.cache_rows)]}


def work(case):
    """Inputs read once, outputs written once; multiply-adds of the aggregations (per stored edge) and of the dense products."""
    V, dims, kind = case["V"], _dims(case), case["kind"]
    edges = case["E"] + V
    weights = sum(a * b for a, b in zip(dims, dims[1:]))
    topology = 8 * case["E"] if kind == "partition" else 4 * edges + 8 * V
    if kind in ("gcn", "gat"):
        tensors = V * (dims[0] + 1) + 2 * weights
        widths = dims[1:] if kind == "gat" else [min(a, b) if case.get("order") == "auto" else a for a, b in zip(dims, dims[1:])]
        passes = [3] * len(widths) if kind == "gat" else [1] + [2] * (len(widths) - 1)      # layer 0 has no input gradient
        agg = sum(p * 2 * edges * w for p, w in zip(passes, widths))
        dense = sum((2 if i == 0 else 3) * 2 * V * a * b for i, (a, b) in enumerate(zip(dims, dims[1:])))
    else:
        both = kind == "layer"
        tensors = V * (dims[0] + dims[1]) + weights
        if kind == "static" or (both and not case["recompute"]):
            tensors += V * dims[0]                                                          # the aggregate is an output
        if both:
            tensors += V * (dims[0] + dims[1]) + weights
        agg = (2 if both else 1) * 2 * edges * dims[0]
        dense = (3 if both else 1) * 2 * V * dims[0] * dims[1]
    return {"bytes": topology + 4 * tensors, "flops": agg + dense}


def tolerance(case):
    """Four times what other orders of the same fp32 sums showed (full rows per wave; duplicates not merged, with work items of
    another length), three passes each: layers up to rel 2.6e-7 and max 2.2e-6, epochs (their loss and updated weights) up to
    one unit of rounding, 1.2e-7.  An epoch's max leaves room for one ReLU derivative that fp32 cannot decide."""
    if case["kind"] in ("gcn", "gat"):
        return {"rel": 5e-7, "max": 4e-6}
    return {"rel": 1e-6, "max": 1e-5}
