"""Maximum size on one GPU: the largest graph of the paper's dataset table at its full scale
(65.6 M vertices, 3.6 billion edges, 128 chunks; the stand-in has the same counts), i.e. more than
2^31 stored edges and about 100 GB of graph arrays in HBM.  The partition is checked on whole
chunks against the oracle, then one layer of the widest shape (256 -> 64, ReLU) runs forward and
backward over all 128 chunks with every tensor in HBM and is checked on about 1000 sampled destination
rows, 200 sampled sources and sampled weight-gradient entries, each recomputed by the oracle in fp64 from the
same inputs.

The oracle never sees the whole graph: for the sampled rows the needed in-edges (out-edges) are cut
from the edge list with torch and relabelled to a small id space; the symmetric normalisation comes
from the full graph's in-degrees.
"""
import gc
import time

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2311_14898_amd import binding as B
from paper_2311_14898_amd import inputs
from tests.util import assert_close

pytestmark = pytest.mark.gpu
D_IN, D_OUT = 256, 64
ROWS_PER_FILL = 1 << 22


@pytest.fixture(autouse=True)
def _give_back_cached_memory():
    """torch keeps freed blocks; the library allocates with hipMalloc and needs them returned."""
    gc.collect()
    torch.cuda.empty_cache()
    yield
    gc.collect()
    torch.cuda.empty_cache()


def _randn_rows(V, d, seed):
    """[V, d] fp32 N(0,1) on the GPU, filled in slabs from a seeded generator."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    t = torch.empty((V, d), dtype=torch.float32, device="cuda")
    for r0 in range(0, V, ROWS_PER_FILL):
        r1 = min(V, r0 + ROWS_PER_FILL)
        t[r0:r1].normal_(generator=gen)
    return t


def _edges_touching(key, other, ids, V):
    """(key, other) of the edges whose `key` endpoint is one of ids, as numpy arrays."""
    table = torch.zeros(V, dtype=torch.bool, device="cuda")
    table[torch.from_numpy(ids).cuda()] = True
    k_out, o_out = [], []
    step = 1 << 29
    for e0 in range(0, key.numel(), step):
        k = key[e0:e0 + step]
        m = table[k.long()]
        k_out.append(k[m].cpu())
        o_out.append(other[e0:e0 + step][m].cpu())
    return torch.cat(k_out).numpy(), torch.cat(o_out).numpy()


def test_cfg5_full_scale_partition_and_one_layer():
    w = inputs.WORKLOADS["cfg5"]
    V, E, n = w.V, w.E, w.n_chunks
    if torch.cuda.mem_get_info()[0] < 285e9:
        pytest.skip("needs a GPU with 285 GB of free memory")
    t_start = time.perf_counter()

    def note(msg):
        print(f"[{time.perf_counter() - t_start:6.1f}s] {msg}", flush=True)

    src, dst = inputs.rmat_edges(V, E, w.graph_seed, device="cuda")
    deg = torch.bincount(dst, minlength=V)                       # in-degrees without the self-loops
    note(f"{src.numel()} edges generated")

    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src, dst, n)
    try:
        info = B.ht_graph_info_get(g)
        note(f"partitioned in {info.partition_ms:.0f} ms, {info.hbm_bytes / 1e9:.0f} GB of graph arrays")
        assert info.V == V and info.n_chunks == n and info.E_stored == E + V > 2 ** 31
        cis = [B.ht_graph_chunk_info(g, j) for j in range(n)]
        assert cis[0].dst_begin == 0 and cis[-1].dst_end == V
        assert all(cis[j].dst_end == cis[j + 1].dst_begin for j in range(n - 1))
        assert sum(c.nnz for c in cis) == E + V
        assert sum(c.n_src for c in cis) == info.v_ori and sum(c.n_load for c in cis) == info.v_load == info.v_ru
        assert all(c.n_reuse + c.n_load == c.n_src for c in cis) and cis[0].n_reuse == 0
        assert max(c.n_src for c in cis) == info.max_nsrc == info.cache_rows
        # edge balance: a boundary can overshoot its target by at most one destination's in-edges
        max_deg = int(deg.max()) + 1
        assert all(abs(c.nnz - (E + V) / n) <= 2 * max_deg for c in cis)

        # ---- whole chunks against the oracle's dedup (a late, vertex-rich chunk and the hub-heavy second one)
        for j in (1, n - 1):
            ch = B.ht_graph_export_chunk(g, j)
            ci = ch["info"]
            nd = ci.dst_end - ci.dst_begin
            d0 = deg[ci.dst_begin:ci.dst_end].cpu().numpy() + 1
            assert np.array_equal(np.diff(ch["indptr"]), d0), f"chunk {j}: in-degrees"
            o = orc.chunk_dedup(ch["indptr"], ch["col"], 0, nd)
            for k, ok in (("nbr", "N"), ("col_local", "col_local"), ("sptr", "sptr"), ("sdst", "sdst")):
                assert np.array_equal(ch[k], o[ok]), f"chunk {j}: {k}"
            prev_N = B.ht_graph_export_chunk(g, j - 1)["nbr"]
            R, Ld = orc.reuse_split(prev_N, o["N"])
            assert np.array_equal(ch["reuse"], R) and np.array_equal(ch["load"], Ld), f"chunk {j}: reuse / load"
            # a few destinations of this chunk against the raw edge list
            vs = np.unique(np.concatenate([[ci.dst_begin, ci.dst_end - 1],
                                           np.random.default_rng(j).integers(ci.dst_begin, ci.dst_end, 6)]))
            kd, ks = _edges_touching(dst, src, vs, V)
            for v in vs.tolist():
                want = np.sort(np.concatenate([ks[kd == v], [v]]))
                got = ch["col"][ch["indptr"][v - ci.dst_begin]:ch["indptr"][v - ci.dst_begin + 1]]
                assert np.array_equal(got, want), f"in-neighbours of {v}"
            note(f"chunk {j} checked ({ci.nnz} edges, {ci.n_src} sources)")
            del ch, o

        # ---- samples for the layer: destination rows with their in-edges, sources with their out-edges
        rng = np.random.default_rng(9)
        # (hubs of bounded degree: the few vertices with millions of edges would cost the CPU side minutes)
        hub_in = int(torch.argmax(torch.where(deg <= 200_000, deg, -1)))
        rows = np.unique(np.concatenate([rng.integers(1000, V, 1000), [hub_in, V - 1]]))
        e_dst, e_src = _edges_touching(dst, src, rows, V)
        odeg = torch.bincount(src, minlength=V)
        hub_out = int(torch.argmax(torch.where(odeg <= 100_000, odeg, -1)))
        del odeg
        us = np.unique(np.concatenate([rng.integers(1000, V, 200), [hub_out, V - 1]]))
        o_src, o_dst = _edges_touching(src, dst, us, V)
        del src, dst
        torch.cuda.empty_cache()
        note(f"samples cut: {len(e_dst)} in-edges of {len(rows)} rows, {len(o_src)} out-edges of {len(us)} sources")

        def s_of(ids):      # symmetric normalisation of the full graph at these vertices, by the oracle's rule
            d = deg[torch.from_numpy(ids).cuda()].cpu().numpy().astype(np.int64) + 1
            return orc.norm(np.concatenate([[0], np.cumsum(d)]))

        # ---- forward
        H = _randn_rows(V, D_IN, 21)
        Wt = inputs.glorot_weights([D_IN, D_OUT])[0]
        Wd = Wt.cuda()
        A = torch.empty((V, D_IN), dtype=torch.float32, device="cuda")
        Hout = torch.empty((V, D_OUT), dtype=torch.float32, device="cuda")
        st = B.ht_layer_fwd(ctx, g, D_IN, D_OUT, B.HT_ACT_RELU, H, Wd, Hout, A_ckpt=A, want_stats=True)
        note(f"layer forward over {n} chunks: {st.t_total_ms:.0f} ms")
        need = np.unique(np.concatenate([e_src, rows]))
        c_src = np.searchsorted(need, np.concatenate([e_src, rows])).astype(np.int32)   # self-loops appended
        c_dst = np.searchsorted(need, np.concatenate([e_dst, rows])).astype(np.int32)
        indptr_c, col_c = orc.csc_build(len(need), c_src, c_dst, add_self_loops=False)
        h_c = H[torch.from_numpy(need).cuda()].cpu().numpy()
        rows_c = np.searchsorted(need, rows)
        a_ref = orc.aggregate(indptr_c, col_c, h_c, s=s_of(need))[rows_c]
        a_dev = A[torch.from_numpy(rows).cuda()].cpu().numpy()
        assert_close(a_dev, a_ref, "a rows")
        h_out_rows = Hout[torch.from_numpy(rows).cuda()].cpu().numpy()
        assert_close(h_out_rows, np.maximum(orc.matmul(a_dev, Wt.numpy()), 0.0), "h' rows")
        note("forward rows checked")
        del h_c

        # ---- backward from the aggregate checkpoint; grad h takes H's memory (H is not read any more)
        dHout = _randn_rows(V, D_OUT, 22)
        dW = torch.zeros((D_IN, D_OUT), dtype=torch.float32, device="cuda")
        dHin = H.zero_()                              # the input gradient is accumulated into
        st = B.ht_layer_bwd(ctx, g, D_IN, D_OUT, B.HT_ACT_RELU, A, Wd, dHout, dW, dH_in=dHin, H_out=Hout,
                            want_stats=True)
        note(f"layer backward: {st.t_total_ms:.0f} ms")
        gW = dW.cpu().numpy()
        scale = np.abs(gW).max()
        for i, k in ((0, 0), (77, 5), (255, 63), (128, 31)):
            a_col = A[:, i].contiguous().cpu().numpy().astype(np.float64)
            dz_col = torch.where(Hout[:, k] > 0, dHout[:, k], torch.zeros((), device="cuda")).cpu().numpy()
            ref = float(np.dot(a_col, dz_col.astype(np.float64)))
            assert abs(gW[i, k] - ref) <= 1e-4 * scale, f"grad W[{i},{k}]: {gW[i, k]} vs {ref}"
        note("weight-gradient entries checked")
        s_us = s_of(us)
        lo, hi = torch.aminmax(dHin)                  # (no |x| temporary: the tensor is 67 GB)
        gscale = max(-float(lo), float(hi))
        for q, u in enumerate(us.tolist()):
            vs = np.concatenate([o_dst[o_src == u], [u]])
            vt = torch.from_numpy(vs).cuda()
            dz = torch.where(Hout[vt] > 0, dHout[vt], torch.zeros((), device="cuda")).cpu().numpy()
            da = orc.matmul_nt(dz, Wt.numpy())
            ref = s_us[q] * (s_of(vs)[:, None] * da).sum(axis=0)
            got = dHin[u].cpu().numpy()
            assert (np.abs(got - ref) <= 1e-4 * gscale).all(), f"grad h of source {u}"
        note("source gradients checked")
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_cfg4_full_scale_partition_with_schedule_aware_buffer():
    """The dataset shape with the most vertices (111 M, 1.6 billion edges, 64 chunks): partition with the buffer
    that releases rows only for room, 1.5 x the largest chunk's sources.  One whole chunk against the oracle's
    dedup; the buffer schedule through its invariants (the oracle's schedule needs the whole graph on the CPU)."""
    w = inputs.WORKLOADS["cfg4"]
    V, E, n = w.V, w.E, w.n_chunks
    if torch.cuda.mem_get_info()[0] < 200e9:
        pytest.skip("needs a GPU with 200 GB of free memory")
    src, dst = inputs.rmat_edges(V, E, w.graph_seed, device="cuda")
    ctx = B.ht_ctx_create(0)
    g = g2 = None
    try:
        g = B.ht_partition(ctx, V, src, dst, n)
        base = B.ht_graph_info_get(g)
        cis = [B.ht_graph_chunk_info(g, j) for j in range(n)]
        assert base.E_stored == E + V == sum(c.nnz for c in cis) and base.v_load == base.v_ru
        j = n // 2
        ch = B.ht_graph_export_chunk(g, j)
        o = orc.chunk_dedup(ch["indptr"], ch["col"], 0, ch["info"].dst_end - ch["info"].dst_begin)
        for k, ok in (("nbr", "N"), ("col_local", "col_local"), ("sptr", "sptr"), ("sdst", "sdst")):
            assert np.array_equal(ch[k], o[ok]), f"chunk {j}: {k}"
        R, Ld = orc.reuse_split(B.ht_graph_export_chunk(g, j - 1)["nbr"], o["N"])
        assert np.array_equal(ch["reuse"], R) and np.array_equal(ch["load"], Ld)
        B.ht_graph_destroy(g)
        g = None
        rows = int(1.5 * base.max_nsrc)
        g2 = B.ht_partition(ctx, V, src, dst, n, cache_rows=rows, cache_policy=B.HT_CACHE_FARTHEST)
        info = B.ht_graph_info_get(g2)
        cis = [B.ht_graph_chunk_info(g2, j) for j in range(n)]
        assert info.cache_rows == rows and info.v_ori == base.v_ori and info.v_ru == base.v_ru
        assert V <= info.v_load < base.v_load                       # every vertex is a source (self-loops)
        assert sum(c.n_load for c in cis) == info.v_load == sum(c.n_leave for c in cis)
        resident = 0
        for c in cis:
            assert c.n_reuse + c.n_load == c.n_src and c.n_reuse <= resident
            resident += c.n_load
            assert resident <= rows
            resident -= c.n_leave
        assert resident == 0
        # the rows the middle chunk finds in the buffer include those of the chunk before it
        ch2 = B.ht_graph_export_chunk(g2, j)
        assert np.array_equal(ch2["nbr"], o["N"]) and np.isin(R, ch2["reuse"]).all()
        assert np.array_equal(np.sort(np.concatenate([ch2["reuse"], ch2["load"]])), o["N"])
        print(f"rows loaded per pass: {base.v_load} (adjacent reuse) -> {info.v_load} (V = {V}), "
              f"partition {base.partition_ms:.0f} / {info.partition_ms:.0f} ms", flush=True)
    finally:
        for x in (g, g2):
            if x is not None:
                B.ht_graph_destroy(x)
        B.ht_ctx_destroy(ctx)


def test_tensors_of_more_than_2_to_32_words():
    """A launch holds fewer than 2^32 threads (a larger grid is not rejected by a plain launch, its excess is
    dropped): whole-tensor kernels must stride.  The library's fill over a 20 GiB tensor, at an address that is not
    16-byte aligned, with a ragged tail; and the per-vertex GAT kernels through a layer whose vertex count alone
    would need 2^32 threads at one wave per vertex (70 M vertices, no edges but the self-loops)."""
    if torch.cuda.mem_get_info()[0] < 120e9:
        pytest.skip("needs a GPU with 120 GB of free memory")
    ctx = B.ht_ctx_create(0)
    try:
        rows, ld = 21_000_003, 256                       # 5.4 G words
        t = torch.ones((rows, ld), dtype=torch.float32, device="cuda")
        B.ht_tensor_zero(ctx, t, ld)
        for r0 in range(0, rows, 1 << 22):
            assert not bool(t[r0:r0 + (1 << 22)].any()), f"rows from {r0} were not cleared"
        flat = torch.ones(5_000_000_007, dtype=torch.float32, device="cuda")
        view = flat[3:3 + 4_999_999_996].view(-1, 4)      # starts 12 bytes past a 16-byte boundary
        B.ht_tensor_zero(ctx, view, 4)
        assert float(flat[:3].sum()) == 3.0 and float(flat[3 + 4_999_999_996:].sum()) == 8.0
        for r0 in range(0, view.shape[0], 1 << 28):
            assert not bool(view[r0:r0 + (1 << 28)].any())
        del t, flat, view
        torch.cuda.empty_cache()
        # GAT layer on 70 M isolated vertices: softmax over the self-loop alone, so h' = relu(H W) row by row
        V, d_in, d_out = 70_000_000, 8, 4
        ids = torch.arange(0, 16, dtype=torch.int32, device="cuda")
        g = B.ht_partition(ctx, V, ids[:0], ids[:0], 64)
        try:
            H = torch.empty((V, d_in), dtype=torch.float32, device="cuda").uniform_(-1, 1, generator=torch.Generator("cuda").manual_seed(3))
            W = inputs.glorot_weights([d_in, d_out])[0].cuda()
            a = torch.full((d_out,), 0.3, device="cuda")
            out = torch.empty((V, B.pad_ld(d_out, B.HT_LOC_DEVICE)), dtype=torch.float32, device="cuda")
            B.ht_gat_layer_fwd(ctx, g, d_in, d_out, B.HT_ACT_RELU, H, W, a, a, out)
            for r0 in (0, V // 2, V - 1_000_000):          # the last range lies beyond 2^32 threads' worth of vertices
                ref = torch.relu(H[r0:r0 + 1_000_000].double() @ W.double())
                got = out[r0:r0 + 1_000_000, :d_out].double()
                assert float((got - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
        finally:
            B.ht_graph_destroy(g)
    finally:
        B.ht_ctx_destroy(ctx)


def test_layer_with_more_items_than_a_launch_holds():
    """A GCN layer, forward and backward, on 70 M isolated vertices: a wave per work item would be 4.5 G threads, more than a
    launch holds.  The aggregation over the self-loops alone is the identity: h' = relu(X W) and its gradients row by row."""
    if torch.cuda.mem_get_info()[0] < 60e9:
        pytest.skip("needs a GPU with 60 GB of free memory")
    V, d = 70_000_000, 4
    ctx = B.ht_ctx_create(0)
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    g = B.ht_partition(ctx, V, none, none, 64)
    try:
        gen = torch.Generator("cuda").manual_seed(5)
        X, dH = (torch.empty((V, d), device="cuda").uniform_(-1, 1, generator=gen) for _ in range(2))
        W = inputs.glorot_weights([d, d])[0].cuda()
        H, A = (torch.full((V, d), 7.0, device="cuda") for _ in range(2))
        dX = torch.zeros((V, d), device="cuda")            # (gradients are added to it)
        dW = torch.empty_like(W)
        B.ht_layer_fwd(ctx, g, d, d, B.HT_ACT_RELU, X, W, H, A)
        B.ht_layer_bwd(ctx, g, d, d, B.HT_ACT_RELU, A, W, dH, dW, H_out=H, dH_in=dX, ckpt_kind=B.HT_CKPT_AGG)
        B.ht_sync(ctx)
        want_dw = torch.zeros((d, d), dtype=torch.float64, device="cuda")
        for r0 in range(0, V, 10_000_000):
            x, h, dz = X[r0:r0 + 10_000_000].double(), H[r0:r0 + 10_000_000], dH[r0:r0 + 10_000_000].double()
            want = torch.relu(x @ W.double())
            # sums of 4 products of values below 1 and 0.87: fp32 rounds 8 times, each by at most 2^-24 of the largest sum, 3.5
            assert float((h.double() - want).abs().max()) <= 8 * 2.0 ** -24 * 3.5, r0
            dz = dz * (h > 0)
            assert float((dX[r0:r0 + 10_000_000].double() - dz @ W.double().t()).abs().max()) <= 8 * 2.0 ** -24 * 3.5, r0
            want_dw += x.t() @ dz
        # 70 M products below 1: each fp32 partial sum is off by at most 2^-24 of a partial sum; far below 1e-4 of the largest entry
        # plus what independent signs leave of the sum (sqrt(V / 18))
        scale = float(want_dw.abs().max()) + (V / 18) ** 0.5
        assert float((dW.double() - want_dw).abs().max()) <= 1e-4 * scale
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_chunk_pass_with_more_than_2_31_chunk_sources():
    """129 chunks that all name each of 2^24 sources: 2^31 + 2^24 (chunk, source) pairs, so positions in the arena of neighbour
    lists need 32 bits.  The backward pass through the gradient buffer finds every row's vertex and buffer position by them."""
    if torch.cuda.mem_get_info()[0] < 240e9:
        pytest.skip("needs a GPU with 240 GB of free memory")
    V, k, d = 1 << 24, 129, 4
    E = V * k
    src, dst = torch.empty(E, dtype=torch.int32, device="cuda"), torch.empty(E, dtype=torch.int32, device="cuda")
    for e0 in range(0, E, V):                          # edge e: e mod V -> e / k; a chunk holds V edges in a row, all sources once
        e = torch.arange(e0, e0 + V, device="cuda")
        src[e0:e0 + V], dst[e0:e0 + V] = e % V, torch.div(e, k, rounding_mode="floor")
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src, dst, k, add_self_loops=False)
    try:
        del src, dst, e
        assert B.ht_graph_info_get(g).v_ori >= 1 << 31
        gen = torch.Generator("cuda").manual_seed(6)
        A, dH = (torch.empty((V, d), device="cuda").uniform_(-1, 1, generator=gen) for _ in range(2))
        W = inputs.glorot_weights([d, d])[0].cuda()
        dX, dW = torch.zeros((V, d), device="cuda"), torch.empty_like(W)
        B.ht_layer_bwd(ctx, g, d, d, B.HT_ACT_NONE, A, W, dH, dW, dH_in=dX, ckpt_kind=B.HT_CKPT_AGG, gather_mode=B.HT_GATHER_BUFFER)
        B.ht_sync(ctx)
        da = dH.double() @ W.double().t()
        want = torch.zeros_like(da)
        u = torch.arange(V, device="cuda")
        for j in range(k):                             # every vertex has k in-edges: both factors of the normalisation are k^-1/2
            want += da[torch.div(u + j * V, k, rounding_mode="floor")] / k
        # k products of values below 2 / k, rounded twice each and once more per addition
        assert float((dX.double() - want).abs().max()) <= (k + 4) * 2.0 ** -24 * 2
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)


def test_partition_with_more_bitmap_words_than_a_launch_holds():
    """2^30 vertices in 257 chunks: a thread per word of every chunk's neighbour bitmap would be more than a launch holds.  Edges
    v -> v + 1 alone, so that every list is known: chunk j's sources are its destinations and the one before, which the chunk
    before it also reads."""
    if torch.cuda.mem_get_info()[0] < 200e9:
        pytest.skip("needs a GPU with 200 GB of free memory")
    V, n = 1 << 30, 257
    src = torch.arange(V - 1, dtype=torch.int32, device="cuda")
    ctx = B.ht_ctx_create(0)
    g = B.ht_partition(ctx, V, src, src + 1, n, balance_mode=B.HT_BALANCE_VERTICES, reorder_chunks=True)
    try:
        del src
        info = B.ht_graph_info_get(g)
        assert info.v_ori == V + n - 1 and info.v_ru == info.v_load == V
        assert np.array_equal(B.ht_graph_chunk_order(g), np.arange(n))
        for j in (0, 1, 128, n - 1):                      # (the last chunk's words lie beyond 2^32 threads)
            ch = B.ht_graph_export_chunk(g, j)
            b0, b1 = j * V // n, (j + 1) * V // n
            first = max(b0 - 1, 0)
            assert np.array_equal(ch["nbr"], np.arange(first, b1)), j
            assert np.array_equal(ch["reuse"], np.arange(first, b0)) and np.array_equal(ch["load"], np.arange(b0, b1)), j
            assert np.array_equal(ch["leave"], np.arange(first, b1 - 1 if j < n - 1 else b1)), j
            assert np.array_equal(ch["nbr"][ch["col_local"]], ch["col"]), j
    finally:
        B.ht_graph_destroy(g)
        B.ht_ctx_destroy(ctx)
