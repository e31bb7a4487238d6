// Per-chunk layer step, forward and backward, and the epoch built from it.
//
//   forward  (Alg. 1, Alg. 2, Eq. 2): neighbour rows reach
//            the aggregation either in place (tensor in HBM) or through the
//            in-place neighbour buffer (reused rows stay, new rows are fetched
//            from HBM or pinned host memory); aggregate; linear + ReLU; rows
//            of a^l and h^{l+1} go to their homes.
//   backward (Alg. 1, Alg. 3, Sec. 2.3, Sec. 4.2): reload
//            the checkpoint, recompute the update stage, grad W, grad a,
//            aggregate backward by source; neighbour gradients accumulate in HBM
//            while their vertex stays buffered and leave to the gradient home
//            (CPU-side add when that home is host memory).
#include <algorithm>
#include <atomic>
#include <cstring>
#include <condition_variable>
#include <mutex>
#include <thread>

#include "ht_internal.h"

struct EpochWs {
  int64_t V = 0;
  std::vector<int32_t> dims;
  int res_h = 0, res_a = 0, res_g = 0;
  bool no_ckpt = false;              // pure recomputation: no a^l for any layer
  uint32_t upd_mask = 0;             // bit l: layer l runs update-first (no a^l is kept for it)
  std::vector<ht_tensor> h, a, gh;  // h[l] = h^l (l >= 1; h[0] unused), a[l], gh[l] = grad h^l (l >= 1)
  std::vector<float*> dW;
  std::vector<size_t> dev_bytes_of;  // for freeing
  std::vector<void*> dev_ptrs;
  std::vector<void*> host_ptrs;
  const float* a0_of = nullptr;      // a[0] holds A_hat X for the X at this address (nullptr: not valid)
  uint64_t a0_graph = 0;             // ... and for the graph with this serial number
  // HIP graph of one epoch's stream work (all tensors in HBM): what it was captured for, and the
  // key of the last epoch that ran eagerly to the end (its scratch sizes are what the capture needs)
  std::vector<uintptr_t> graph_key, warm_key, bad_key;   // bad_key: a capture of this key failed, it stays eager
  hipGraphExec_t graph_exec = nullptr;
};

namespace {

__global__ void k_noop() {}

int check_tensor(ht_ctx* ctx, const ht_tensor* t, int64_t rows, int32_t cols, const char* name) {
  if (!t || !t->ptr) return ht_set_err(ctx, HT_EINVAL, "%s: null tensor", name);
  if (t->rows != rows || t->cols != cols)
    return ht_set_err(ctx, HT_ESHAPE, "%s: shape [%lld x %d], expected [%lld x %d]", name, (long long)t->rows, t->cols,
                      (long long)rows, cols);
  if (t->ld < t->cols || (t->ld & 3))
    return ht_set_err(ctx, HT_ESHAPE, "%s: row pitch %lld must be >= cols and a multiple of 4", name, (long long)t->ld);
  if (t->loc != HT_LOC_DEVICE && t->loc != HT_LOC_HOST_PINNED)
    return ht_set_err(ctx, HT_ESHAPE, "%s: unknown location %d", name, t->loc);
  if ((uintptr_t)t->ptr & 15) return ht_set_err(ctx, HT_ESHAPE, "%s: base pointer must be 16-byte aligned", name);
  return HT_OK;
}

// Pointer the GPU can dereference.
int gpu_ptr(ht_ctx* ctx, const ht_tensor* t, float** out) {
  if (t->loc == HT_LOC_DEVICE) {
    *out = t->ptr;
    return HT_OK;
  }
  void* d = nullptr;
  hipError_t e = hipHostGetDevicePointer(&d, t->ptr, 0);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return ht_set_err(ctx, HT_ESHAPE, "host tensor is not page-locked / GPU-addressable: %s", hipGetErrorString(e));
  }
  *out = (float*)d;
  return HT_OK;
}

int host_threads(ht_ctx* ctx) {
  if (ctx->n_threads <= 0) {
    unsigned hc = std::thread::hardware_concurrency();
    ctx->n_threads = (int)std::min<unsigned>(hc ? hc : 4u, 16u);
  }
  return ctx->n_threads;
}

// grad[ids[k]] += rows[k] on the host cores (Alg. 3); ids are unique.
void cpu_accumulate(ht_ctx* ctx, float* grad, int64_t ld, const int32_t* ids, const float* rows, int64_t rows_ld,
                    int64_t n, int d) {
  const int nt = (int)std::min<int64_t>(host_threads(ctx), std::max<int64_t>(1, n / 256));
  auto work = [&](int64_t k0, int64_t k1) {
    for (int64_t k = k0; k < k1; ++k) {
      float* g = grad + (int64_t)ids[k] * ld;
      const float* r = rows + k * rows_ld;
      for (int c = 0; c < d; ++c) g[c] += r[c];
    }
  };
  if (nt <= 1) {
    work(0, n);
    return;
  }
  std::vector<std::thread> th;
  const int64_t per = (n + nt - 1) / nt;
  for (int t = 0; t < nt; ++t) {
    const int64_t k0 = t * per, k1 = std::min<int64_t>(n, k0 + per);
    if (k0 < k1) th.emplace_back(work, k0, k1);
  }
  for (auto& t : th) t.join();
}

struct Run {
  ht_ctx* ctx;
  const ht_graph* g;
  Timer tm;
  ht_stats* st;  // never null inside (a local one is used when the caller passes none)
  int layer = 0; // index into the per-layer statistics
  bool dhin_fresh = false;  // dH_in counts as zeros: a host tensor holds them (leaving rows may be stored, not added), a device
                            // tensor holds anything and every row is written or cleared first
  bool planned = false;     // one of many passes over this graph: it may make and use the graph's plan (ht_dense.hip)
  // An aggregate that no tensor keeps is made again by the backward pass and must be the same there, to the last bit: ReLU's mask and grad W
  // belong to the activations that the forward pass has returned.  It takes the plan only inside an epoch whose tensors are all in HBM
  // (again_ok), and the layers in which it did are noted for the backward pass.
  bool again_ok = false;
  std::vector<char> again;
  bool made_planned() const { return (size_t)layer < again.size() && again[layer]; }
  void note_planned(bool yes) {
    if ((size_t)layer >= again.size()) again.resize((size_t)layer + 1);
    again[layer] = yes;
  }
  bool changed = false;     // the caller's gradients may have been added to: the call cannot be made again
  Run(ht_ctx* c, const ht_graph* gr, ht_stats* s, bool timed) : ctx(c), g(gr), tm(c, c->stream, timed), st(s) {}
};

double spmm_alg_bytes(const ChunkMeta& c, int d) {
  const double nd = (double)(c.dst1 - c.dst0);
  return 4.0 * c.nnz + 8.0 * nd + 4.0 * d * (double)c.nsrc + 4.0 * d * nd + 4.0 * ((double)c.nsrc + nd);
}

// Streams of the per-chunk pipeline: compute on the context's stream, neighbour
// gather / H2D row copies on side[0], D2H row copies on side[1], host functions
// (CPU-side gradient accumulation) on side[2].  Stages are ordered by events.
struct Pipe {
  ht_ctx* ctx;
  hipStream_t s_c, s_in, s_out, s_host;
  bool used_in = false, used_out = false, used_host = false;
  explicit Pipe(ht_ctx* c) : ctx(c), s_c(c->stream), s_in(c->side[0]), s_out(c->side[1]), s_host(c->side[2]) {}
  // A failed call must not leave side-stream work that refers to the caller's locals.
  ~Pipe() {
    if (used_in) (void)hipStreamSynchronize(s_in);
    if (used_out) (void)hipStreamSynchronize(s_out);
    if (used_host) (void)hipStreamSynchronize(s_host);
  }
  int rec(hipStream_t s, hipEvent_t* out) {
    hipEvent_t e = ht_event(ctx);
    if (!e) return ht_set_err(ctx, HT_EHIP, "hipEventCreate failed");
    HT_HIP(ctx, hipEventRecord(e, s));
    *out = e;
    return HT_OK;
  }
  int wait(hipStream_t s, hipEvent_t e) {
    if (!e) return HT_OK;
    HT_HIP(ctx, hipStreamWaitEvent(s, e, 0));
    return HT_OK;
  }
};

// Rows of N_j \ N_{j-1} from H_in (HBM or pinned host, read in place by the
// kernel) into their positions of the in-place neighbour buffer, scaled by s_u
// on the way (Alg. 2).
int gather_chunk(Run& R, int j, const ht_tensor* H_in, const float* Hin, int d, float* nbuf, hipStream_t st) {
  const ht_graph* g = R.g;
  const ChunkMeta& c = g->chunks[j];
  const int id = R.tm.begin_on(&R.st->t_gather_ms, st);
  HT_TRY(ht_gather_rows(R.ctx, st, Hin, H_in->ld, g->load.p + c.load_off, nbuf, H_in->ld, g->load_slot.p + c.load_off,
                        c.n_load, d, g->s.p, H_in->loc == HT_LOC_HOST_PINNED ? R.ctx->gather_blocks : 0));
  R.tm.end_id(id);
  R.st->rows_loaded += c.n_load;
  R.st->rows_reused += c.n_reuse;
  if (H_in->loc == HT_LOC_HOST_PINNED) R.st->bytes_h2d += (int64_t)c.n_load * d * 4;
  R.st->bytes_h2d_nodedup += (int64_t)c.nsrc * d * 4;
  return HT_OK;
}

// The graph's entries for an aggregation: forward (rows = destinations, entries name sources by global id or by buffer
// position) or backward (rows = positions of the N arena, entries name destination rows of their chunk).
void agg_entries(const ht_graph* g, bool fwd, bool buffer, SpmmArgs* a) {
  if (g->merged) {
    a->idx = !fwd ? g->usdst.p : buffer ? g->ucol_slot.p : g->ucol.p;
    a->w_edge = !fwd ? g->uw_bwd.p : buffer ? g->umult.p : g->uw_fwd.p;
  } else {
    a->idx = !fwd ? g->sdst.p : buffer ? g->col_slot.p : g->col.p;
    a->ew = (!fwd || buffer) ? nullptr : g->s.p;
  }
}
void agg_items(const GraphItems& gi, const ItemRange& r, SpmmArgs* a) {
  a->items = gi.items.p + r.it0; a->n_items = r.n_items;
  a->cuts = gi.cuts.p + r.cut0; a->n_fix = r.n_cut;
  a->part0 = r.part0;
}
// ... and those of chunk c
void agg_args(const ht_graph* g, const ChunkMeta& c, bool fwd, bool buffer, SpmmArgs* a) {
  agg_items(fwd ? g->fwd_items : g->bwd_items, fwd ? c.fwd : c.bwd, a);
  agg_entries(g, fwd, buffer, a);
  if (!fwd && !g->merged) a->ew = g->s.p + c.dst0;
  a->row0 = fwd ? c.dst0 : c.nbr_off;
  a->n_edges = g->merged ? c.nu : c.nnz;
}

// Aggregate of chunk j into out rows [0, ndst) (pitch out_ld) on the compute
// stream.  src/src_ld: H_in read in place, or the neighbour buffer (rows already
// scaled by s_u, indexed by buffer position).
int spmm_chunk(Run& R, int j, bool buffer, const float* src, int64_t src_ld, int d, float* out, int64_t out_ld) {
  ht_ctx* ctx = R.ctx;
  const ht_graph* g = R.g;
  const ChunkMeta& c = g->chunks[j];
  hipStream_t st = ctx->stream;
  float* partial = nullptr;
  if (c.fwd.n_part > 0) HT_TRY(ht_scratch(ctx, HT_S_SPART, (size_t)g->max_fpart * out_ld * 4, (void**)&partial));
  SpmmArgs a{};
  agg_args(g, c, true, buffer, &a);
  a.src = src;
  a.src_ld = src_ld;
  a.d = d;
  a.out = out; a.out_ld = out_ld; a.out_idx = nullptr;
  a.post = g->s.p; a.post_idx = nullptr;
  a.accumulate = 0;
  a.partial = partial;
  a.max_slabs = ctx->slabs_fwd;
  const int li = R.layer < HT_MAX_LAYERS ? R.layer : HT_MAX_LAYERS - 1;
  a.tm = &R.tm;
  a.t_items = &R.st->t_agg_fwd_layer_ms[li];
  a.t_fix = &R.st->t_agg_fix_ms;
  HT_TRY(ht_spmm_launch(ctx, st, a));
  R.st->n_spmm_fwd += 1;
  R.st->n_agg_fwd_layer[li] += 1;
  R.st->edges += c.nnz;
  R.st->spmm_fwd_alg_bytes += spmm_alg_bytes(c, d);
  R.st->agg_fwd_layer_alg_bytes[li] += spmm_alg_bytes(c, d);
  return HT_OK;
}

// ---- all chunks at once.  With the rows that an aggregation reads in HBM and no neighbour buffer between chunks, nothing
// orders one chunk before another: the chunks' work items run as one launch (a launch per chunk leaves the GPU short of
// waves at its ends and costs its latency: an epoch on 10,000 vertices in 4 chunks 311 -> 203 us, on 2.45 M vertices in 16
// chunks 72.1 -> 65.7 ms; a forward of 20,000 vertices in 4 chunks 96 -> 42 us).  A range of chunks in vertex order is closed early only where its partial sums
// (or the aggregates, when no tensor keeps them) would take more scratch memory than this.
constexpr int64_t HT_RANGE_BYTES = (int64_t)2 << 30;

struct ChunkRange {
  int k0, k1;                // chunk ids
  ItemRange items;
  int64_t row0, rows, edges, entries;
};

// part_bytes, row_bytes: scratch memory per partial sum and per row (0: none)
std::vector<ChunkRange> chunk_ranges(const ht_graph* g, int64_t part_bytes, int64_t row_bytes, int64_t cap) {
  std::vector<ChunkRange> out;
  for (int k = 0; k < g->n; ++k) {
    const ChunkMeta& c = g->chunks[g->pos[k]];
    const int64_t rows = c.dst1 - c.dst0;
    if (rows == 0) continue;
    if (!out.empty()) {
      ChunkRange& r = out.back();
      if ((r.items.n_part + c.fwd.n_part) * part_bytes + (r.rows + rows) * row_bytes <= cap) {
        r.k1 = k + 1;
        r.items.n_items += c.fwd.n_items;
        r.items.n_part += c.fwd.n_part;
        r.items.n_cut += c.fwd.n_cut;
        r.rows += rows;
        r.edges += c.nnz;
        r.entries += g->merged ? c.nu : c.nnz;
        continue;
      }
    }
    out.push_back(ChunkRange{k, k + 1, c.fwd, c.dst0, rows, c.nnz, g->merged ? c.nu : c.nnz});
  }
  return out;
}

ChunkRange whole_graph(const ht_graph* g) {
  ChunkRange r{0, g->n, ItemRange{}, 0, g->V, g->Ep, g->merged ? g->n_unique : g->Ep};
  r.items.n_items = g->fwd_items.n_items;
  r.items.n_part = g->fwd_items.n_part;
  r.items.n_cut = g->fwd_items.n_cut;
  return r;
}

// compulsory bytes of one launch over `rows` destination rows that may name every vertex
double agg_all_bytes(const ht_graph* g, int64_t edges, int64_t rows, int d) {
  return 4.0 * edges + 8.0 * rows + 4.0 * d * (double)g->V + 4.0 * d * (double)rows + 4.0 * ((double)g->V + (double)rows);
}

// Scratch memory up to which a planned pass keeps partial sums.  (8 GiB of them in items of 48 entries are up to 12 in items of 32: a graph's rule for the length asks for no width.
// 100 k vertices, 4.6 M entries left, 18,000 columns, 10.8 GB of sums: a forward pass 35.6 ms over the plan, 44.3 without.)
constexpr int64_t HT_PLAN_BYTES = (int64_t)12 << 30;

// What a pass over rows of d columns at pitch src_ld, partial sums at pitch ld, takes of the graph's plan, and the scratch memory of that; nothing
// where there is none or no memory for it.
int take_plan(Run& R, bool fwd, int d, int64_t src_ld, int64_t ld, PassPlan* out) {
  ht_ctx* ctx = R.ctx;
  *out = PassPlan();
  if (!R.planned || ctx->agg_variant != 0) return HT_OK;
  PassPlan p;
  HT_TRY(ht_pass_plan(ctx, R.g, fwd, d, src_ld, &p));
  const int64_t part_bytes = p.parts() * ld * 4;
  if (!p.items || part_bytes > HT_PLAN_BYTES) return HT_OK;
  if (ctx->scratch_bytes[HT_S_SPART] < (size_t)part_bytes && ht_caller_captures(ctx)) return HT_OK;
  const int rc = ht_scratch_all(ctx, {{HT_S_SPART, (size_t)part_bytes}});
  if (rc == HT_OK) *out = p;
  return rc == HT_ENOMEM ? (int)HT_OK : rc;
}
// The pass's launches, `a` being those of the unplanned pass over the whole graph with the partial sums in place.
int planned_launch(Run& R, const PassPlan& p, SpmmArgs a) {
  const ht_graph* g = R.g;
  if ((size_t)(p.parts() * a.out_ld) * 4 > R.ctx->scratch_bytes[HT_S_SPART])
    return ht_set_err(R.ctx, HT_ESTATE, "aggregation: %lld partial sums of %lld floats, more than their slot was asked for", (long long)p.parts(), (long long)a.out_ld);
  a.items = p.items->items.p; a.n_items = p.items->n_items;
  a.cuts = p.items->cuts.p; a.n_fix = p.items->n_cut;
  a.part0 = 0;
  a.row0 = 0;
  a.units = true;
  a.src_rows = g->V;
  if (p.dense) {
    const DenseSide& D = *p.dense;
    a.n_edges = D.n_rest;
    a.idx = D.idx.p;
    a.w_edge = D.w.p;
    a.dense_pos = D.pos.p; a.dense_seg0 = D.seg0.p;
    a.dense_part = p.items->n_part;
    if (a.tm && a.t_items) a.tm->begin(a.t_items);
    HT_TRY(ht_dense_launch(R.ctx, R.ctx->stream, D, a.src, a.src_ld, g->s.p, a.d, a.partial + p.items->n_part * a.out_ld, a.out_ld));
    if (a.tm && a.t_items) a.tm->end();
  }
  return ht_spmm_launch(R.ctx, R.ctx->stream, a);
}

// Aggregate of one range of chunks, rows of src read in place by vertex id, into out (row of the range's first destination).
int agg_range(Run& R, const ChunkRange& r, const float* src, int64_t src_ld, int d, float* out, int64_t out_ld, int relu, float* partial,
              const PassPlan& plan = PassPlan()) {   // (a plan's range is the whole graph)
  const ht_graph* g = R.g;
  SpmmArgs a{};
  agg_items(g->fwd_items, r.items, &a);
  agg_entries(g, true, false, &a);
  a.row0 = r.row0;
  a.n_edges = r.entries;
  a.src = src; a.src_ld = src_ld; a.d = d;
  a.out = out; a.out_ld = out_ld;
  a.post = g->s.p;
  a.relu = relu;
  a.partial = partial;
  a.max_slabs = R.ctx->slabs_fwd;
  const int li = R.layer < HT_MAX_LAYERS ? R.layer : HT_MAX_LAYERS - 1;
  a.tm = &R.tm;
  a.t_items = &R.st->t_agg_fwd_layer_ms[li];
  a.t_fix = &R.st->t_agg_fix_ms;
  HT_TRY(plan.items ? planned_launch(R, plan, a) : ht_spmm_launch(R.ctx, R.ctx->stream, a));
  int64_t live = 0;          // chunk aggregations, whatever number of launches they take
  for (int k = r.k0; k < r.k1; ++k) live += g->bounds[k + 1] > g->bounds[k];
  R.st->n_spmm_fwd += live;
  R.st->n_agg_fwd_layer[li] += live;
  R.st->edges += r.edges;
  const double bytes = agg_all_bytes(g, r.edges, r.rows, d);
  R.st->spmm_fwd_alg_bytes += bytes;
  R.st->agg_fwd_layer_alg_bytes[li] += bytes;
  return HT_OK;
}

int64_t most_parts(const std::vector<ChunkRange>& ranges) {
  int64_t parts = 0;
  for (const ChunkRange& r : ranges) parts = std::max(parts, r.items.n_part);
  return parts;
}

// Aggregates of all destinations: out row = vertex.  `plan`: what was taken of the graph's plan, with its scratch memory.
int agg_all(Run& R, const float* src, int64_t src_ld, int d, float* out, int64_t out_ld, int relu, const PassPlan& plan) {
  if (plan.items) return agg_range(R, whole_graph(R.g), src, src_ld, d, out, out_ld, relu, (float*)R.ctx->scratch[HT_S_SPART], plan);
  auto ranges = chunk_ranges(R.g, out_ld * 4, 0, ht_may_spend(R.ctx) ? HT_RANGE_BYTES : 0);
  int64_t parts = most_parts(ranges);
  const int rc = ht_scratch_all(R.ctx, {{HT_S_SPART, (size_t)(parts * out_ld) * 4}});
  if (rc == HT_ENOMEM) {   // less memory at a time: chunk by chunk
    ranges = chunk_ranges(R.g, out_ld * 4, 0, 0);
    parts = most_parts(ranges);
  } else {
    HT_TRY(rc);
  }
  float* partial = nullptr;
  if (parts > 0) HT_TRY(ht_scratch(R.ctx, HT_S_SPART, (size_t)parts * out_ld * 4, (void**)&partial));
  for (const ChunkRange& r : ranges) HT_TRY(agg_range(R, r, src, src_ld, d, out + r.row0 * out_ld, out_ld, relu, partial));
  return HT_OK;
}

// Scratch memory up to which a backward pass holds dz and grad a of all vertices at once.
constexpr int64_t HT_DIRECT_BYTES = (int64_t)8 << 30;

// Whether an aggregate of di columns that nothing keeps may take the plan: only where by its sizes the backward pass of the layer holds all
// rows at once (layer_bwd_direct) and can take the plan too.
bool again_fits(const Run& R, int di, int dn) {
  const ht_graph* g = R.g;
  const int64_t ld_i = ht_row_pitch(di, true), ld_o = ht_row_pitch(dn, true), entries = g->merged ? g->n_unique : g->Ep;
  return R.again_ok && ht_may_spend(R.ctx) && g->V * (2 * ld_i + ld_o) * 4 <= HT_DIRECT_BYTES && ht_by_source_parts_bound(entries) * ld_i * 4 <= HT_RANGE_BYTES;
}

// Forward of one layer with everything in HBM and rows read in place.
int layer_fwd_direct(Run& R, const ht_layer_desc* desc, const ht_tensor* H_in, const float* W, ht_tensor* H_out, ht_tensor* A_ckpt) {
  ht_ctx* ctx = R.ctx;
  const ht_graph* g = R.g;
  const int di = desc->d_in, dn = desc->d_out;
  const int64_t a_ld = A_ckpt ? A_ckpt->ld : ht_row_pitch(di, true);
  auto gemm = [&](const float* a, int64_t row0, int64_t rows) -> int {
    R.tm.begin(&R.st->t_gemm_ms);
    HT_TRY(ht_gemm_nn(ctx, ctx->stream, a, a_ld, W, H_out->ptr + row0 * H_out->ld, H_out->ld, rows, di, dn, desc->act == HT_ACT_RELU));
    R.tm.end();
    R.st->n_gemm += 1;
    R.st->gemm_flops += 2.0 * rows * di * dn;
    return HT_OK;
  };
  std::vector<ChunkRange> ranges;
  int64_t parts = 0, rows = 0;
  auto plan = [&](int64_t cap) {
    ranges = chunk_ranges(g, a_ld * 4, A_ckpt ? 0 : a_ld * 4, cap);
    parts = most_parts(ranges);
    rows = 0;
    for (const ChunkRange& r : ranges) rows = std::max(rows, r.rows);
  };
  PassPlan planned;
  if (A_ckpt || again_fits(R, di, dn)) HT_TRY(take_plan(R, true, di, H_in->ld, a_ld, &planned));
  R.note_planned(false);
  if (planned.items) {
    const int rc = ht_scratch_all(ctx, {{HT_S_ACHUNK, A_ckpt ? 0 : (size_t)(g->V * a_ld) * 4}, {HT_S_PACKW, (size_t)ht_packed_w_bytes(di, dn)}});
    if (rc == HT_OK) {
      float* a = A_ckpt ? A_ckpt->ptr : (float*)ctx->scratch[HT_S_ACHUNK];
      R.note_planned(!A_ckpt);
      HT_TRY(agg_range(R, whole_graph(g), H_in->ptr, H_in->ld, di, a, a_ld, 0, (float*)ctx->scratch[HT_S_SPART], planned));
      return gemm(a, 0, g->V);
    }
    if (rc != HT_ENOMEM) HT_TRY(rc);
  }
  // (the allocation-free call's array also holds the packed copy of W)
  if (ctx->static_mode) plan((int64_t)HT_STATIC_SCRATCH_BYTES - ht_packed_w_bytes(di, dn) - 512);
  else {
    plan(ht_may_spend(ctx) ? HT_RANGE_BYTES : 0);
    const int rc = ht_scratch_all(ctx, {{HT_S_SPART, (size_t)(parts * a_ld) * 4}, {HT_S_ACHUNK, A_ckpt ? 0 : (size_t)(rows * a_ld) * 4},
                                        {HT_S_PACKW, (size_t)ht_packed_w_bytes(di, dn)}});
    if (rc == HT_ENOMEM) plan(0);   // less memory at a time: chunk by chunk
    else HT_TRY(rc);
  }
  float *partial = nullptr, *a_rows = nullptr;
  if (parts > 0) HT_TRY(ht_scratch(ctx, HT_S_SPART, (size_t)parts * a_ld * 4, (void**)&partial));
  if (!A_ckpt) HT_TRY(ht_scratch(ctx, HT_S_ACHUNK, (size_t)rows * a_ld * 4, (void**)&a_rows));
  for (const ChunkRange& r : ranges) {
    HT_TRY(agg_range(R, r, H_in->ptr, H_in->ld, di, A_ckpt ? A_ckpt->ptr + r.row0 * a_ld : a_rows, a_ld, 0, partial));
    if (!A_ckpt) HT_TRY(gemm(a_rows, r.row0, r.rows));
  }
  return A_ckpt ? gemm(A_ckpt->ptr, 0, g->V) : HT_OK;
}

int resolve_gather(ht_ctx* ctx, int mode, const ht_tensor* t, bool* buffer) {
  if (mode == HT_GATHER_AUTO) *buffer = t->loc != HT_LOC_DEVICE;
  else if (mode == HT_GATHER_DIRECT) {
    if (t->loc != HT_LOC_DEVICE) return ht_set_err(ctx, HT_ESHAPE, "direct gather needs the tensor in HBM");
    *buffer = false;
  } else if (mode == HT_GATHER_BUFFER) *buffer = true;
  else return ht_set_err(ctx, HT_EINVAL, "unknown gather mode %d", mode);
  return HT_OK;
}

// Contiguous row range between HBM and pinned host memory.  host_gpu is the
// GPU-usable alias of the host side (dst for D2H, src for H2D).
int copy_rows(Run& R, hipStream_t st, void* dst, const void* src, size_t bytes, hipMemcpyKind kind) {
  if (bytes == 0) return HT_OK;
  ht_ctx* ctx = R.ctx;
  const int id = R.tm.begin_on(&R.st->t_copy_ms, st);
  const int lm = ctx->link_memcpy;   // 1: both directions, 2: device to host only, 3: host to device only
  if (lm == 1 || (lm == 2 && kind == hipMemcpyDeviceToHost) || (lm == 3 && kind == hipMemcpyHostToDevice)) {
    HT_HIP(ctx, hipMemcpyAsync(dst, src, bytes, kind, st));
  } else {
    void* d = dst;
    const void* s = src;
    void* mapped = nullptr;
    if (kind == hipMemcpyDeviceToHost) {
      HT_HIP(ctx, hipHostGetDevicePointer(&mapped, dst, 0));
      d = mapped;
    } else if (kind == hipMemcpyHostToDevice) {
      HT_HIP(ctx, hipHostGetDevicePointer(&mapped, const_cast<void*>(src), 0));
      s = mapped;
    }
    HT_TRY(ht_copy_link(ctx, st, d, s, bytes, ctx->link_blocks));
  }
  R.tm.end_id(id);
  if (kind == hipMemcpyHostToDevice) R.st->bytes_h2d += (int64_t)bytes;
  if (kind == hipMemcpyDeviceToHost) R.st->bytes_d2h += (int64_t)bytes;
  return HT_OK;
}

int layer_fwd_impl(Run& R, const ht_layer_desc* desc, const ht_tensor* H_in, const float* W, ht_tensor* H_out,
                   ht_tensor* A_ckpt) {
  ht_ctx* ctx = R.ctx;
  const ht_graph* g = R.g;
  const int di = desc->d_in, dn = desc->d_out;
  HT_TRY(check_tensor(ctx, H_in, g->V, di, "H_in"));
  HT_TRY(check_tensor(ctx, H_out, g->V, dn, "H_out"));
  if (A_ckpt) HT_TRY(check_tensor(ctx, A_ckpt, g->V, di, "A_ckpt"));
  if (!W) return ht_set_err(ctx, HT_EINVAL, "W is null");
  bool buffer = false;
  HT_TRY(resolve_gather(ctx, desc->gather_mode, H_in, &buffer));
  float* Hin = nullptr;
  HT_TRY(gpu_ptr(ctx, H_in, &Hin));

  const bool a_dev = A_ckpt && A_ckpt->loc == HT_LOC_DEVICE;
  const bool a_host = A_ckpt && !a_dev;
  const bool h_dev = H_out->loc == HT_LOC_DEVICE;
  const bool staged = a_host || !h_dev;                              // some rows leave through the output stream
  const bool side_in = buffer && H_in->loc == HT_LOC_HOST_PINNED;    // gather runs beside the compute
  const int64_t a_ld = A_ckpt ? A_ckpt->ld : ht_row_pitch(di, true);
  const int64_t mx = std::max<int64_t>(g->max_ndst, 1);
  float* a_stage[2] = {nullptr, nullptr};
  float* h_stage[2] = {nullptr, nullptr};
  float* nbuf = nullptr;
  // A/B variant: no aggregate is kept and everything is in HBM: aggregate and transform in one kernel (ht_fused.hip)
  const bool fused = ctx->fuse_update && !A_ckpt && h_dev && !buffer && H_in->loc == HT_LOC_DEVICE && di <= 1024;
  if (!buffer && !staged && !fused) return layer_fwd_direct(R, desc, H_in, W, H_out, A_ckpt);
  if (!a_dev && !fused) {
    HT_TRY(ht_scratch(ctx, HT_S_ACHUNK, (size_t)mx * a_ld * 4 * 2, (void**)&a_stage[0]));
    a_stage[1] = a_stage[0] + mx * a_ld;
  }
  if (!h_dev) {
    HT_TRY(ht_scratch(ctx, HT_S_OCHUNK, (size_t)mx * H_out->ld * 4 * 2, (void**)&h_stage[0]));
    h_stage[1] = h_stage[0] + mx * H_out->ld;
  }
  if (buffer) HT_TRY(ht_scratch(ctx, HT_S_NBUF, (size_t)g->cache_rows * H_in->ld * 4, (void**)&nbuf));

  Pipe P(ctx);
  if (side_in) {
    hipEvent_t ev_start = nullptr;
    HT_TRY(P.rec(P.s_c, &ev_start));
    HT_TRY(P.wait(P.s_in, ev_start));
    P.used_in = true;
  }
  hipEvent_t ev_out[2] = {nullptr, nullptr};   // D2H of the staging pair b has finished
  hipEvent_t ev_agg_prev = nullptr;            // the previous chunk's aggregation has read the buffer
  // With a^l and h^{l+1} both in HBM the update stage of neighbouring chunks runs as one GEMM over their joint row
  // range (chunks are balanced by edges, and a hub chunk of a thousand rows cannot fill the matrix cores); each output
  // row is the same sum whatever range it is computed in.
  const bool merge_dense = a_dev && h_dev;
  int64_t pend0 = -1, pend1 = -1;
  auto flush_dense = [&]() -> int {
    if (pend0 < 0) return HT_OK;
    const int64_t nr = pend1 - pend0;
    R.tm.begin(&R.st->t_gemm_ms);
    HT_TRY(ht_gemm_nn(ctx, P.s_c, A_ckpt->ptr + pend0 * a_ld, a_ld, W, H_out->ptr + pend0 * H_out->ld, H_out->ld, nr, di, dn,
                      desc->act == HT_ACT_RELU));
    R.tm.end();
    R.st->n_gemm += 1;
    R.st->gemm_flops += 2.0 * nr * di * dn;
    pend0 = pend1 = -1;
    return HT_OK;
  };
  int q = 0;
  for (int j = 0; j < g->n; ++j) {
    const ChunkMeta& c = g->chunks[j];
    const int64_t ndst = c.dst1 - c.dst0;
    if (ndst == 0) continue;
    const int b = q & 1;
    ++q;
    if (buffer) {
      if (side_in) {
        HT_TRY(P.wait(P.s_in, ev_agg_prev));   // the buffer is updated in place
        HT_TRY(gather_chunk(R, j, H_in, Hin, di, nbuf, P.s_in));
        hipEvent_t ev_g = nullptr;
        HT_TRY(P.rec(P.s_in, &ev_g));
        HT_TRY(P.wait(P.s_c, ev_g));
      } else {
        HT_TRY(gather_chunk(R, j, H_in, Hin, di, nbuf, P.s_c));
      }
    }
    if (fused) {
      const int li = R.layer < HT_MAX_LAYERS ? R.layer : HT_MAX_LAYERS - 1;
      R.tm.begin(&R.st->t_agg_fwd_layer_ms[li]);
      HT_TRY(ht_agg_update_fused(ctx, P.s_c, g, c, Hin, H_in->ld, di, W, dn, desc->act == HT_ACT_RELU, H_out->ptr, H_out->ld));
      R.tm.end();
      R.st->n_spmm_fwd += 1;
      R.st->n_agg_fwd_layer[li] += 1;
      R.st->edges += c.nnz;
      R.st->spmm_fwd_alg_bytes += spmm_alg_bytes(c, di);
      R.st->agg_fwd_layer_alg_bytes[li] += spmm_alg_bytes(c, di);
      R.st->n_gemm += 1;
      R.st->gemm_flops += 2.0 * ndst * di * dn;
      continue;
    }
    if (staged) HT_TRY(P.wait(P.s_c, ev_out[b]));
    float* a_dst = a_dev ? A_ckpt->ptr + c.dst0 * a_ld : a_stage[b];
    HT_TRY(spmm_chunk(R, j, buffer, buffer ? nbuf : Hin, H_in->ld, di, a_dst, a_ld));
    if (side_in) HT_TRY(P.rec(P.s_c, &ev_agg_prev));
    if (merge_dense) {
      if (pend0 >= 0 && c.dst0 != pend1) HT_TRY(flush_dense());   // not adjacent in vertex order (reorganised schedule)
      if (pend0 < 0) pend0 = c.dst0;
      pend1 = c.dst1;
      if (pend1 - pend0 >= HT_DENSE_MERGE_ROWS) HT_TRY(flush_dense());
      continue;
    }
    float* h_dst = h_dev ? H_out->ptr + c.dst0 * H_out->ld : h_stage[b];
    R.tm.begin(&R.st->t_gemm_ms);
    HT_TRY(ht_gemm_nn(ctx, P.s_c, a_dst, a_ld, W, h_dst, H_out->ld, ndst, di, dn, desc->act == HT_ACT_RELU));
    R.tm.end();
    R.st->n_gemm += 1;
    R.st->gemm_flops += 2.0 * ndst * di * dn;
    if (staged) {
      hipEvent_t ev_c = nullptr;
      HT_TRY(P.rec(P.s_c, &ev_c));
      HT_TRY(P.wait(P.s_out, ev_c));
      P.used_out = true;
      if (a_host)
        HT_TRY(copy_rows(R, P.s_out, A_ckpt->ptr + c.dst0 * a_ld, a_stage[b], (size_t)ndst * a_ld * 4, hipMemcpyDeviceToHost));
      if (!h_dev)
        HT_TRY(copy_rows(R, P.s_out, H_out->ptr + c.dst0 * H_out->ld, h_stage[b], (size_t)ndst * H_out->ld * 4,
                         hipMemcpyDeviceToHost));
      HT_TRY(P.rec(P.s_out, &ev_out[b]));
    }
  }
  HT_TRY(flush_dense());
  // later work on the compute stream sees every row at its home
  HT_TRY(P.wait(P.s_c, ev_out[0]));
  HT_TRY(P.wait(P.s_c, ev_out[1]));
  P.used_in = P.used_out = false;   // everything is ordered behind the compute stream now
  return HT_OK;
}

// Layer forward from a cached aggregate: h' = act(a W) per chunk, a^l read from A (HBM in place,
// or pinned host memory through a staging pair).  Used for layer 0 when a^0 = A_hat X of an earlier
// epoch is still valid.
int layer_fwd_from_ckpt(Run& R, const ht_layer_desc* desc, const ht_tensor* A, const float* W, ht_tensor* H_out) {
  ht_ctx* ctx = R.ctx;
  const ht_graph* g = R.g;
  const int di = desc->d_in, dn = desc->d_out;
  HT_TRY(check_tensor(ctx, A, g->V, di, "A_ckpt"));
  HT_TRY(check_tensor(ctx, H_out, g->V, dn, "H_out"));
  const bool a_host = A->loc == HT_LOC_HOST_PINNED;
  const bool h_dev = H_out->loc == HT_LOC_DEVICE;
  const int64_t mx = std::max<int64_t>(g->max_ndst, 1);
  float* a_stage[2] = {nullptr, nullptr};
  float* h_stage[2] = {nullptr, nullptr};
  if (a_host) {
    HT_TRY(ht_scratch(ctx, HT_S_ACHUNK, (size_t)mx * A->ld * 4 * 2, (void**)&a_stage[0]));
    a_stage[1] = a_stage[0] + mx * A->ld;
  }
  if (!h_dev) {
    HT_TRY(ht_scratch(ctx, HT_S_OCHUNK, (size_t)mx * H_out->ld * 4 * 2, (void**)&h_stage[0]));
    h_stage[1] = h_stage[0] + mx * H_out->ld;
  }
  Pipe P(ctx);
  if (a_host) {
    hipEvent_t ev_start = nullptr;
    HT_TRY(P.rec(P.s_c, &ev_start));
    HT_TRY(P.wait(P.s_in, ev_start));
    P.used_in = true;
  }
  hipEvent_t ev_out[2] = {nullptr, nullptr}, ev_cdone[2] = {nullptr, nullptr};
  int q = 0;
  for (int j = 0; j < g->n; ++j) {
    const ChunkMeta& c = g->chunks[j];
    const int64_t ndst = c.dst1 - c.dst0;
    if (ndst == 0) continue;
    const int b = q & 1;
    ++q;
    const float* a_rows = A->ptr + c.dst0 * A->ld;
    if (a_host) {
      hipEvent_t ev_in = nullptr;
      HT_TRY(P.wait(P.s_in, ev_cdone[b]));
      HT_TRY(copy_rows(R, P.s_in, a_stage[b], a_rows, (size_t)ndst * A->ld * 4, hipMemcpyHostToDevice));
      HT_TRY(P.rec(P.s_in, &ev_in));
      HT_TRY(P.wait(P.s_c, ev_in));
      a_rows = a_stage[b];
    }
    if (!h_dev) HT_TRY(P.wait(P.s_c, ev_out[b]));
    float* h_dst = h_dev ? H_out->ptr + c.dst0 * H_out->ld : h_stage[b];
    R.tm.begin(&R.st->t_gemm_ms);
    HT_TRY(ht_gemm_nn(ctx, P.s_c, a_rows, A->ld, W, h_dst, H_out->ld, ndst, di, dn, desc->act == HT_ACT_RELU));
    R.tm.end();
    R.st->n_gemm += 1;
    R.st->gemm_flops += 2.0 * ndst * di * dn;
    if (a_host) HT_TRY(P.rec(P.s_c, &ev_cdone[b]));
    if (!h_dev) {
      hipEvent_t ev_c = nullptr;
      HT_TRY(P.rec(P.s_c, &ev_c));
      HT_TRY(P.wait(P.s_out, ev_c));
      P.used_out = true;
      HT_TRY(copy_rows(R, P.s_out, H_out->ptr + c.dst0 * H_out->ld, h_stage[b], (size_t)ndst * H_out->ld * 4,
                       hipMemcpyDeviceToHost));
      HT_TRY(P.rec(P.s_out, &ev_out[b]));
    }
  }
  HT_TRY(P.wait(P.s_c, ev_out[0]));
  HT_TRY(P.wait(P.s_c, ev_out[1]));
  P.used_in = P.used_out = false;
  return HT_OK;
}

struct AccTask {
  hipEvent_t ready;   // the D2H of `rows` has finished
  float* grad;
  int64_t ld;
  const int32_t* ids;
  const float* rows;
  int64_t rows_ld;
  int64_t n;
  int d;
};

// Host-side gradient accumulation beside the GPU work (Alg. 3).  A worker
// thread waits for each task's D2H event on the host and adds the rows; the
// enqueueing thread only blocks when it is about to reuse a staging buffer whose
// task has not finished.  (A host function enqueued in a HIP stream would do the
// same, but it occupies a hardware queue other streams share while it runs.)
class AccWorker {
 public:
  AccWorker(ht_ctx* ctx) : ctx_(ctx) {}
  ~AccWorker() { finish(); }
  void start() {
    if (!th_.joinable()) th_ = std::thread([this] { run(); });
  }
  void push(const AccTask& t) {
    std::lock_guard<std::mutex> lk(mu_);
    q_.push_back(t);
    cv_.notify_all();
  }
  // block until at least `count` tasks have completed
  void wait_done(int64_t count) {
    std::unique_lock<std::mutex> lk(mu_);
    cv_.wait(lk, [&] { return done_ >= count || failed_; });
  }
  void finish() {
    if (!th_.joinable()) return;
    {
      std::lock_guard<std::mutex> lk(mu_);
      stop_ = true;
      cv_.notify_all();
    }
    th_.join();
  }
  bool failed() const { return failed_; }
  double ms() const { return ms_; }

 private:
  void run() {
    (void)hipSetDevice(ctx_->device);
    int64_t next = 0;
    for (;;) {
      AccTask t;
      {
        std::unique_lock<std::mutex> lk(mu_);
        cv_.wait(lk, [&] { return stop_ || next < (int64_t)q_.size(); });
        if (next >= (int64_t)q_.size()) return;   // stop requested and queue drained
        t = q_[next];
      }
      if (hipEventSynchronize(t.ready) != hipSuccess) {
        std::lock_guard<std::mutex> lk(mu_);
        failed_ = true;
        cv_.notify_all();
        return;
      }
      auto t0 = std::chrono::steady_clock::now();
      cpu_accumulate(ctx_, t.grad, t.ld, t.ids, t.rows, t.rows_ld, t.n, t.d);
      const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
      {
        std::lock_guard<std::mutex> lk(mu_);
        ms_ += ms;
        ++next;
        done_ = next;
        cv_.notify_all();
      }
    }
  }
  ht_ctx* ctx_;
  std::thread th_;
  std::mutex mu_;
  std::condition_variable cv_;
  std::vector<AccTask> q_;
  int64_t done_ = 0;
  bool stop_ = false;
  std::atomic<bool> failed_{false};   // read by the enqueueing thread without the lock
  double ms_ = 0.0;
};

// dst[u] = s_u * sum over u's entries of s_v src[v] for all sources u at once (src row = destination vertex): overwritten,
// or added to.  g->by_src is there, its partial sums fit `partial`.
int agg_by_source(Run& R, const float* src, int64_t src_ld, int d, float* dst, int64_t dst_ld, bool add, float* partial, const PassPlan& plan) {
  const ht_graph* g = R.g;
  const SourceRows& S = g->by_src;
  SpmmArgs a{};
  a.items = S.items.items.p; a.n_items = S.items.n_items;
  a.cuts = S.items.cuts.p; a.n_fix = S.items.n_cut;
  a.n_edges = g->merged ? g->n_unique : g->Ep;
  a.idx = S.idx.p;
  if (g->merged) a.w_edge = S.w.p;
  else a.ew = g->s.p;
  a.src = src; a.src_ld = src_ld; a.d = d;
  a.out = dst; a.out_ld = dst_ld;
  a.post = g->s.p;
  a.accumulate = add;
  a.partial = partial;
  a.max_slabs = R.ctx->slabs_bwd;
  R.tm.begin(&R.st->t_spmm_bwd_ms);
  HT_TRY(plan.items ? planned_launch(R, plan, a) : ht_spmm_launch(R.ctx, R.ctx->stream, a));
  R.tm.end();
  for (const ChunkMeta& c : g->chunks) R.st->n_spmm_bwd += c.dst1 > c.dst0;
  R.st->edges += g->Ep;
  R.st->spmm_bwd_alg_bytes += agg_all_bytes(g, g->Ep, g->V, d);
  return HT_OK;
}
// A by-source pass over rows of pitch ld keeps this many bytes of partial sums (of a list that is there).
size_t by_source_parts(const ht_graph* g, int64_t ld) { return (size_t)(g->by_src.items.n_part * ld) * 4; }
// Takes the slots and the by-source list, or HT_ENOMEM and nothing larger than before.  parts: bytes of other partial sums that share
// their slot.  slot: one that is written after the list was made.
int take_by_source(ht_ctx* ctx, const ht_graph* g, std::vector<ScratchWant> want, int64_t ld, size_t parts, int slot) {
  if (!ht_may_spend(ctx) || by_source_parts(g, ld) > (size_t)HT_RANGE_BYTES) return HT_ENOMEM;
  ScratchMark mark(ctx);
  int64_t list;
  size_t making;
  ht_graph_by_source_bytes(g, &list, &making);
  want.push_back({slot, making});
  int rc = ht_scratch_all(ctx, want, list);
  if (rc == HT_OK) rc = ht_graph_by_source(ctx, g, slot);
  if (rc == HT_OK) {
    const size_t mine = by_source_parts(g, ld);
    want.push_back({HT_S_SPART, std::max(mine, parts)});
    rc = mine > (size_t)HT_RANGE_BYTES ? HT_ENOMEM : ht_scratch_all(ctx, want);
  }
  if (rc == HT_ENOMEM) mark.undo();
  return rc;
}

// Backward of one layer with everything in HBM, all destinations at once: one launch of every dense kernel, and an
// aggregation by source over the whole graph, which reads and writes every row of dH_in once (chunk by chunk a row is read and
// written again for every chunk that names its vertex, and the work items are as many times shorter: 1 M vertices, 20 M edges,
// 64 columns, 16 chunks, forward and backward 6.6 -> 3.2 ms).  *done = false: it would
// take more scratch memory than it may have, nothing was enqueued.
int layer_bwd_direct(Run& R, const ht_layer_desc* desc, const ht_tensor* ckpt, const float* W, const ht_tensor* dH_out,
                     const ht_tensor* H_out, ht_tensor* dH_in, float* dW, bool* done) {
  ht_ctx* ctx = R.ctx;
  const ht_graph* g = R.g;
  hipStream_t st = ctx->stream;
  const int di = desc->d_in, dn = desc->d_out;
  const int64_t V = g->V, ld_i = ht_row_pitch(di, true), ld_o = ht_row_pitch(dn, true);
  const bool relu = desc->act == HT_ACT_RELU, agg_ckpt = desc->ckpt_kind == HT_CKPT_AGG;
  const int64_t a_ld = agg_ckpt ? ckpt->ld : ld_i;
  *done = false;
  float *a_all = nullptr, *dz_all = nullptr, *da_all = nullptr, *partial = nullptr;
  // (dz: for grad a, or for the activations made again; grad W alone masks its rows on the way)
  const size_t a_bytes = agg_ckpt ? 0 : (size_t)V * a_ld * 4, dz_bytes = relu && (dH_in || !H_out) ? (size_t)V * ld_o * 4 : 0,
               da_bytes = dH_in ? (size_t)V * ld_i * 4 : 0;
  if (!ht_may_spend(ctx) || (int64_t)(a_bytes + dz_bytes + da_bytes) > HT_DIRECT_BYTES) return HT_OK;
  // everything that this pass will ask for: nothing may fail once dH_in is being added to
  const size_t fwd_parts = agg_ckpt ? 0 : (size_t)(most_parts(chunk_ranges(g, a_ld * 4, 0, HT_RANGE_BYTES)) * a_ld) * 4;
  std::vector<ScratchWant> want = {{HT_S_ACHUNK, a_bytes}, {HT_S_DZCHUNK, dz_bytes}, {HT_S_DACHUNK, da_bytes}, {HT_S_SPART, fwd_parts},
                                   {HT_S_PACKW, (size_t)std::max(ht_packed_w_bytes(di, dn), ht_packed_w_bytes(dn, di))}};
  ht_gemm_groups_wants(di, dn, g->dense_groups, &want);
  const int rc = dH_in ? take_by_source(ctx, g, want, dH_in->ld, fwd_parts, HT_S_DACHUNK) : ht_scratch_all(ctx, want);
  if (rc == HT_ENOMEM) return HT_OK;
  HT_TRY(rc);
  PassPlan plan, again;
  if (!agg_ckpt && R.made_planned()) {
    HT_TRY(take_plan(R, true, di, ckpt->ld, a_ld, &again));
    if (!again.items) return HT_OK;
  }
  if (dH_in) HT_TRY(take_plan(R, false, di, ld_i, dH_in->ld, &plan));
  // Every slot again before a pointer into one is kept: plans let them grow, and one that was refused memory half-way may have left them smaller.
  if (dH_in && !plan.items) want.push_back({HT_S_SPART, by_source_parts(g, dH_in->ld)});
  want.push_back({HT_S_SPART, (size_t)(again.parts() * a_ld) * 4});
  HT_TRY(ht_scratch_each(ctx, want));
  if (a_bytes) a_all = (float*)ctx->scratch[HT_S_ACHUNK];
  if (dz_bytes) dz_all = (float*)ctx->scratch[HT_S_DZCHUNK];
  if (da_bytes) da_all = (float*)ctx->scratch[HT_S_DACHUNK];
  partial = (float*)ctx->scratch[HT_S_SPART];
  *done = true;
  const float* a_rows = ckpt->ptr;
  if (!agg_ckpt) {   // pure recomputation: aggregate again from h^l
    HT_TRY(agg_all(R, ckpt->ptr, ckpt->ld, di, a_all, a_ld, 0, again));
    a_rows = a_all;
  }
  R.changed = true;
  const double flops = 2.0 * V * di * dn;
  auto timed_gemm = [&](auto&& f) -> int {
    R.tm.begin(&R.st->t_gemm_ms);
    HT_TRY(f());
    R.tm.end();
    R.st->n_gemm += 1;
    R.st->gemm_flops += flops;
    return HT_OK;
  };
  const float* dz = dH_out->ptr;
  int64_t dz_ld = dH_out->ld;
  ReluMask mask;
  if (relu) {
    const float* ref = H_out ? H_out->ptr : dz_all;
    const int64_t ref_ld = H_out ? H_out->ld : ld_o;
    if (!H_out)   // re-forward of the update stage (Alg. 1)
      HT_TRY(timed_gemm([&] { return ht_gemm_nn(ctx, st, a_rows, a_ld, W, dz_all, ld_o, V, di, dn, 0); }));
    if (!dH_in) {   // grad W alone reads dz, and masks it on the way
      mask = ReluMask{ref, ref_ld};
    } else if (ht_gemm_tn_writes(V, di, dn)) {   // ... and leaves it for the other product
      mask = ReluMask{ref, ref_ld, dz_all, ld_o};
    } else {
      HT_TRY(ht_relu_mask(ctx, st, dH_out->ptr, dH_out->ld, ref, ref_ld, dz_all, ld_o, V, dn));
      dz = dz_all;
      dz_ld = ld_o;
    }
  }
  TnLater later;
  HT_TRY(timed_gemm([&] { return ht_gemm_tn_groups(ctx, st, a_rows, a_ld, dz, dz_ld, dW, di, dn, g->dense_groups, g->d_dense_groups.p, &later, mask); }));
  if (!dH_in) return HT_OK;
  if (mask.to) {
    dz = mask.to;
    dz_ld = mask.to_ld;
  }
  HT_TRY(timed_gemm([&] { return ht_gemm_nt(ctx, st, dz, dz_ld, W, da_all, ld_i, V, dn, di, 0); }));
  return agg_by_source(R, da_all, ld_i, di, dH_in->ptr, dH_in->ld, !R.dhin_fresh, partial, plan);
}

int layer_bwd_impl(Run& R, const ht_layer_desc* desc, const ht_tensor* ckpt, const float* W, const ht_tensor* dH_out,
                   const ht_tensor* H_out, ht_tensor* dH_in, float* dW) {
  ht_ctx* ctx = R.ctx;
  const ht_graph* g = R.g;
  hipStream_t st = ctx->stream;
  const int di = desc->d_in, dn = desc->d_out;
  HT_TRY(check_tensor(ctx, ckpt, g->V, di, "ckpt"));
  HT_TRY(check_tensor(ctx, dH_out, g->V, dn, "dH_out"));
  if (H_out) HT_TRY(check_tensor(ctx, H_out, g->V, dn, "H_out"));
  if (dH_in) HT_TRY(check_tensor(ctx, dH_in, g->V, di, "dH_in"));
  if (!W || !dW) return ht_set_err(ctx, HT_EINVAL, "W or dW is null");
  if (desc->ckpt_kind != HT_CKPT_AGG && desc->ckpt_kind != HT_CKPT_INPUT)
    return ht_set_err(ctx, HT_EINVAL, "unknown checkpoint kind %d", desc->ckpt_kind);
  const bool relu = desc->act == HT_ACT_RELU;
  const bool agg_ckpt = desc->ckpt_kind == HT_CKPT_AGG;
  const int64_t mx = std::max<int64_t>(g->max_ndst, 1);
  const int64_t ld_i = ht_row_pitch(di, true), ld_o = ht_row_pitch(dn, true);

  // forward-side inputs
  bool agg_buffer = false;
  float* Hin = nullptr;
  float* nbuf = nullptr;
  if (!agg_ckpt) {
    HT_TRY(resolve_gather(ctx, desc->gather_mode, ckpt, &agg_buffer));
    HT_TRY(gpu_ptr(ctx, ckpt, &Hin));
    if (agg_buffer) HT_TRY(ht_scratch(ctx, HT_S_NBUF, (size_t)g->cache_rows * ckpt->ld * 4, (void**)&nbuf));
  }
  // gradient side: direct accumulation into dH_in (HBM) or through the in-place gradient buffer
  bool gbuffer = false;
  if (dH_in) HT_TRY(resolve_gather(ctx, desc->gather_mode, dH_in, &gbuffer));

  const bool a_host = agg_ckpt && ckpt->loc != HT_LOC_DEVICE;
  const bool dh_host = dH_out->loc != HT_LOC_DEVICE;
  const bool ho_host = relu && H_out && H_out->loc != HT_LOC_DEVICE;
  const bool in_host = a_host || dh_host || ho_host;   // some rows arrive through the input stream
  float* a_stage[2] = {nullptr, nullptr};
  float* dh_stage[2] = {nullptr, nullptr};
  float* z_stage[2] = {nullptr, nullptr};
  float *dz_chunk = nullptr, *da_chunk = nullptr, *gbuf = nullptr;
  const int64_t a_ld = agg_ckpt ? ckpt->ld : ld_i;
  // The dense work (mask, grad W, grad a) of neighbouring chunks runs as one launch over their joint row range when
  // everything it touches is in HBM and no buffer is updated in place between chunks: chunks are balanced by edges, and a
  // hub chunk of a thousand rows cannot fill the matrix cores.  The grouping depends on the graph and on where the
  // tensors live only, so every intermediate-data mode sums grad W in the same order.  Each group is a run of chunks
  // adjacent in schedule and in vertex order, closed once it holds HT_DENSE_MERGE_ROWS rows; elsewhere one chunk each.
  const bool merge_ok = !in_host && !agg_buffer && !(dH_in && gbuffer);
  std::vector<std::pair<int, int>> groups;
  int64_t gmax = mx;
  for (int j = 0; j < g->n;) {
    int k = j;
    if (merge_ok && g->chunks[j].dst1 > g->chunks[j].dst0)
      while (k + 1 < g->n && g->chunks[k + 1].dst1 > g->chunks[k + 1].dst0 && g->chunks[k + 1].dst0 == g->chunks[k].dst1 &&
             g->chunks[k].dst1 - g->chunks[j].dst0 < HT_DENSE_MERGE_ROWS)
        ++k;
    groups.emplace_back(j, k);
    gmax = std::max(gmax, g->chunks[k].dst1 - g->chunks[j].dst0);
    j = k + 1;
  }
  if (merge_ok) {   // everything in HBM, nothing updated in place between chunks
    bool done = false;
    HT_TRY(layer_bwd_direct(R, desc, ckpt, W, dH_out, relu ? H_out : nullptr, dH_in, dW, &done));
    if (done) return HT_OK;
  }
  // (there was memory for the forward pass's plan and is none now: the call is made again, without)
  if (!agg_ckpt && R.made_planned()) return ht_set_err(ctx, HT_ENOMEM, "backward pass: no memory for the aggregate that the forward pass has not kept");
  if (dH_in && R.dhin_fresh && dH_in->loc == HT_LOC_DEVICE) HT_TRY(ht_fill_zero(ctx, st, dH_in->ptr, (size_t)dH_in->rows * dH_in->ld * 4));
  if (!agg_ckpt || a_host) {
    HT_TRY(ht_scratch(ctx, HT_S_ACHUNK, (size_t)gmax * a_ld * 4 * 2, (void**)&a_stage[0]));
    a_stage[1] = a_stage[0] + gmax * a_ld;
  }
  if (dh_host) {
    HT_TRY(ht_scratch(ctx, HT_S_OCHUNK, (size_t)mx * dH_out->ld * 4 * 2, (void**)&dh_stage[0]));
    dh_stage[1] = dh_stage[0] + mx * dH_out->ld;
  }
  if (relu) {
    const int64_t zl = H_out ? H_out->ld : ld_o;
    if (!H_out || ho_host) {
      HT_TRY(ht_scratch(ctx, HT_S_ZCHUNK, (size_t)gmax * zl * 4 * 2, (void**)&z_stage[0]));
      z_stage[1] = z_stage[0] + gmax * zl;
    }
    HT_TRY(ht_scratch(ctx, HT_S_DZCHUNK, (size_t)gmax * ld_o * 4, (void**)&dz_chunk));
  }
  if (dH_in) {
    HT_TRY(ht_scratch(ctx, HT_S_DACHUNK, (size_t)gmax * ld_i * 4, (void**)&da_chunk));
    if (gbuffer) HT_TRY(ht_scratch(ctx, HT_S_MISC, (size_t)g->cache_rows * ld_i * 4, (void**)&gbuf));
  }
  // what the chunks ask for on the way, each in turn: nothing may fail once dH_in is being added to
  {
    const int64_t out_ld = dH_in ? (gbuffer ? ld_i : dH_in->ld) : 0;
    std::vector<ScratchWant> want = {{HT_S_SPART, (size_t)std::max(agg_ckpt ? 0 : g->max_fpart * a_ld, g->max_bpart * out_ld) * 4}};
    if (relu && !H_out) want.push_back({HT_S_PACKW, (size_t)ht_packed_w_bytes(di, dn)});
    if (dH_in) want.push_back({HT_S_PACKW, (size_t)ht_packed_w_bytes(dn, di)});
    for (const auto& gr : groups)
      want.push_back({HT_S_TNPART, ht_gemm_tn_bytes(g->chunks[gr.second].dst1 - g->chunks[gr.first].dst0, di, dn)});
    HT_TRY(ht_scratch_each(ctx, want));
  }
  // CPU-side accumulation (Alg. 3): host copy of the leave lists, device and pinned staging pairs
  // When the schedule loads every row once per pass, each row also leaves exactly once, after the last
  // chunk that adds to it: if dH_in is known to hold zeros the rows are stored straight to their home
  // by a link kernel, no host-side add.
  const bool store_home = dH_in && gbuffer && dH_in->loc == HT_LOC_HOST_PINNED && g->single_leave && R.dhin_fresh;
  const bool cpu_accum = dH_in && gbuffer && dH_in->loc == HT_LOC_HOST_PINNED && !store_home;
  float* dhin_gpu = nullptr;
  if (store_home) HT_TRY(gpu_ptr(ctx, dH_in, &dhin_gpu));
  constexpr int NLV = 4;   // depth of the leave staging rings: D2H runs ahead of the host-side adds
  constexpr int64_t LEAVE_BATCH = 262144;   // rows per compaction / D2H / host-add task
  float* leave_dev[NLV] = {};
  float* leave_pin[NLV] = {};
  if (cpu_accum) {
    int64_t mxl = 1;
    for (const ChunkMeta& c : g->chunks) mxl = std::max(mxl, c.n_leave);
    mxl = std::min(mxl, LEAVE_BATCH);
    if (g->leave_host.empty()) {
      g->leave_host.resize((size_t)std::max<int64_t>(g->v_load, 1));
      HT_HIP(ctx, hipMemcpy(g->leave_host.data(), g->leave.p, (size_t)g->v_load * 4, hipMemcpyDeviceToHost));
    }
    HT_TRY(ht_scratch(ctx, HT_S_LEAVE, (size_t)mxl * ld_i * 4 * NLV, (void**)&leave_dev[0]));
    HT_TRY(ht_host_scratch(ctx, 0, (size_t)mxl * ld_i * 4 * NLV, (void**)&leave_pin[0]));
    for (int k = 1; k < NLV; ++k) {
      leave_dev[k] = leave_dev[0] + (int64_t)k * mxl * ld_i;
      leave_pin[k] = leave_pin[0] + (int64_t)k * mxl * ld_i;
    }
    (void)host_threads(ctx);
  }

  Pipe P(ctx);
  AccWorker worker(ctx);   // declared after P: joined before P's destructor waits for the streams
  if (cpu_accum) worker.start();
  R.changed = true;
  if (in_host) {
    hipEvent_t ev_start = nullptr;
    HT_TRY(P.rec(P.s_c, &ev_start));
    HT_TRY(P.wait(P.s_in, ev_start));
    P.used_in = true;
  }
  hipEvent_t ev_cdone[2] = {nullptr, nullptr};     // compute that read the input staging pair b has finished
  hipEvent_t ev_leave_free[NLV] = {};              // D2H out of leave_dev[r] has finished
  int n_left = 0;
  bool first = true;
  int q = 0;
  // ---- rows that the schedule releases after a chunk leave the gradient buffer (Alg. 3)
  hipEvent_t ev_stored = nullptr;   // the last store of leaving rows straight to their home
  auto leave_rows = [&](const ChunkMeta& c) -> int {
    if (!(dH_in && gbuffer && c.n_leave > 0)) return HT_OK;
    if (store_home) {
      hipEvent_t ev_done = nullptr, ev_st = nullptr;
      HT_TRY(P.rec(P.s_c, &ev_done));
      HT_TRY(P.wait(P.s_out, ev_done));
      P.used_out = true;
      const int id = R.tm.begin_on(&R.st->t_copy_ms, P.s_out);
      HT_TRY(ht_gather_rows(ctx, P.s_out, gbuf, ld_i, g->leave_slot.p + c.leave_off, dhin_gpu, dH_in->ld,
                            g->leave.p + c.leave_off, c.n_leave, di, nullptr, ctx->link_blocks));
      R.tm.end_id(id);
      R.st->bytes_d2h += c.n_leave * (int64_t)di * 4;
      HT_TRY(P.rec(P.s_out, &ev_st));
      ev_stored = ev_st;   // waited for before the next aggregation writes freed positions, and at the end
    } else if (!cpu_accum) {
      HT_TRY(ht_add_rows(ctx, st, gbuf, ld_i, g->leave_slot.p + c.leave_off, dH_in->ptr, dH_in->ld,
                         g->leave.p + c.leave_off, c.n_leave, di));
    } else {
      // compaction on the compute stream (the next chunk overwrites freed positions), D2H on the
      // output stream, the add on the host beside the next chunks' GPU work
      for (int64_t k0 = 0; k0 < c.n_leave; k0 += LEAVE_BATCH) {
        const int64_t nk = std::min(LEAVE_BATCH, c.n_leave - k0);
        const int64_t off = c.leave_off + k0;
        const int r = n_left++ % NLV;
        HT_TRY(P.wait(P.s_c, ev_leave_free[r]));
        HT_TRY(ht_gather_rows(ctx, st, gbuf, ld_i, g->leave_slot.p + off, leave_dev[r], ld_i, nullptr, nk, di, nullptr));
        hipEvent_t ev_comp = nullptr;
        HT_TRY(P.rec(P.s_c, &ev_comp));
        HT_TRY(P.wait(P.s_out, ev_comp));
        if (n_left > NLV) worker.wait_done(n_left - NLV);   // the host has consumed leave_pin[r]
        if (worker.failed()) return ht_set_err(ctx, HT_EHIP, "host-side accumulation: waiting for a copy failed");
        P.used_out = true;
        HT_TRY(copy_rows(R, P.s_out, leave_pin[r], leave_dev[r], (size_t)nk * ld_i * 4, hipMemcpyDeviceToHost));
        HT_TRY(P.rec(P.s_out, &ev_leave_free[r]));
        worker.push(AccTask{ev_leave_free[r], dH_in->ptr, dH_in->ld, g->leave_host.data() + off, leave_pin[r], ld_i, nk, di});
      }
    }
    return HT_OK;
  };
  for (const auto& grp : groups) {
    const int j0 = grp.first, j1 = grp.second;
    const ChunkMeta& c = g->chunks[j0];                       // the group's first chunk: its rows start the range
    const int64_t ndst = g->chunks[j1].dst1 - c.dst0;         // destination rows of the whole group
    if (ndst == 0) {   // no destinations: no edges, no neighbours; the schedule may still release rows here
      HT_TRY(leave_rows(c));
      continue;
    }
    const int b = q & 1;
    ++q;
    // ---- inputs (Alg. 1)
    const float* a_rows = nullptr;
    const float* dh_rows = nullptr;
    const float* ref = nullptr;
    int64_t ref_ld = 0;
    if (in_host) {
      HT_TRY(P.wait(P.s_in, ev_cdone[b]));
    }
    if (agg_ckpt) {
      if (a_host) {
        HT_TRY(copy_rows(R, P.s_in, a_stage[b], ckpt->ptr + c.dst0 * a_ld, (size_t)ndst * a_ld * 4, hipMemcpyHostToDevice));
        a_rows = a_stage[b];
      } else {
        a_rows = ckpt->ptr + c.dst0 * a_ld;
      }
    }
    if (dh_host) {
      HT_TRY(copy_rows(R, P.s_in, dh_stage[b], dH_out->ptr + c.dst0 * dH_out->ld, (size_t)ndst * dH_out->ld * 4,
                       hipMemcpyHostToDevice));
      dh_rows = dh_stage[b];
    } else {
      dh_rows = dH_out->ptr + c.dst0 * dH_out->ld;
    }
    if (relu && H_out) {
      ref_ld = H_out->ld;
      if (ho_host) {
        HT_TRY(copy_rows(R, P.s_in, z_stage[b], H_out->ptr + c.dst0 * H_out->ld, (size_t)ndst * H_out->ld * 4,
                         hipMemcpyHostToDevice));
        ref = z_stage[b];
      } else {
        ref = H_out->ptr + c.dst0 * H_out->ld;
      }
    }
    if (in_host) {
      hipEvent_t ev_in = nullptr;
      HT_TRY(P.rec(P.s_in, &ev_in));
      HT_TRY(P.wait(P.s_c, ev_in));
    }
    // ---- compute
    if (!agg_ckpt) {   // pure recomputation: aggregate again from h^l, chunk by chunk into the group's rows
      for (int j = j0; j <= j1; ++j) {
        const ChunkMeta& cj = g->chunks[j];
        if (agg_buffer) HT_TRY(gather_chunk(R, j, ckpt, Hin, di, nbuf, st));
        HT_TRY(spmm_chunk(R, j, agg_buffer, agg_buffer ? nbuf : Hin, ckpt->ld, di, a_stage[b] + (cj.dst0 - c.dst0) * a_ld, a_ld));
      }
      a_rows = a_stage[b];
    }
    const float* dz_rows = dh_rows;
    int64_t dz_ld = dH_out->ld;
    if (relu) {
      if (!H_out) {  // re-forward of the update stage (Alg. 1)
        R.tm.begin(&R.st->t_gemm_ms);
        HT_TRY(ht_gemm_nn(ctx, st, a_rows, a_ld, W, z_stage[0], ld_o, ndst, di, dn, 0));
        R.tm.end();
        R.st->n_gemm += 1;
        R.st->gemm_flops += 2.0 * ndst * di * dn;
        ref = z_stage[0];
        ref_ld = ld_o;
      }
      HT_TRY(ht_relu_mask(ctx, st, dh_rows, dH_out->ld, ref, ref_ld, dz_chunk, ld_o, ndst, dn));
      dz_rows = dz_chunk;
      dz_ld = ld_o;
    }
    R.tm.begin(&R.st->t_gemm_ms);
    HT_TRY(ht_gemm_tn(ctx, st, a_rows, a_ld, dz_rows, dz_ld, dW, ndst, di, dn, first ? 0 : 1));
    R.tm.end();
    R.st->n_gemm += 1;
    R.st->gemm_flops += 2.0 * ndst * di * dn;
    first = false;
    if (dH_in) {
      R.tm.begin(&R.st->t_gemm_ms);
      HT_TRY(ht_gemm_nt(ctx, st, dz_rows, dz_ld, W, da_chunk, ld_i, ndst, dn, di, 0));
      R.tm.end();
      R.st->n_gemm += 1;
      R.st->gemm_flops += 2.0 * ndst * di * dn;
    }
    if (in_host) HT_TRY(P.rec(P.s_c, &ev_cdone[b]));   // the staged inputs have been consumed
    for (int j = j0; j <= j1; ++j) {
      const ChunkMeta& cj = g->chunks[j];
      if (dH_in) {
        float* partial = nullptr;
        const int64_t out_ld = gbuffer ? ld_i : dH_in->ld;
        if (cj.bwd.n_part > 0) HT_TRY(ht_scratch(ctx, HT_S_SPART, (size_t)g->max_bpart * out_ld * 4, (void**)&partial));
        SpmmArgs a{};
        agg_args(g, cj, false, false, &a);
        a.src = da_chunk + (cj.dst0 - c.dst0) * ld_i;      // the chunk's rows inside the group's grad a
        a.src_ld = ld_i;
        a.d = di;
        a.out = gbuffer ? gbuf : dH_in->ptr;
        a.out_ld = out_ld;
        a.out_idx = gbuffer ? g->gslot.p : g->nbr.p;
        a.post = g->s.p;
        a.post_idx = g->nbr.p;
        a.accumulate = 1;
        a.partial = partial;
        a.max_slabs = ctx->slabs_bwd;
        HT_TRY(P.wait(P.s_c, ev_stored));   // positions freed by the last store are written from here on
        R.tm.begin(&R.st->t_spmm_bwd_ms);
        HT_TRY(ht_spmm_launch(ctx, st, a));
        R.tm.end();
        R.st->n_spmm_bwd += 1;
        R.st->edges += cj.nnz;
        R.st->spmm_bwd_alg_bytes += spmm_alg_bytes(cj, di);
      }
      HT_TRY(leave_rows(cj));
    }
  }
  if (first) HT_TRY(ht_fill_zero(ctx, st, dW, (size_t)di * dn * 4));
  if (store_home) {   // dH_in is complete for later work on the stream
    HT_TRY(P.wait(P.s_c, ev_stored));
    P.used_out = false;
  }
  if (cpu_accum) {
    // the gradient tensor is complete once every host-side add has run
    worker.finish();
    if (worker.failed()) return ht_set_err(ctx, HT_EHIP, "host-side accumulation: waiting for a copy failed");
    R.st->t_cpu_accum_ms += worker.ms();
    P.used_out = false;
  }
  P.used_in = false;   // every input copy was waited for by the compute stream
  return HT_OK;
}

// ---- update-first order: H' = act(A_hat (H W)).  Same function as Eq. 2 (both stages are
// linear), aggregating rows of width d_out.  Everything lives in HBM here.

int need_hbm(ht_ctx* ctx, const ht_tensor* t, const char* name) {
  if (t->loc != HT_LOC_DEVICE)
    return ht_set_err(ctx, HT_ESHAPE, "update-first order: %s must be in HBM", name);
  return HT_OK;
}

int layer_fwd_update_first(Run& R, const ht_layer_desc* desc, const ht_tensor* H_in, const float* W, ht_tensor* H_out) {
  ht_ctx* ctx = R.ctx;
  const ht_graph* g = R.g;
  hipStream_t st = ctx->stream;
  const int di = desc->d_in, dn = desc->d_out;
  HT_TRY(check_tensor(ctx, H_in, g->V, di, "H_in"));
  HT_TRY(check_tensor(ctx, H_out, g->V, dn, "H_out"));
  HT_TRY(need_hbm(ctx, H_in, "H_in"));
  HT_TRY(need_hbm(ctx, H_out, "H_out"));
  if (!W) return ht_set_err(ctx, HT_EINVAL, "W is null");
  const int64_t ld_t = ht_row_pitch(dn, true);
  float* T = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_TFULL, (size_t)std::max<int64_t>(g->V, 1) * ld_t * 4, (void**)&T));
  // t = H_in W for every vertex (row ranges keep the launches within the grid limits)
  const int64_t step = (int64_t)1 << 22;
  for (int64_t r0 = 0; r0 < g->V; r0 += step) {
    const int64_t nr = std::min(step, g->V - r0);
    R.tm.begin(&R.st->t_gemm_ms);
    HT_TRY(ht_gemm_nn(ctx, st, H_in->ptr + r0 * H_in->ld, H_in->ld, W, T + r0 * ld_t, ld_t, nr, di, dn, 0));
    R.tm.end();
    R.st->n_gemm += 1;
    R.st->gemm_flops += 2.0 * nr * di * dn;
  }
  PassPlan plan;
  HT_TRY(take_plan(R, true, dn, ld_t, H_out->ld, &plan));
  return agg_all(R, T, ld_t, dn, H_out->ptr, H_out->ld, desc->act == HT_ACT_RELU, plan);
}

int layer_bwd_update_first(Run& R, const ht_layer_desc* desc, const ht_tensor* H_in, const float* W,
                           const ht_tensor* dH_out, const ht_tensor* H_out, ht_tensor* dH_in, float* dW) {
  ht_ctx* ctx = R.ctx;
  const ht_graph* g = R.g;
  hipStream_t st = ctx->stream;
  const int di = desc->d_in, dn = desc->d_out;
  const bool relu = desc->act == HT_ACT_RELU;
  HT_TRY(check_tensor(ctx, H_in, g->V, di, "ckpt"));
  HT_TRY(check_tensor(ctx, dH_out, g->V, dn, "dH_out"));
  HT_TRY(need_hbm(ctx, H_in, "ckpt"));
  HT_TRY(need_hbm(ctx, dH_out, "dH_out"));
  if (relu && !H_out) return ht_set_err(ctx, HT_EINVAL, "update-first backward with ReLU needs H_out");
  if (H_out) {
    HT_TRY(check_tensor(ctx, H_out, g->V, dn, "H_out"));
    HT_TRY(need_hbm(ctx, H_out, "H_out"));
  }
  if (dH_in) {
    HT_TRY(check_tensor(ctx, dH_in, g->V, di, "dH_in"));
    HT_TRY(need_hbm(ctx, dH_in, "dH_in"));
  }
  if (!W || !dW) return ht_set_err(ctx, HT_EINVAL, "W or dW is null");
  const int64_t ld_t = ht_row_pitch(dn, true);
  const int64_t mx = std::max<int64_t>(g->max_ndst, 1);
  float *dT = nullptr, *dz_chunk = nullptr, *partial = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_TFULL, (size_t)std::max<int64_t>(g->V, 1) * ld_t * 4, (void**)&dT));
  const int64_t step = (int64_t)1 << 22;   // rows per dense launch
  std::vector<ScratchWant> want = {{HT_S_TNPART, ht_gemm_tn_bytes(std::min(step, g->V), di, dn)},
                                   {HT_S_TNPART, ht_gemm_tn_bytes(g->V % step, di, dn)}};
  if (dH_in) want.push_back({HT_S_PACKW, (size_t)ht_packed_w_bytes(dn, di)});
  // dt = A_hat^T dz over all sources at once where dz of all vertices and the by-source list fit (see layer_bwd_direct)
  bool at_once = (int64_t)g->V * ld_t * 4 <= HT_DIRECT_BYTES;
  if (at_once) {
    std::vector<ScratchWant> all = want;
    if (relu) all.push_back({HT_S_DZCHUNK, (size_t)g->V * ld_t * 4});
    const int rc = take_by_source(ctx, g, all, ld_t, 0, HT_S_DZCHUNK);
    at_once = rc == HT_OK;
    if (rc != HT_ENOMEM) HT_TRY(rc);
  }
  const size_t dz_bytes = relu ? (size_t)(at_once ? g->V : mx) * ld_t * 4 : 0,
               part_bytes = at_once ? by_source_parts(g, ld_t) : (size_t)(g->max_bpart * ld_t) * 4;
  want.push_back({HT_S_DZCHUNK, dz_bytes});
  want.push_back({HT_S_SPART, part_bytes});
  PassPlan plan;
  if (at_once) HT_TRY(take_plan(R, false, dn, relu ? ld_t : dH_out->ld, ld_t, &plan));
  HT_TRY(ht_scratch_each(ctx, want));   // (behind the plan: one that was refused memory half-way may have left slots smaller)
  dz_chunk = (float*)ctx->scratch[HT_S_DZCHUNK];
  partial = (float*)ctx->scratch[HT_S_SPART];
  R.changed = true;
  if (at_once) {
    if (relu) HT_TRY(ht_relu_mask(ctx, st, dH_out->ptr, dH_out->ld, H_out->ptr, H_out->ld, dz_chunk, ld_t, g->V, dn));
    HT_TRY(agg_by_source(R, relu ? dz_chunk : dH_out->ptr, relu ? ld_t : dH_out->ld, dn, dT, ld_t, false, partial, plan));
  } else {
    HT_TRY(ht_fill_zero(ctx, st, dT, (size_t)g->V * ld_t * 4));
  }
  // dt[N_j] += s_u * sum_v s_v dz[v], chunk by chunk
  for (int j = 0; !at_once && j < g->n; ++j) {
    const ChunkMeta& c = g->chunks[j];
    const int64_t ndst = c.dst1 - c.dst0;
    if (ndst == 0) continue;
    const float* dz_rows = dH_out->ptr + c.dst0 * dH_out->ld;
    int64_t dz_ld = dH_out->ld;
    if (relu) {
      HT_TRY(ht_relu_mask(ctx, st, dz_rows, dz_ld, H_out->ptr + c.dst0 * H_out->ld, H_out->ld, dz_chunk, ld_t, ndst, dn));
      dz_rows = dz_chunk;
      dz_ld = ld_t;
    }
    SpmmArgs a{};
    agg_args(g, c, false, false, &a);
    a.src = dz_rows; a.src_ld = dz_ld; a.d = dn;
    a.out = dT; a.out_ld = ld_t;
    a.out_idx = g->nbr.p;
    a.post = g->s.p; a.post_idx = g->nbr.p;
    a.accumulate = 1;
    a.partial = partial;
    a.max_slabs = ctx->slabs_bwd;
    R.tm.begin(&R.st->t_spmm_bwd_ms);
    HT_TRY(ht_spmm_launch(ctx, st, a));
    R.tm.end();
    R.st->n_spmm_bwd += 1;
    R.st->edges += c.nnz;
    R.st->spmm_bwd_alg_bytes += spmm_alg_bytes(c, dn);
  }
  // dW = h^T dt, dH_in += dt W^T over row ranges
  bool first = true;
  for (int64_t r0 = 0; r0 < g->V; r0 += step) {
    const int64_t nr = std::min(step, g->V - r0);
    R.tm.begin(&R.st->t_gemm_ms);
    TnLater later;
    HT_TRY(ht_gemm_tn(ctx, st, H_in->ptr + r0 * H_in->ld, H_in->ld, dT + r0 * ld_t, ld_t, dW, nr, di, dn, first ? 0 : 1, nr == g->V ? &later : nullptr));
    R.tm.end();
    R.st->n_gemm += 1;
    R.st->gemm_flops += 2.0 * nr * di * dn;
    first = false;
    if (dH_in) {
      R.tm.begin(&R.st->t_gemm_ms);
      HT_TRY(ht_gemm_nt(ctx, st, dT + r0 * ld_t, ld_t, W, dH_in->ptr + r0 * dH_in->ld, dH_in->ld, nr, dn, di, R.dhin_fresh ? 0 : 1));
      R.tm.end();
      R.st->n_gemm += 1;
      R.st->gemm_flops += 2.0 * nr * di * dn;
    }
  }
  if (first) HT_TRY(ht_fill_zero(ctx, st, dW, (size_t)di * dn * 4));
  return HT_OK;
}

int finish(Run& R, ht_stats* user, const std::chrono::steady_clock::time_point& t0, bool sync) {
  ht_ctx* ctx = R.ctx;
  if (sync || user) {
    HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
    HT_TRY(R.tm.resolve());
  }
  ctx->ev_next = 0;
  if (user) {
    for (int l = 0; l < HT_MAX_LAYERS; ++l) R.st->t_spmm_fwd_ms += R.st->t_agg_fwd_layer_ms[l];
    R.st->t_spmm_fwd_ms += R.st->t_agg_fix_ms;
    R.st->t_total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    *user = *R.st;
  }
  return HT_OK;
}

}  // namespace

void ht_epoch_ws_free(ht_ctx* ctx) {
  EpochWs* ws = ctx->ws;
  if (!ws) return;
  (void)hipStreamSynchronize(ctx->stream);
  for (size_t i = 0; i < ws->dev_ptrs.size(); ++i) ht_dev_free(ctx, ws->dev_ptrs[i], ws->dev_bytes_of[i]);
  for (void* p : ws->host_ptrs) (void)hipHostFree(p);
  if (ws->graph_exec) (void)hipGraphExecDestroy(ws->graph_exec);
  delete ws;
  ctx->ws = nullptr;
}

namespace {

int ws_tensor(ht_ctx* ctx, EpochWs* ws, int64_t V, int32_t d, int res, ht_tensor* t) {
  t->rows = V;
  t->cols = d;
  t->ld = ht_row_pitch(d, res != HT_RES_HOST);
  const size_t bytes = (size_t)V * t->ld * 4;
  if (res == HT_RES_HOST) {
    void* p = nullptr;
    hipError_t e = hipHostMalloc(&p, bytes, hipHostMallocDefault);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return ht_set_err(ctx, HT_ENOMEM, "hipHostMalloc(%zu): %s", bytes, hipGetErrorString(e));
    }
    ws->host_ptrs.push_back(p);
    t->ptr = (float*)p;
    t->loc = HT_LOC_HOST_PINNED;
  } else {
    void* p = nullptr;
    HT_TRY(ht_dev_alloc(ctx, &p, bytes));
    ws->dev_ptrs.push_back(p);
    ws->dev_bytes_of.push_back(bytes);
    t->ptr = (float*)p;
    t->loc = HT_LOC_DEVICE;
  }
  return HT_OK;
}

int zero_tensor(ht_ctx* ctx, ht_tensor* t) {
  const size_t bytes = (size_t)t->rows * t->ld * 4;
  if (t->loc == HT_LOC_DEVICE) return ht_fill_zero(ctx, ctx->stream, t->ptr, bytes);
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  std::memset(t->ptr, 0, bytes);
  return HT_OK;
}

}  // namespace

extern "C" {

int ht_layer_fwd(ht_ctx* ctx, const ht_graph* g, const ht_layer_desc* desc, const ht_tensor* H_in, const float* W,
                 ht_tensor* H_out, ht_tensor* A_ckpt, ht_stats* stats) {
  if (!ctx) return HT_EINVAL;
  if (!g || !desc || !H_in || !H_out) return ht_set_err(ctx, HT_EINVAL, "ht_layer_fwd: null argument");
  if (g->ctx != ctx) return ht_set_err(ctx, HT_ESTATE, "graph belongs to another context");
  if (desc->d_in <= 0 || desc->d_out <= 0) return ht_set_err(ctx, HT_ESHAPE, "layer widths must be positive");
  HT_HIP(ctx, hipSetDevice(ctx->device));
  if (desc->order != HT_ORDER_AGG_FIRST && desc->order != HT_ORDER_UPDATE_FIRST)
    return ht_set_err(ctx, HT_EINVAL, "unknown stage order %d", desc->order);
  return ht_with_room(ctx, [&]() -> int {
    auto t0 = std::chrono::steady_clock::now();
    ht_stats local{};
    Run R(ctx, g, &local, stats != nullptr);
    R.planned = A_ckpt != nullptr;
    int rc = desc->order == HT_ORDER_UPDATE_FIRST ? layer_fwd_update_first(R, desc, H_in, W, H_out)
                                                  : layer_fwd_impl(R, desc, H_in, W, H_out, A_ckpt);
    if (rc != HT_OK) {
      (void)hipStreamSynchronize(ctx->stream);
      ctx->ev_next = 0;
      return rc;
    }
    return finish(R, stats, t0, false);
  });
}

// ht_layer_fwd for callers that cannot allocate: the kernels of a forward that keeps no aggregate, in the same order (no plan is taken), with the two
// scratch buffers of the all-in-HBM path (the packed copy of W, the partial sums of cut rows) taken from the device's static array.
int ht_layer_fwd_static(ht_ctx* ctx, const ht_graph* g, const ht_layer_desc* desc, const ht_tensor* H_in, const float* W,
                        ht_tensor* H_out, ht_tensor* A_ckpt) {
  if (!ctx) return HT_EINVAL;
  if (!g || !desc || !H_in || !H_out || !A_ckpt || !W) return ht_set_err(ctx, HT_EINVAL, "ht_layer_fwd_static: null argument");
  if (g->ctx != ctx) return ht_set_err(ctx, HT_ESTATE, "graph belongs to another context");
  if (desc->d_in <= 0 || desc->d_out <= 0) return ht_set_err(ctx, HT_ESHAPE, "layer widths must be positive");
  if (desc->order != HT_ORDER_AGG_FIRST) return ht_set_err(ctx, HT_EINVAL, "ht_layer_fwd_static: aggregate-first order only");
  if (desc->gather_mode == HT_GATHER_BUFFER)
    return ht_set_err(ctx, HT_EINVAL, "ht_layer_fwd_static: the neighbour buffer is not available here (rows are read in place)");
  if (H_in->loc != HT_LOC_DEVICE || H_out->loc != HT_LOC_DEVICE || A_ckpt->loc != HT_LOC_DEVICE)
    return ht_set_err(ctx, HT_ESHAPE, "ht_layer_fwd_static: H_in, H_out and A_ckpt must be in HBM");
  // sizes are checked against the static array before anything is launched
  const size_t need_w = (size_t)ht_packed_w_bytes(desc->d_in, desc->d_out);
  const size_t need_p = (size_t)g->max_fpart * (size_t)A_ckpt->ld * 4;
  if (need_w + need_p + 512 > HT_STATIC_SCRATCH_BYTES)
    return ht_set_err(ctx, HT_ENOMEM, "ht_layer_fwd_static: this layer needs %zu bytes of scratch memory (packed W %zu, partial sums "
                      "of %lld cut rows' items %zu); the static array holds %zu: use ht_layer_fwd", need_w + need_p, need_w,
                      (long long)g->max_fpart, need_p, HT_STATIC_SCRATCH_BYTES);
  HT_HIP(ctx, hipSetDevice(ctx->device));
  ht_stats local{};
  Run R(ctx, g, &local, false);
  ht_static_begin(ctx);
  int rc = layer_fwd_impl(R, desc, H_in, W, H_out, A_ckpt);
  ht_static_end(ctx);
  ctx->ev_next = 0;
  if (rc != HT_OK) (void)hipStreamSynchronize(ctx->stream);
  return rc;
}

int ht_layer_bwd(ht_ctx* ctx, const ht_graph* g, const ht_layer_desc* desc, const ht_tensor* ckpt, const float* W,
                 const ht_tensor* dH_out, const ht_tensor* H_out, ht_tensor* dH_in, float* dW, ht_stats* stats) {
  if (!ctx) return HT_EINVAL;
  if (!g || !desc || !ckpt || !dH_out) return ht_set_err(ctx, HT_EINVAL, "ht_layer_bwd: null argument");
  if (g->ctx != ctx) return ht_set_err(ctx, HT_ESTATE, "graph belongs to another context");
  if (desc->d_in <= 0 || desc->d_out <= 0) return ht_set_err(ctx, HT_ESHAPE, "layer widths must be positive");
  HT_HIP(ctx, hipSetDevice(ctx->device));
  if (desc->order != HT_ORDER_AGG_FIRST && desc->order != HT_ORDER_UPDATE_FIRST)
    return ht_set_err(ctx, HT_EINVAL, "unknown stage order %d", desc->order);
  bool changed = false;
  return ht_with_room(ctx, [&]() -> int {
    auto t0 = std::chrono::steady_clock::now();
    ht_stats local{};
    Run R(ctx, g, &local, stats != nullptr);
    R.planned = true;
    int rc = desc->order == HT_ORDER_UPDATE_FIRST ? layer_bwd_update_first(R, desc, ckpt, W, dH_out, H_out, dH_in, dW)
                                                  : layer_bwd_impl(R, desc, ckpt, W, dH_out, H_out, dH_in, dW);
    changed = R.changed;
    if (rc != HT_OK) {
      (void)hipStreamSynchronize(ctx->stream);
      ctx->ev_next = 0;
      return rc;
    }
    return finish(R, stats, t0, false);
  }, &changed);
}

static int epoch_impl(ht_ctx* ctx, const ht_graph* g, const ht_model* model, const ht_tensor* X, const int32_t* labels,
                      const ht_plan_opts* plan, float* loss_out, ht_stats* stats) {
  if (!g || !model || !X || !labels || !loss_out) return ht_set_err(ctx, HT_EINVAL, "ht_epoch: null argument");
  if (g->ctx != ctx) return ht_set_err(ctx, HT_ESTATE, "graph belongs to another context");
  const int L = model->n_layers;
  if (L < 1 || !model->dims || !model->W) return ht_set_err(ctx, HT_EINVAL, "ht_epoch: bad model");
  for (int l = 0; l <= L; ++l)
    if (model->dims[l] <= 0) return ht_set_err(ctx, HT_ESHAPE, "ht_epoch: layer widths must be positive");
  for (int l = 0; l < L; ++l)
    if (!model->W[l]) return ht_set_err(ctx, HT_EINVAL, "ht_epoch: W[%d] is null", l);
  HT_HIP(ctx, hipSetDevice(ctx->device));
  HT_TRY(check_tensor(ctx, X, g->V, model->dims[0], "X"));
  auto t0 = std::chrono::steady_clock::now();
  const int64_t V = g->V;

  // ---- residency plan (Sec. 4.2 sized to this GPU)
  int res_h = plan ? plan->res_h : HT_RES_AUTO, res_a = plan ? plan->res_a : HT_RES_AUTO,
      res_g = plan ? plan->res_g : HT_RES_AUTO;
  int inter = plan ? plan->inter : HT_INTER_AUTO;
  const int gather_mode = plan ? plan->gather_mode : HT_GATHER_AUTO;
  int64_t budget = plan ? plan->hbm_budget_bytes : 0;
  if (budget == 0) {
    budget = ht_device_free(ctx) - ((int64_t)2 << 30);
    // buffers of a previous epoch with the same shape are reused, so count them as free
    if (ctx->ws)
      for (size_t b : ctx->ws->dev_bytes_of) budget += (int64_t)b;
    // so is what calls before this one keep for later ones: it is given back where the tensors need it, and must not move them to the
    // host in the second epoch
    budget += ht_held(ctx);
  }
  auto bytes_of = [&](int l0, int l1) {
    int64_t b = 0;
    for (int l = l0; l <= l1; ++l) b += V * ht_row_pitch(model->dims[l], true) * 4;
    return b;
  };
  int64_t left = budget;
  // the output layer's logits and their gradient stay in HBM (the loss runs on them in place)
  left -= 2 * bytes_of(L, L);
  if (res_g == HT_RES_AUTO) { if (L > 1 && bytes_of(1, L - 1) <= left) { res_g = HT_RES_HBM; left -= bytes_of(1, L - 1); } else res_g = L > 1 ? HT_RES_HOST : HT_RES_HBM; }
  bool a_spills = false;      // the planner, not the caller, put a^l in host memory
  if (inter == HT_INTER_RECOMPUTE) res_a = HT_RES_HBM;   // no checkpoint tensors exist: nothing to place
  else if (res_a == HT_RES_AUTO) {
    if (bytes_of(0, L - 1) <= left) { res_a = HT_RES_HBM; left -= bytes_of(0, L - 1); }
    else { res_a = HT_RES_HOST; a_spills = true; }
  }
  if (res_h == HT_RES_AUTO) { if (L > 1 && bytes_of(1, L - 1) <= left) { res_h = HT_RES_HBM; left -= bytes_of(1, L - 1); } else res_h = L > 1 ? HT_RES_HOST : HT_RES_HBM; }
  if (inter == HT_INTER_AUTO && a_spills) {
    // Sec. 4.2's trade-off priced for this GPU.  Host-side cache: a^l crosses the link twice.  Recomputation:
    // the rows of a host-resident h^l that the buffer schedule loads cross it once more, and every layer
    // is aggregated a second time.
    double t_cache = 0.0, t_again = 0.0;
    const double pairs = (double)(g->merged ? g->n_unique : g->Ep);
    for (int l = 0; l < L; ++l) {
      const double row = 4.0 * (double)model->dims[l];
      const bool in_host = l == 0 ? X->loc == HT_LOC_HOST_PINNED : res_h == HT_RES_HOST;
      t_cache += 2.0 * (double)V * row / HT_LINK_BYTES_PER_S;
      t_again += (in_host ? (double)g->v_load * row / HT_LINK_BYTES_PER_S : 0.0) + pairs * row / HT_GATHER_BYTES_PER_S;
    }
    if (t_again < t_cache) {
      inter = HT_INTER_RECOMPUTE;
      res_a = HT_RES_HBM;
    }
  }
  if (inter == HT_INTER_AUTO) inter = res_h == HT_RES_HBM ? HT_INTER_MASK : HT_INTER_HYBRID;
  if (inter != HT_INTER_MASK && inter != HT_INTER_HYBRID && inter != HT_INTER_RECOMPUTE)
    return ht_set_err(ctx, HT_EINVAL, "ht_epoch: unknown intermediate-data mode %d", inter);
  const bool recompute = inter == HT_INTER_RECOMPUTE;
  // ---- stage order per layer: update-first only where every tensor of the layer is in HBM
  const int order = plan ? plan->order : HT_ORDER_AGG_FIRST;
  if (order != HT_ORDER_AGG_FIRST && order != HT_ORDER_UPDATE_FIRST && order != HT_ORDER_AUTO)
    return ht_set_err(ctx, HT_EINVAL, "ht_epoch: unknown stage order %d", order);
  const bool want_reuse0 = plan && plan->reuse_input_aggregate && !recompute;
  uint32_t upd_mask = 0;
  if (order != HT_ORDER_AGG_FIRST && L <= 32 && gather_mode != HT_GATHER_BUFFER) {
    for (int l = want_reuse0 ? 1 : 0; l < L; ++l) {   // (a^0 is only kept by the printed stage order)
      const bool in_hbm = l == 0 ? X->loc == HT_LOC_DEVICE : res_h == HT_RES_HBM;
      const bool out_hbm = l == L - 1 || res_h == HT_RES_HBM;
      const bool gout_hbm = l == L - 1 || res_g == HT_RES_HBM;
      const bool gin_hbm = l == 0 || res_g == HT_RES_HBM;
      const bool narrower = model->dims[l + 1] < model->dims[l];
      if (in_hbm && out_hbm && gout_hbm && gin_hbm && (order == HT_ORDER_UPDATE_FIRST || narrower)) upd_mask |= 1u << l;
    }
  }

  // ---- workspace
  EpochWs* ws = ctx->ws;
  bool reuse = ws && ws->V == V && (int)ws->dims.size() == L + 1 && ws->res_h == res_h && ws->res_a == res_a &&
               ws->res_g == res_g && ws->upd_mask == upd_mask && ws->no_ckpt == recompute;
  if (reuse)
    for (int l = 0; l <= L; ++l) reuse = reuse && ws->dims[l] == model->dims[l];
  const bool reuse0 = reuse && want_reuse0 && ws->a0_of == X->ptr && ws->a0_graph == g->serial && ws->a[0].ptr;
  if (!reuse) {
    ht_epoch_ws_free(ctx);
    ws = new (std::nothrow) EpochWs();
    if (!ws) return ht_set_err(ctx, HT_ENOMEM, "ht_epoch: host allocation failed");
    ctx->ws = ws;
    ws->V = V;
    ws->dims.assign(model->dims, model->dims + L + 1);
    ws->res_h = res_h; ws->res_a = res_a; ws->res_g = res_g;
    ws->upd_mask = upd_mask;
    ws->no_ckpt = recompute;
    ws->h.assign(L + 1, ht_tensor{});
    ws->a.assign(L, ht_tensor{});
    ws->gh.assign(L + 1, ht_tensor{});
    ws->dW.assign(L, nullptr);
    int rc = HT_OK;
    for (int l = 1; l <= L && rc == HT_OK; ++l) rc = ws_tensor(ctx, ws, V, model->dims[l], l == L ? HT_RES_HBM : res_h, &ws->h[l]);
    for (int l = 0; l < L && rc == HT_OK; ++l)
      if (!((upd_mask >> l) & 1) && !recompute) rc = ws_tensor(ctx, ws, V, model->dims[l], res_a, &ws->a[l]);
    for (int l = 1; l <= L && rc == HT_OK; ++l) rc = ws_tensor(ctx, ws, V, model->dims[l], l == L ? HT_RES_HBM : res_g, &ws->gh[l]);
    for (int l = 0; l < L && rc == HT_OK; ++l) {
      void* p = nullptr;
      const size_t b = (size_t)model->dims[l] * model->dims[l + 1] * 4;
      rc = ht_dev_alloc(ctx, &p, b);
      if (rc == HT_OK) { ws->dW[l] = (float*)p; ws->dev_ptrs.push_back(p); ws->dev_bytes_of.push_back(b); }
    }
    if (rc != HT_OK) {
      ht_epoch_ws_free(ctx);
      return rc;
    }
  }

  ht_stats local{};
  Run R(ctx, g, &local, stats != nullptr);
  R.planned = true;
  R.again_ok = recompute && res_h == HT_RES_HBM && res_g == HT_RES_HBM && gather_mode != HT_GATHER_BUFFER;
  if (plan && plan->stats_detail == HT_STATS_AGG_FWD) {
    R.tm.only_lo = &local.t_agg_fwd_layer_ms[0];
    R.tm.only_hi = &local.t_agg_fwd_layer_ms[0] + HT_MAX_LAYERS;
  } else if (plan && plan->stats_detail != HT_STATS_ALL)
    return ht_set_err(ctx, HT_EINVAL, "ht_epoch: unknown stats_detail %d", plan->stats_detail);
  auto fail = [&](int rc) {
    (void)hipStreamSynchronize(ctx->stream);
    (void)ht_flush_products(ctx, ctx->stream, true);
    ctx->ev_next = 0;
    return rc;
  };
  // Host-resident gradient tensors that the backward pass adds into start as zeros.  They are not
  // touched before the backward pass, so a helper thread clears them beside the forward pass
  // instead of the GPU waiting for a memset between two layers.
  auto stored_once = [&](int l) {   // a never-evicting gradient buffer stores every row of a host-resident grad h^l exactly once
    return g->single_leave && g->v_load == V && ws->gh[l].loc == HT_LOC_HOST_PINNED && gather_mode != HT_GATHER_DIRECT;
  };
  struct Joiner {
    std::thread th;
    ~Joiner() { if (th.joinable()) th.join(); }
  } zeroer;
  {
    std::vector<ht_tensor*> todo;
    for (int l = 1; l < L; ++l)
      if (ws->gh[l].loc == HT_LOC_HOST_PINNED && !stored_once(l)) todo.push_back(&ws->gh[l]);
    if (!todo.empty())
      zeroer.th = std::thread([todo] {
        for (ht_tensor* t : todo) std::memset(t->ptr, 0, (size_t)t->rows * t->ld * 4);
      });
  }
  // ---- the epoch's stream work.  With every tensor in HBM it is kernels on one stream only, so it
  // can be recorded once into a HIP graph and replayed (ht_plan_opts.use_graph): the first epoch of a
  // key runs eagerly (it sizes the scratch memory, which a capture may not allocate), the second is
  // captured, instantiated and launched, later ones are one graph launch.
  bool in_capture = false;
  float *loss_host = nullptr, *loss_gpu = nullptr;
  HT_TRY(ht_host_scratch(ctx, HT_HS_LOSS, 64, (void**)&loss_host));
  HT_HIP(ctx, hipHostGetDevicePointer((void**)&loss_gpu, loss_host, 0));
  auto enqueue = [&]() -> int {
    std::vector<size_t> products;
    for (int l = 0; l < L; ++l)
      products.push_back((upd_mask >> l) & 1 ? ht_gemm_tn_bytes(V, model->dims[l], model->dims[l + 1])
                                             : ht_gemm_groups_bytes(model->dims[l], model->dims[l + 1], g->dense_groups));
    HT_TRY(ht_defer_products(ctx, products));
    // ---- forward (Alg. 1)
    for (int l = 0; l < L; ++l) {
      ht_layer_desc d{};
      d.d_in = model->dims[l]; d.d_out = model->dims[l + 1];
      d.act = l < L - 1 ? HT_ACT_RELU : HT_ACT_NONE;
      d.gather_mode = gather_mode;
      R.layer = l;
      const bool upd = (upd_mask >> l) & 1;
      d.order = upd ? HT_ORDER_UPDATE_FIRST : HT_ORDER_AGG_FIRST;
      int rc = upd                ? layer_fwd_update_first(R, &d, l == 0 ? X : &ws->h[l], model->W[l], &ws->h[l + 1])
               : (l == 0 && reuse0) ? layer_fwd_from_ckpt(R, &d, &ws->a[0], model->W[0], &ws->h[1])
                                    : layer_fwd_impl(R, &d, l == 0 ? X : &ws->h[l], model->W[l], &ws->h[l + 1],
                                                     recompute ? nullptr : &ws->a[l]);
      if (rc != HT_OK) {
        ws->a0_of = nullptr;
        return rc;
      }
      if (l == 0) {   // a^0 = A_hat X is in a[0] from here on (the backward pass only reads it)
        const bool kept = !upd && !recompute;
        ws->a0_of = kept ? X->ptr : nullptr;
        ws->a0_graph = kept ? g->serial : 0;
      }
    }
    // ---- downstream task and its gradient (Alg. 1)
    LossParts loss_parts{};
    {
      R.tm.begin(&R.st->t_loss_ms);
      int rc = ht_softmax_ce(ctx, ctx->stream, ws->h[L].ptr, ws->h[L].ld, labels, V, model->dims[L], ws->gh[L].ptr,
                             ws->gh[L].ld, &loss_parts);
      R.tm.end();
      if (rc != HT_OK) return rc;
    }
    if (in_capture)
      if (const char* dbg = getenv("HT_GRAPH_DEBUG"))
        if (atoi(dbg) == 3) {   // a launch the runtime rejects on the host, to exercise the fallback after a broken capture
          k_noop<<<1, 4096, 0, ctx->stream>>>();
          HT_LAUNCH_CHECK(ctx);
        }
    // ---- backward (Alg. 1)
    for (int l = L - 1; l >= 0; --l) {
      ht_layer_desc d{};
      d.d_in = model->dims[l]; d.d_out = model->dims[l + 1];
      d.act = l < L - 1 ? HT_ACT_RELU : HT_ACT_NONE;
      d.gather_mode = gather_mode;
      d.ckpt_kind = recompute ? HT_CKPT_INPUT : HT_CKPT_AGG;
      R.dhin_fresh = false;
      if (l > 0) {
        // a host-resident tensor is cleared beside the forward pass (or stored exactly once)
        if (ws->gh[l].loc == HT_LOC_HOST_PINNED && zeroer.th.joinable()) zeroer.th.join();
        R.dhin_fresh = true;
      }
      R.layer = l;
      const bool mask_ok = inter == HT_INTER_MASK || (recompute && ws->h[l + 1].loc == HT_LOC_DEVICE);
      const ht_tensor* mask_from = (mask_ok && l < L - 1) ? &ws->h[l + 1] : nullptr;
      const ht_tensor* ckpt = recompute ? (l == 0 ? X : &ws->h[l]) : &ws->a[l];
      const bool upd = (upd_mask >> l) & 1;
      d.order = upd ? HT_ORDER_UPDATE_FIRST : HT_ORDER_AGG_FIRST;
      int rc = upd ? layer_bwd_update_first(R, &d, l == 0 ? X : &ws->h[l], model->W[l], &ws->gh[l + 1],
                                            l < L - 1 ? &ws->h[l + 1] : nullptr, l > 0 ? &ws->gh[l] : nullptr, ws->dW[l])
                   : layer_bwd_impl(R, &d, ckpt, model->W[l], &ws->gh[l + 1], mask_from,
                                    l > 0 ? &ws->gh[l] : nullptr, ws->dW[l]);
      if (rc != HT_OK) return rc;
    }
    // ---- parameter update (Alg. 1)
    R.tm.begin(&R.st->t_update_ms);
    std::vector<ht_sgd_item> params;
    for (int l = 0; l < L; ++l) params.push_back({model->W[l], ws->dW[l], (int64_t)model->dims[l] * model->dims[l + 1]});
    HT_TRY(ht_step(ctx, ctx->stream, params, model->lr, loss_parts, loss_gpu));
    R.tm.end();
    return HT_OK;
  };
  const bool all_hbm = X->loc == HT_LOC_DEVICE && res_h == HT_RES_HBM && res_g == HT_RES_HBM && (recompute || res_a == HT_RES_HBM);
  std::vector<uintptr_t> key;
  if (plan && plan->use_graph && all_hbm && !stats) {
    key = {(uintptr_t)g->serial, (uintptr_t)ctx->scratch_gen, (uintptr_t)X->ptr, (uintptr_t)X->ld, (uintptr_t)labels, (uintptr_t)inter, (uintptr_t)upd_mask,
           (uintptr_t)reuse0, (uintptr_t)gather_mode, (uintptr_t)L};
    uint32_t lr_bits;
    std::memcpy(&lr_bits, &model->lr, 4);
    key.push_back(lr_bits);
    for (int l = 0; l < L; ++l) key.push_back((uintptr_t)model->W[l]);
  }
  bool launched = false;
  if (!key.empty() && ws->graph_exec && ws->graph_key == key) {
    hipError_t e = hipGraphLaunch(ws->graph_exec, ctx->stream);
    if (e != hipSuccess) return fail(ht_set_err(ctx, HT_EHIP, "hipGraphLaunch: %s", hipGetErrorString(e)));
    launched = true;
    ++ctx->graph_launches;
  } else if (!key.empty() && ws->warm_key == key && ws->bad_key != key) {
    if (ws->graph_exec) {
      (void)hipGraphExecDestroy(ws->graph_exec);
      ws->graph_exec = nullptr;
      ws->graph_key.clear();
    }
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamBeginCapture(ctx->stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return fail(ht_set_err(ctx, HT_EHIP, "hipStreamBeginCapture: %s", hipGetErrorString(e)));
    in_capture = ctx->no_grow = true;
    int rc = enqueue();
    in_capture = ctx->no_grow = false;
    e = hipStreamEndCapture(ctx->stream, &graph);
    if (const char* dbg = getenv("HT_GRAPH_DEBUG"))
      if (atoi(dbg) == 2 && rc == HT_OK) rc = ht_set_err(ctx, HT_ESTATE, "capture discarded on request");   // exercises the fallback
    if (rc == HT_OK && e == hipSuccess && graph) {
      e = hipGraphInstantiate(&ws->graph_exec, graph, nullptr, nullptr, 0);
      if (e == hipSuccess) e = hipGraphLaunch(ws->graph_exec, ctx->stream);
      if (e == hipSuccess) {
        ws->graph_key = key;
        launched = true;
        ++ctx->graph_launches;
      } else if (ws->graph_exec) {
        (void)hipGraphExecDestroy(ws->graph_exec);
        ws->graph_exec = nullptr;
      }
    }
    if (graph) (void)hipGraphDestroy(graph);
    if (rc != HT_OK) (void)ht_flush_products(ctx, ctx->stream, true);
    if (!launched) {   // nothing has run: this epoch runs eagerly below, and the key is not tried again
      if (getenv("HT_GRAPH_DEBUG"))
        fprintf(stderr, "ht_epoch: graph capture failed (enqueue rc %d: %s; hip: %s)\n", rc, ctx->err.c_str(), hipGetErrorString(e));
      (void)hipGetLastError();
      ws->bad_key = key;
      ws->a0_of = reuse0 ? ws->a0_of : nullptr;
    }
  }
  if (!launched) {
    const int rc = enqueue();
    if (rc != HT_OK) return fail(rc);
    ws->warm_key = key;
  }
  local.plan_inter = inter;
  local.plan_res_h = res_h;
  local.plan_res_a = recompute ? 0 : res_a;
  local.plan_res_g = res_g;
  HT_TRY(finish(R, stats, t0, true));
  *loss_out = *(volatile float*)loss_host;
  return HT_OK;
}

int ht_epoch(ht_ctx* ctx, const ht_graph* g, const ht_model* model, const ht_tensor* X, const int32_t* labels,
             const ht_plan_opts* plan, float* loss_out, ht_stats* stats) {
  if (!ctx) return HT_EINVAL;
  // (the caller's weights change in the last launch, behind everything that takes memory)
  return ht_with_room(ctx, [&] { return epoch_impl(ctx, g, model, X, labels, plan, loss_out, stats); });
}

int ht_tensor_zero(ht_ctx* ctx, ht_tensor* t) {
  if (!ctx) return HT_EINVAL;
  if (!t || !t->ptr || t->rows < 0 || t->ld < t->cols || (t->ld & 3))
    return ht_set_err(ctx, HT_EINVAL, "ht_tensor_zero: bad tensor");
  HT_HIP(ctx, hipSetDevice(ctx->device));
  HT_TRY(zero_tensor(ctx, t));
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return HT_OK;
}

int ht_epoch_buffer(ht_ctx* ctx, int32_t kind, int32_t layer, ht_tensor* out) {
  if (!ctx || !out) return HT_EINVAL;
  EpochWs* ws = ctx->ws;
  if (!ws) return ht_set_err(ctx, HT_ESTATE, "no epoch has run on this context");
  const int L = (int)ws->dims.size() - 1;
  switch (kind) {
    case HT_BUF_H:
      if (layer < 1 || layer > L) return ht_set_err(ctx, HT_EINVAL, "layer out of range");
      *out = ws->h[layer];
      return HT_OK;
    case HT_BUF_A:
      if (layer < 0 || layer >= L) return ht_set_err(ctx, HT_EINVAL, "layer out of range");
      if (!ws->a[layer].ptr) return ht_set_err(ctx, HT_ESTATE, "layer %d keeps no aggregate checkpoint", layer);
      *out = ws->a[layer];
      return HT_OK;
    case HT_BUF_GH:
      if (layer < 1 || layer > L) return ht_set_err(ctx, HT_EINVAL, "layer out of range");
      *out = ws->gh[layer];
      return HT_OK;
    case HT_BUF_DW:
      if (layer < 0 || layer >= L) return ht_set_err(ctx, HT_EINVAL, "layer out of range");
      out->ptr = ws->dW[layer];
      out->rows = ws->dims[layer];
      out->cols = ws->dims[layer + 1];
      out->ld = ws->dims[layer + 1];
      out->loc = HT_LOC_DEVICE;
      return HT_OK;
    default:
      return ht_set_err(ctx, HT_EINVAL, "unknown buffer kind %d", kind);
  }
}

int ht_tensor_to_host(ht_ctx* ctx, const ht_tensor* t, float* dst) {
  if (!ctx || !t || !dst) return HT_EINVAL;
  if (!t->ptr || t->rows < 0 || t->cols <= 0 || t->ld < t->cols) return ht_set_err(ctx, HT_ESHAPE, "bad tensor");
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  if (t->rows == 0) return HT_OK;
  // rows [r0, r1) of `from` (pitch ld) into the dense destination, on the host cores
  auto pack = [&](const float* from, int64_t r0, int64_t r1) {
    const int nt = (int)std::min<int64_t>(host_threads(ctx), std::max<int64_t>(1, (r1 - r0) / 4096));
    auto work = [&](int64_t a, int64_t b) {
      for (int64_t r = a; r < b; ++r)
        std::memcpy(dst + r * t->cols, from + (r - r0) * t->ld, (size_t)t->cols * 4);
    };
    if (nt <= 1) return work(r0, r1);
    std::vector<std::thread> th;
    const int64_t per = (r1 - r0 + nt - 1) / nt;
    for (int k = 0; k < nt; ++k) {
      const int64_t a = r0 + k * per, b = std::min(r1, a + per);
      if (a < b) th.emplace_back(work, a, b);
    }
    for (auto& x : th) x.join();
  };
  if (t->loc != HT_LOC_DEVICE) {
    pack(t->ptr, 0, t->rows);
    return HT_OK;
  }
  // HBM: whole padded rows through a page-locked bounce buffer (a pitched copy into pageable
  // memory runs at a fraction of the link rate), then packed on the host
  const int64_t rows_per = std::max<int64_t>(1, ((int64_t)64 << 20) / (t->ld * 4));
  float* bounce = nullptr;
  HT_TRY(ht_host_scratch(ctx, 1, (size_t)rows_per * t->ld * 4, (void**)&bounce));
  for (int64_t r0 = 0; r0 < t->rows; r0 += rows_per) {
    const int64_t r1 = std::min(t->rows, r0 + rows_per);
    HT_HIP(ctx, hipMemcpy(bounce, t->ptr + r0 * t->ld, (size_t)(r1 - r0) * t->ld * 4, hipMemcpyDeviceToHost));
    pack(bounce, r0, r1);
  }
  return HT_OK;
}

}  // extern "C"
