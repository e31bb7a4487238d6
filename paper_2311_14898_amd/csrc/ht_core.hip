// Context, error reporting, allocation accounting, event timers.
#include <algorithm>
#include <cstdarg>
#include <cstdlib>

#include "ht_internal.h"

#include <mutex>

// Scratch memory of the allocation-free entry point (ht_layer_fwd_static): part of the code object, so every GPU the
// library runs on holds HT_STATIC_SCRATCH_BYTES of it from load to exit, and no call has to allocate.  In host code
// this name is only a handle for hipGetSymbolAddress; kernels get the device address taken below.  (No
// __attribute__((used)) here: it pins the device symbol to local binding, and the runtime, which finds the variable
// by name in the code object, aborts when it cannot; referenced from host code alone the compiler exports it.)
static __device__ __align__(256) unsigned char scratch[HT_STATIC_SCRATCH_BYTES];

namespace {
constexpr int HT_MAX_DEVICES = 64;
std::mutex g_static_mu;
unsigned char* g_static_ptr[HT_MAX_DEVICES] = {};

// Address of `scratch` on the current device (each GPU has its own copy at its own address); taken once per device.
int static_scratch_address(int device, unsigned char** out) {
  *out = nullptr;
  if (device < 0 || device >= HT_MAX_DEVICES) return HT_EINVAL;
  std::lock_guard<std::mutex> lk(g_static_mu);
  if (!g_static_ptr[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return HT_EHIP;
    }
    g_static_ptr[device] = (unsigned char*)p;
  }
  *out = g_static_ptr[device];
  return HT_OK;
}
thread_local bool g_orphans = false;   // what is being freed belonged to a context that is gone
}  // namespace

void ht_free_orphan(ht_graph* g) {
  g_orphans = true;
  delete g;
  g_orphans = false;
}

void ht_static_begin(ht_ctx* ctx) {
  ctx->static_mode = true;
  ctx->static_used = 0;
  for (int i = 0; i < HT_N_SCRATCH; ++i) ctx->static_off[i] = ctx->static_len[i] = 0;
}

void ht_static_end(ht_ctx* ctx) { ctx->static_mode = false; }

int ht_set_err(ht_ctx* ctx, int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  if (ctx) ctx->err = buf;
  return code;
}

// An allocation or a release costs 50 to 200 us of the host, a release some 3 ms per GiB, and makes the device idle; a graph that is
// seen once takes a dozen blocks.  Blocks that a context frees are therefore kept and handed out again, to the same context, where they fit well:
// work on a context's stream is in order, and what runs beside it is waited for by that stream before a call ends.  A context keeps up to
// HT_KEPT_BYTES, those of a device together up to HT_KEPT_ALL.  Nothing is kept under a byte budget, nor of scratch slots once a caller has recorded a pass, which works in
// them; a graph's end keeps nothing where less than an eighth of the device is free; and whatever any context keeps is given back where an
// allocation of another fails, by ht_ctx_set_hbm_budget and with the context.  Partition and one layer of a graph seen once: 10 k vertices 567 -> 502 us,
// 2.45 M vertices, 62 M edges 14.8 -> 13.6 ms.
namespace {
struct KeptBlock {
  void* p;
  size_t bytes;
  ht_ctx* ctx;
};
std::mutex g_kept_lock;              // contexts may be used by several threads, one each
std::vector<KeptBlock>& g_kept = *new std::vector<KeptBlock>();       // oldest first (contexts may be destroyed as late as they like)

// Takes the blocks that `which` says off the list and releases them.
template <class F>
void kept_drop(F&& which) {
  std::vector<KeptBlock> drop;
  {
    std::lock_guard<std::mutex> hold(g_kept_lock);
    const auto keep = std::stable_partition(g_kept.begin(), g_kept.end(), [&](const KeptBlock& k) { return !which(k); });
    drop.assign(keep, g_kept.end());
    g_kept.erase(keep, g_kept.end());
  }
  if (drop.empty()) return;
  (void)hipDeviceSynchronize();      // (a context's own work may still be on them)
  for (const KeptBlock& k : drop) (void)hipFree(k.p);
}
size_t kept_bytes(int device) {
  std::lock_guard<std::mutex> hold(g_kept_lock);
  size_t sum = 0;
  for (const KeptBlock& k : g_kept) sum += k.ctx->device == device ? k.bytes : 0;
  return sum;
}
// The smallest of the context's blocks that fits `bytes` well.
bool kept_take(ht_ctx* ctx, size_t bytes, KeptBlock* out) {
  std::lock_guard<std::mutex> hold(g_kept_lock);
  auto best = g_kept.end();
  for (auto k = g_kept.begin(); k != g_kept.end(); ++k)
    if (k->ctx == ctx && k->bytes >= bytes && k->bytes <= bytes + bytes / 4 + 65536 && (best == g_kept.end() || k->bytes < best->bytes)) best = k;
  if (best == g_kept.end()) return false;
  *out = *best;
  g_kept.erase(best);
  return true;
}
// false: the caller releases it.  The context's oldest blocks make room for it.
bool kept_put(ht_ctx* ctx, void* p, size_t bytes) {
  std::vector<KeptBlock> drop;
  bool put = true;
  {
    std::lock_guard<std::mutex> hold(g_kept_lock);
    for (;;) {
      size_t all = bytes, own = bytes, blocks = 0;
      auto oldest = g_kept.end();
      for (auto k = g_kept.begin(); k != g_kept.end(); ++k) {
        if (k->ctx->device != ctx->device) continue;
        all += k->bytes;
        if (k->ctx != ctx) continue;
        own += k->bytes;
        ++blocks;
        if (oldest == g_kept.end()) oldest = k;
      }
      if (own <= HT_KEPT_BYTES && all <= HT_KEPT_ALL && blocks < HT_KEPT_BLOCKS) break;
      if (oldest == g_kept.end()) {
        put = false;
        break;
      }
      drop.push_back(*oldest);
      g_kept.erase(oldest);
    }
    if (put) g_kept.push_back(KeptBlock{p, bytes, ctx});
  }
  for (const KeptBlock& k : drop) (void)hipFree(k.p);
  return put;
}
}  // namespace

void ht_kept_release(ht_ctx* ctx) {
  kept_drop([&](const KeptBlock& k) { return k.ctx == ctx; });
}

void ht_kept_trim(ht_ctx* ctx) {
  if (kept_bytes(ctx->device) < ((size_t)64 << 20)) return;
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  if (ctx->device_bytes > 0) {
    total_b = (size_t)ctx->device_bytes;
    free_b = (size_t)std::max<int64_t>(0, ctx->device_bytes - ctx->hbm_used);
  }
  if (free_b < total_b / 8) ht_kept_release(ctx);
}

int ht_dev_alloc(ht_ctx* ctx, void** out, size_t bytes) {
  *out = nullptr;
  if (bytes == 0) return HT_OK;
  if (ctx->static_mode) return ht_set_err(ctx, HT_ESTATE, "a device allocation of %zu bytes was asked for inside the allocation-free entry point", bytes);
  if (ctx->hbm_budget > 0 && ctx->hbm_used + (int64_t)bytes > ctx->hbm_budget)
    return ht_set_err(ctx, HT_ENOMEM, "HBM budget exceeded: %lld in use + %zu requested > %lld",
                      (long long)ctx->hbm_used, bytes, (long long)ctx->hbm_budget);
  if (ctx->refuse_alloc > 0 && --ctx->refuse_alloc == 0) return ht_set_err(ctx, HT_ENOMEM, "allocation of %zu bytes refused (HT_REFUSE_ALLOC)", bytes);
  KeptBlock k;
  if (kept_take(ctx, bytes, &k)) {
    if (k.bytes != bytes) ctx->larger[k.p] = k.bytes;
    *out = k.p;
    ctx->hbm_used += (int64_t)bytes;
    return HT_OK;
  }
  const bool refuse = ctx->refuse_alloc < 0 && ++ctx->refuse_alloc == 0;
  hipError_t e = refuse ? hipErrorOutOfMemory : hipMalloc(out, bytes);
  if (e != hipSuccess && kept_bytes(ctx->device) > 0) {
    (void)hipGetLastError();
    kept_drop([&](const KeptBlock& b) { return b.ctx->device == ctx->device; });
    e = hipMalloc(out, bytes);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    *out = nullptr;
    return ht_set_err(ctx, HT_ENOMEM, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
  }
  ctx->hbm_used += (int64_t)bytes;
  return HT_OK;
}

static void dev_free(ht_ctx* ctx, void* p, size_t bytes, bool keep) {
  if (!p) return;
  if (!ctx || g_orphans) {      // (the context is gone)
    (void)hipFree(p);
    return;
  }
  ctx->hbm_used -= (int64_t)bytes;
  size_t have = bytes;          // what the block really holds
  const auto it = ctx->larger.find(p);
  if (it != ctx->larger.end()) {
    have = it->second;
    ctx->larger.erase(it);
  }
  if (!keep || ctx->hbm_budget > 0 || have > HT_KEPT_BYTES || !kept_put(ctx, p, have)) (void)hipFree(p);
}
void ht_dev_free(ht_ctx* ctx, void* p, size_t bytes) { dev_free(ctx, p, bytes, true); }

static size_t ht_scratch_size(size_t bytes) { return bytes + bytes / 8 + 256; }   // of a slot that is asked for so many

int ht_scratch(ht_ctx* ctx, int slot, size_t bytes, void** out) {
  if (ctx->static_mode) {
    // a piece of the static array per slot: cut at the slot's first request of this call, kept for its later ones
    *out = nullptr;
    if (!ctx->static_base) return ht_set_err(ctx, HT_ESTATE, "the static scratch array has no address on this device");
    if (ctx->static_len[slot] < bytes) {
      if (ctx->static_len[slot] != 0)
        return ht_set_err(ctx, HT_ESTATE, "scratch slot %d grew from %zu to %zu bytes inside one allocation-free call", slot,
                          ctx->static_len[slot], bytes);
      const size_t off = (ctx->static_used + 255) & ~(size_t)255;
      if (bytes > HT_STATIC_SCRATCH_BYTES || off > HT_STATIC_SCRATCH_BYTES - bytes)
        return ht_set_err(ctx, HT_ENOMEM, "the allocation-free entry point needs %zu more bytes of scratch memory (slot %d) after "
                          "%zu in use; its static array holds %zu: use the allocating entry point for this size", bytes, slot,
                          ctx->static_used, HT_STATIC_SCRATCH_BYTES);
      ctx->static_off[slot] = off;
      ctx->static_len[slot] = bytes;
      ctx->static_used = off + bytes;
    }
    *out = ctx->static_base + ctx->static_off[slot];
    return HT_OK;
  }
  if (ctx->scratch_bytes[slot] < bytes) {
    if (ctx->scratch[slot]) {
      if (slot == HT_S_TNPART) HT_TRY(ht_flush_products(ctx, ctx->stream));   // (sums that were left to the end of the epoch are in there)
      HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
      dev_free(ctx, ctx->scratch[slot], ctx->scratch_bytes[slot], !ctx->recorded);
      ctx->scratch[slot] = nullptr;
      ctx->scratch_bytes[slot] = 0;
    }
    const size_t want = ht_scratch_size(bytes);
    int rc = ht_dev_alloc(ctx, &ctx->scratch[slot], want);
    if (rc != HT_OK) return rc;
    ctx->scratch_bytes[slot] = want;
    ++ctx->scratch_gen;
  }
  *out = ctx->scratch[slot];
  return HT_OK;
}

int ht_scratch_release(ht_ctx* ctx, int slot) {
  if (ctx->static_mode || !ctx->scratch[slot]) return HT_OK;
  if (slot == HT_S_TNPART) HT_TRY(ht_flush_products(ctx, ctx->stream));
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  dev_free(ctx, ctx->scratch[slot], ctx->scratch_bytes[slot], !ctx->recorded);
  ctx->scratch[slot] = nullptr;
  ctx->scratch_bytes[slot] = 0;
  ++ctx->scratch_gen;
  return HT_OK;
}

int64_t ht_device_free(ht_ctx* ctx) {
  int64_t room = INT64_MAX;
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) == hipSuccess) room = (int64_t)(free_b + kept_bytes(ctx->device));
  else (void)hipGetLastError();
  if (ctx->device_bytes > 0) room = std::min(room, std::max<int64_t>(0, ctx->device_bytes - ctx->hbm_used));
  return room;
}

int64_t ht_room(ht_ctx* ctx) {
  int64_t room = ht_device_free(ctx);
  if (ctx->hbm_budget > 0) room = std::min(room, std::max<int64_t>(0, ctx->hbm_budget - ctx->hbm_used));
  return room;
}

ScratchMark::ScratchMark(ht_ctx* c) : ctx(c) { std::copy(c->scratch_bytes, c->scratch_bytes + HT_N_SCRATCH, was); }
void ScratchMark::undo() {
  for (int k = 0; k < HT_N_SCRATCH; ++k)
    if (ctx->scratch_bytes[k] > was[k] && !(k == HT_S_LIST && ctx->list_owner)) (void)ht_scratch_release(ctx, k);
}

int ht_scratch_all(ht_ctx* ctx, const std::vector<ScratchWant>& want, int64_t beside) {
  size_t need[HT_N_SCRATCH] = {};
  for (const ScratchWant& w : want) need[w.slot] = std::max(need[w.slot], w.bytes);
  int64_t grow = beside, freed = 0;
  for (int k = 0; k < HT_N_SCRATCH; ++k)
    if (need[k] > ctx->scratch_bytes[k]) {
      grow += (int64_t)ht_scratch_size(need[k]);
      freed += (int64_t)ctx->scratch_bytes[k];
    }
  if (grow == 0) return HT_OK;
  if (ctx->no_grow || grow - freed > ht_room(ctx)) return HT_ENOMEM;
  ScratchMark mark(ctx);
  for (int k = 0; k < HT_N_SCRATCH; ++k) {
    void* p = nullptr;
    const int rc = need[k] > 0 ? ht_scratch(ctx, k, need[k], &p) : HT_OK;
    if (rc == HT_OK) continue;
    mark.undo();
    if (rc == HT_ENOMEM) ctx->tight_room = ht_room(ctx);   // (there was room by the figures, and yet none)
    return rc;
  }
  return HT_OK;
}

int ht_scratch_each(ht_ctx* ctx, const std::vector<ScratchWant>& want) {
  for (const ScratchWant& w : want) {
    void* p = nullptr;
    HT_TRY(ht_scratch(ctx, w.slot, w.bytes, &p));
  }
  return HT_OK;
}

bool ht_may_spend(ht_ctx* ctx) {
  if (ctx->lean) return false;
  if (ctx->tight_room < 0) return true;
  if (ctx->no_grow || ht_room(ctx) <= ctx->tight_room) return false;
  ctx->tight_room = -1;
  return true;
}

int64_t ht_held(const ht_ctx* ctx) {
  int64_t held = 0;
  for (size_t b : ctx->scratch_bytes) held += (int64_t)b;
  for (const ht_graph* g : ctx->graphs)
    held += (int64_t)((g == ctx->list_owner ? 0 : g->by_src.blk.mem.bytes()) + g->by_src.mult.bytes()) + g->plan_fwd.bytes() + g->plan_bwd.bytes() +
            (int64_t)g->ranks.mem.mem.bytes();
  return held;
}

bool ht_caller_captures(ht_ctx* ctx) {
  hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(ctx->stream, &capturing) != hipSuccess || capturing != hipStreamCaptureStatusNone;
}

bool ht_give_back(ht_ctx* ctx) {
  if (ctx->static_mode || ctx->no_grow || ctx->lean || ht_held(ctx) == 0) return false;
  if (ht_caller_captures(ctx)) return false;
  (void)hipStreamSynchronize(ctx->stream);
  for (hipStream_t s : ctx->side) (void)hipStreamSynchronize(s);
  for (int k = 0; k < HT_N_SCRATCH; ++k) (void)ht_scratch_release(ctx, k);
  for (const ht_graph* g : ctx->graphs) {
    g->by_src = SourceRows();
    g->plan_fwd.release();
    g->plan_bwd.release();
    g->ranks = DegreeRanks();
  }
  ctx->list_owner = nullptr;
  ht_kept_release(ctx);
  ++ctx->scratch_gen;      // (captured epochs hold pointers into the lists as well)
  return true;
}

int ht_host_scratch(ht_ctx* ctx, int slot, size_t bytes, void** out) {
  if (ctx->hscratch_bytes[slot] < bytes) {
    if (ctx->hscratch[slot]) {
      HT_HIP(ctx, hipDeviceSynchronize());
      (void)hipHostFree(ctx->hscratch[slot]);
      ctx->hscratch[slot] = nullptr;
      ctx->hscratch_bytes[slot] = 0;
    }
    size_t want = bytes + bytes / 8 + 256;
    hipError_t e = hipHostMalloc(&ctx->hscratch[slot], want, hipHostMallocDefault);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      ctx->hscratch[slot] = nullptr;
      return ht_set_err(ctx, HT_ENOMEM, "hipHostMalloc(%zu): %s", want, hipGetErrorString(e));
    }
    ctx->hscratch_bytes[slot] = want;
  }
  *out = ctx->hscratch[slot];
  return HT_OK;
}

hipEvent_t ht_event(ht_ctx* ctx) {
  if (ctx->ev_next == ctx->ev_pool.size()) {
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    ctx->ev_pool.push_back(e);
  }
  return ctx->ev_pool[ctx->ev_next++];
}

int Timer::begin_on(double* acc, hipStream_t s) {
  if (!on) return -1;
  if (only_lo && (acc < only_lo || acc >= only_hi)) return -1;
  hipEvent_t a = ht_event(ctx), b = ht_event(ctx);
  if (!a || !b) {
    on = false;
    return -1;
  }
  (void)hipEventRecord(a, s);
  ev.push_back(Ent{a, b, s, acc});
  return (int)ev.size() - 1;
}

void Timer::end_id(int id) {
  if (!on || id < 0 || id >= (int)ev.size()) return;
  (void)hipEventRecord(ev[id].b, ev[id].s);
}

int Timer::resolve() {
  for (size_t i = 0; i < ev.size(); ++i) {
    float ms = 0.f;
    hipError_t e = hipEventElapsedTime(&ms, ev[i].a, ev[i].b);
    if (e != hipSuccess) return ht_set_err(ctx, HT_EHIP, "hipEventElapsedTime: %s", hipGetErrorString(e));
    *ev[i].dst += (double)ms;
  }
  ev.clear();
  return HT_OK;
}

void ht_epoch_ws_free(ht_ctx* ctx);

extern "C" {

int ht_ctx_create(ht_ctx** out, int device, void* hip_stream) {
  if (!out) return HT_EINVAL;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return HT_EHIP;
  if (hipSetDevice(device) != hipSuccess) return HT_EHIP;
  ht_ctx* c = new (std::nothrow) ht_ctx();
  if (!c) return HT_ENOMEM;
  c->device = device;
  if (static_scratch_address(device, &c->static_base) != HT_OK) {
    delete c;
    return HT_EHIP;
  }
  if (const char* v = getenv("HT_AGG_VARIANT")) c->agg_variant = atoi(v);
  if (const char* v = getenv("HT_LINK_BLOCKS")) c->link_blocks = atoi(v) > 0 ? atoi(v) : c->link_blocks;
  if (const char* v = getenv("HT_GATHER_BLOCKS")) c->gather_blocks = atoi(v) > 0 ? atoi(v) : 128;
  if (const char* v = getenv("HT_XCD_CONTIG")) c->xcd_contig = atoi(v);
  if (const char* v = getenv("HT_LINK_MEMCPY")) c->link_memcpy = atoi(v);
  if (const char* v = getenv("HT_SLABS_FWD")) c->slabs_fwd = atoi(v);
  if (const char* v = getenv("HT_SLABS_BWD")) c->slabs_bwd = atoi(v);
  if (const char* v = getenv("HT_AGG_UNROLL")) c->agg_unroll = atoi(v) == 8 ? 8 : 4;
  if (const char* v = getenv("HT_AGG_UNIFORM")) c->agg_uniform = atoi(v);
  if (const char* v = getenv("HT_SLAB_ALIGN")) c->slab_align = atoi(v);
  if (const char* v = getenv("HT_DENSE")) c->dense = atoi(v);
  if (const char* v = getenv("HT_FINE")) c->fine = atoi(v);
  if (const char* v = getenv("HT_DENSE_WORK")) c->dense_work = std::max<int64_t>(1, atoll(v));
  if (const char* v = getenv("HT_DENSE_WIDE")) c->dense_wide = atoll(v);
  if (const char* v = getenv("HT_FINE_WORK")) {
    c->fine_work = std::max<int64_t>(1, atoll(v));
    c->fine_rows = 0;
  }
  if (const char* v = getenv("HT_FINE_ROWS")) c->fine_rows = atoll(v);
  if (const char* v = getenv("HT_UNIT_SMALL")) c->unit_small = std::min<int64_t>(atoll(v), c->unit_small);
  if (const char* v = getenv("HT_FUSE_UPDATE")) c->fuse_update = atoi(v);
  if (const char* v = getenv("HT_AGG_PHASES")) c->agg_phases = atoi(v) > 1 ? atoi(v) : 1;
  if (const char* v = getenv("HT_REFUSE_ALLOC")) c->refuse_alloc = atoll(v);
  if (const char* v = getenv("HT_DEVICE_BYTES")) c->device_bytes = atoll(v);
  if (const char* v = getenv("HT_LINK_BLOCK_ROWS")) c->link_block_rows = atoll(v) > 0 ? atoll(v) : c->link_block_rows;
  if (hip_stream) {
    c->stream = (hipStream_t)hip_stream;
  } else {
    if (hipStreamCreate(&c->stream) != hipSuccess) {
      delete c;
      return HT_EHIP;
    }
    c->own_stream = true;
  }
  for (int i = 0; i < 3; ++i)
    if (hipStreamCreate(&c->side[i]) != hipSuccess) {
      delete c;
      return HT_EHIP;
    }
  *out = c;
  return HT_OK;
}

int ht_ctx_destroy(ht_ctx* ctx) {
  if (!ctx) return HT_EINVAL;
  (void)hipSetDevice(ctx->device);
  (void)hipStreamSynchronize(ctx->stream);
  for (int i = 0; i < 3; ++i)
    if (ctx->side[i]) {
      (void)hipStreamSynchronize(ctx->side[i]);
      (void)hipStreamDestroy(ctx->side[i]);
    }
  ht_epoch_ws_free(ctx);
  for (ht_graph* g : ctx->graphs) g->ctx = nullptr;
  for (int i = 0; i < HT_N_SCRATCH; ++i)
    if (ctx->scratch[i]) dev_free(ctx, ctx->scratch[i], ctx->scratch_bytes[i], false);
  ht_kept_release(ctx);
  for (int i = 0; i < HT_N_HS; ++i)
    if (ctx->hscratch[i]) (void)hipHostFree(ctx->hscratch[i]);
  for (hipEvent_t e : ctx->ev_pool) (void)hipEventDestroy(e);
  if (ctx->own_stream) (void)hipStreamDestroy(ctx->stream);
  delete ctx;
  return HT_OK;
}

int ht_sync(ht_ctx* ctx) {
  if (!ctx) return HT_EINVAL;
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (int i = 0; i < 3; ++i) HT_HIP(ctx, hipStreamSynchronize(ctx->side[i]));
  return HT_OK;
}

int64_t ht_ctx_graph_launches(const ht_ctx* ctx) { return ctx ? ctx->graph_launches : -1; }

int ht_ctx_set_hbm_budget(ht_ctx* ctx, int64_t bytes) {
  if (!ctx || bytes < 0) return HT_EINVAL;
  (void)hipSetDevice(ctx->device);
  ht_kept_release(ctx);
  ctx->hbm_budget = bytes;
  ctx->tight_room = -1;
  ctx->gat_keep_limit = 0;
  return HT_OK;
}

const char* ht_strerror(int code) {
  switch (code) {
    case HT_OK: return "ok";
    case HT_EINVAL: return "invalid argument";
    case HT_ENOMEM: return "out of memory or over the byte budget";
    case HT_EHIP: return "HIP runtime error";
    case HT_ESHAPE: return "tensor shape, pitch or location does not fit";
    case HT_ESTATE: return "call not valid in this state";
    default: return "unknown error code";
  }
}

const char* ht_last_error(const ht_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

int ht_memory_model(int64_t V, int32_t n_layers, const int32_t* dims, double* vertex_bytes,
                    double* intermediate_bytes) {
  if (V < 0 || n_layers < 1 || !dims) return HT_EINVAL;
  double sum = 0.0;
  for (int l = 0; l <= n_layers; ++l) sum += dims[l];
  if (vertex_bytes) *vertex_bytes = (double)V * sum * 4.0 * 2.0;
  double mid = 0.0;
  for (int l = 1; l < n_layers; ++l) mid += 2.0 * dims[l];
  mid += 3.0 * dims[n_layers];
  if (intermediate_bytes) *intermediate_bytes = (double)V * mid * 4.0;
  return HT_OK;
}

double ht_chunk_rows_model(int64_t V, int32_t n_chunks, double alpha) {
  if (n_chunks <= 0) return 0.0;
  return (1.0 + alpha) * (double)V / (double)n_chunks;
}

double ht_comm_cost_model(int64_t v_ori, int64_t v_p2p, int64_t v_ru, int64_t bytes_per_row, double t_hd, double t_dd,
                          double t_ru) {
  if (v_ru < 0 || v_ru > v_p2p || v_p2p > v_ori || bytes_per_row < 0) return -1.0;
  const double b = (double)bytes_per_row;
  double c = 0.0;
  const int64_t parts[3] = {v_ru, v_ori - v_p2p, v_p2p - v_ru};
  const double thr[3] = {t_hd, t_dd, t_ru};
  for (int k = 0; k < 3; ++k) {
    if (parts[k] == 0) continue;
    if (!(thr[k] > 0.0)) return -1.0;
    c += (double)parts[k] * b / thr[k];
  }
  return c;
}

}  // extern "C"
