// Internal declarations shared by the translation units of libhongtu.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <chrono>
#include <cstdio>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/hongtu.h"

// Edges one forward aggregation work item covers at most (backward items take half).  Rows
// longer than this are cut into several items whose partial sums are added in item order.
// Shorter items read a narrower range of source rows, which is what keeps them in L2.
constexpr int HT_SEG = 256;

// Entries times columns of one pass from which a graph's plan is made and used (ht_dense.hip): entries in dense tiles, all entries.  Layers
// forward and backward, us without | with tiles at millions in them: 3e4 vertices, 3 M edges, 300 columns (360) 491 | 499, 1e4, 4 M, 128
// (170) 195 | 195, 1e5, 10 M, 128 (510) 675 | 696; 3e4, 12 M, 300 (1,200) 1,096 | 824, 1e5, 40 M, 128 (2,200) 1,581 | 1,162.  A plan takes a
// millisecond or two to make, so it is left where a pass would gain less than some 100 us; short items (0.2 ms) where it would gain less than 5.
constexpr int64_t HT_DENSE_WORK = 1000000000, HT_FINE_WORK = 200000000;
// Dense tiles times blocks of 128 columns from which those are taken and not blocks of 64 (both sides: ht_dense_launch).
constexpr int64_t HT_DENSE_WIDE = 32768;
// ... and bytes of rows for short items: fewer stay in the L2s whatever the order (which shapes gain beyond that: short_items_pay).
constexpr int64_t HT_FINE_ROWS = (int64_t)24 << 20;

struct EpochWs;
struct ht_graph;

enum {
  HT_S_PACKW = 0, HT_S_TNPART, HT_S_LOSS, HT_S_ACHUNK, HT_S_OCHUNK, HT_S_ZCHUNK, HT_S_DZCHUNK, HT_S_DACHUNK,
  HT_S_NBUF, HT_S_SPART, HT_S_LEAVE, HT_S_MISC, HT_S_TFULL, HT_S_TFULL2, HT_S_GATV, HT_S_GATE, HT_S_GATWS, HT_S_GATP, HT_S_GATKEEP,
  HT_S_LINK0, HT_S_LINK1, HT_S_LINK2, HT_S_SCAN, HT_S_RSORT, HT_S_TNTAB, HT_S_LIST, HT_S_DENSE, HT_N_SCRATCH
};

constexpr int HT_HS_READBACK = 3, HT_HS_LOSS = 4, HT_N_HS = 5;

// A product A^T B whose slices (n values each) are not added up yet: the end of the epoch does it beside the update (ht_step).
struct PendingTn {
  const float* P;
  int64_t n;
  int slices;
  float* C;                    // [n], or, of width 4, its first two columns apart:
  float* column[2];
};

// Device blocks that a context keeps for its next allocations, and all of a device's contexts together.
constexpr size_t HT_KEPT_BYTES = (size_t)4 << 30, HT_KEPT_BLOCKS = 64, HT_KEPT_ALL = (size_t)12 << 30;

struct ht_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  hipStream_t side[3] = {nullptr, nullptr, nullptr};  // input (gather / H2D), output (D2H), host-function streams
  std::string err;
  int64_t hbm_budget = 0;  // 0 = unlimited
  int64_t hbm_used = 0;
  std::unordered_map<void*, size_t> larger;    // blocks in use that hold more than was asked for
  std::vector<hipEvent_t> ev_pool;
  size_t ev_next = 0;
  EpochWs* ws = nullptr;  // buffers of the last ht_epoch
  // device scratch that calls keep between invocations (grow-only)
  int64_t graph_launches = 0; // epochs that ran as one HIP graph launch
  uint64_t scratch_gen = 0;   // bumped whenever a scratch slot is (re)allocated: captured pointers into scratch are stale then
  void* scratch[HT_N_SCRATCH] = {};
  size_t scratch_bytes[HT_N_SCRATCH] = {};
  // The device's statically allocated scratch array (ht_core.hip), its address taken once at ht_ctx_create.
  // While static_mode is set (inside ht_layer_fwd_static) ht_scratch hands out pieces of it and nothing allocates.
  unsigned char* static_base = nullptr;
  bool static_mode = false;
  size_t static_used = 0;
  size_t static_off[HT_N_SCRATCH] = {};
  size_t static_len[HT_N_SCRATCH] = {};
  // pinned host scratch (slots 0-2: D2H staging of gradient rows; HT_HS_READBACK: small counts read back by ht_partition; HT_HS_LOSS: an
  // epoch's loss, of one size always, so that captured epochs may keep its address)
  void* hscratch[HT_N_HS] = {};
  size_t hscratch_bytes[HT_N_HS] = {};
  int xcd_contig = 0;     // 1: XCDs take contiguous parts of the item list instead of interleaving it
                          // (HT_XCD_CONTIG; measured slower at cfg2: 30.7 vs 26.0 ms per epoch)
  // workgroups of a kernel that moves rows over the host link (HT_LINK_BLOCKS): the link takes no more than a few give it, and the others only
  // stand in the way of the gather and the compute beside it (64, 32, 16, 8: 612 k vertices, 15 M edges, h and grad h on the host 159.6, 154.7,
  // 152.3, 154.4 ms an epoch, with a^l there too 206, 197, 194; GAT 179, 176, 173)
  int link_blocks = 16;
  int gather_blocks = 128; // workgroups of the neighbour-row gather from host memory (HT_GATHER_BLOCKS): beside a D2H
                           // copy the gather's read requests queue behind the write data, and more waves keep more in flight
  int link_memcpy = 0;    // hipMemcpyAsync for contiguous host<->device row ranges: 1 both ways, 2 to the host only, 3 from the host only (HT_LINK_MEMCPY)
  int slabs_fwd = 0, slabs_bwd = 0;  // caps on feature slabs (HT_SLABS_FWD / HT_SLABS_BWD), 0 = by width
  int agg_unroll = 4;     // HT_AGG_UNROLL: row reads in flight per lane (4 or 8)
  int agg_uniform = 1;    // HT_AGG_UNIFORM=0: no wave-uniform fast path for one-edge-per-step shapes
  int slab_align = 1;     // HT_SLAB_ALIGN=0: do not round slabs to whole cache lines
  int agg_phases = 1;     // HT_AGG_PHASES: slabs are spread over this many consecutive launches
  int64_t link_block_rows = (int64_t)1 << 20;   // HT_LINK_BLOCK_ROWS: rows per staged block of a host-resident tensor (GAT path)
  int agg_variant = 0;  // 0: feature slabs per XCD; 1: full-width rows per wave (HT_AGG_VARIANT, for A/B runs)
  const ht_graph* list_owner = nullptr;  // whose by-source list is in HT_S_LIST (null: nobody's)
  std::vector<ht_graph*> graphs;   // the graphs of this context (each may hold a by-source list)
  bool lean = false;           // the call is being made again with as little memory as it can do with (ht_with_room)
  bool no_grow = false;        // inside a stream capture: nothing may be allocated
  int64_t tight_room = -1;     // room that was left after the last such call (-1: none since memory was plentiful)
  size_t gat_keep_limit = 0;   // a GAT epoch that kept this many bytes between its passes ran out of memory (0: none did) ...
  int64_t gat_keep_room = 0;   // ... and had this much room without them
  bool recorded = false;       // the owner of the stream has recorded a pass, which may be replayed for as long as it likes
  int64_t refuse_alloc = 0;    // HT_REFUSE_ALLOC=k: the context's k-th allocation is refused; -k: its k-th hipMalloc fails (tests)
  int64_t device_bytes = 0;    // HT_DEVICE_BYTES: plan as if the device had no more memory than this for the context (0: as it reports)
  bool tn_defer = false;       // inside an epoch: products that allow it leave their slices (slot HT_S_TNPART, from tn_used bytes on) to ht_step
  size_t tn_used = 0;
  std::vector<PendingTn> tn_pending;
  int dense = 1;               // HT_DENSE=0: no products over a graph's dense tiles (ht_dense.hip)
  int fine = 1;                // HT_FINE=0: no shorter work items for training passes
  int64_t dense_work = HT_DENSE_WORK, fine_work = HT_FINE_WORK, fine_rows = HT_FINE_ROWS;   // HT_DENSE_WORK, HT_FINE_WORK, HT_FINE_ROWS
  int64_t dense_wide = HT_DENSE_WIDE;   // HT_DENSE_WIDE
  int64_t unit_small = (int64_t)1 << 30;   // floats of rows below which column units address them in 32 bits (HT_UNIT_SMALL)
  int fuse_update = 0;  // HT_FUSE_UPDATE=1: layers that keep no aggregate run aggregate + transform as one kernel (A/B)
  int n_threads = 0;  // host threads for CPU-side accumulation (0 = chosen on first use)
};

int ht_set_err(ht_ctx* ctx, int code, const char* fmt, ...);

#define HT_HIP(ctx, call)                                                                  \
  do {                                                                                     \
    hipError_t e_ = (call);                                                                \
    if (e_ != hipSuccess)                                                                  \
      return ht_set_err((ctx), e_ == hipErrorOutOfMemory ? HT_ENOMEM : HT_EHIP, "%s: %s",  \
                        #call, hipGetErrorString(e_));                                     \
  } while (0)

#define HT_TRY(expr)            \
  do {                          \
    int rc_ = (expr);           \
    if (rc_ != HT_OK) return rc_; \
  } while (0)

#define HT_LAUNCH_CHECK(ctx) HT_HIP(ctx, hipGetLastError())

// HT_STATIC_SCRATCH_BYTES (hongtu.h): bytes of the statically allocated device scratch array that the
// allocation-free entry point works in.
void ht_static_begin(ht_ctx* ctx);   // ht_scratch serves from the static array until ht_static_end
void ht_static_end(ht_ctx* ctx);

// Device allocation with budget accounting.
int ht_dev_alloc(ht_ctx* ctx, void** out, size_t bytes);
void ht_dev_free(ht_ctx* ctx, void* p, size_t bytes);
void ht_kept_release(ht_ctx* ctx);  // gives back the blocks that the context keeps ...
void ht_kept_trim(ht_ctx* ctx);     // ... where the device is nearly full
void ht_free_orphan(ht_graph* g);   // a graph whose context is gone
// Grow-only scratch slot (kept on the context).
int ht_scratch(ht_ctx* ctx, int slot, size_t bytes, void** out);
// Gives a slot's memory back (after the work in flight).
int ht_scratch_release(ht_ctx* ctx, int slot);
// What the device reports free.
int64_t ht_device_free(ht_ctx* ctx);
// Bytes that can still be allocated: by the byte budget and by the device's free memory.
int64_t ht_room(ht_ctx* ctx);

// Several slots that a pass takes together.
struct ScratchWant { int slot; size_t bytes; };
// All of them at these sizes, or HT_ENOMEM and none of them larger than before.  What has to grow is looked up in ht_room first (with
// `beside` further bytes that the caller is about to take), so that a pass that does not fit frees and allocates nothing, call after call.
// Where the device refuses memory that the figures promised, a slot may be left smaller than before, or empty: whoever goes on after
// HT_ENOMEM asks for every slot again before using it.
int ht_scratch_all(ht_ctx* ctx, const std::vector<ScratchWant>& want, int64_t beside = 0);
// The slots one after the other, whatever it takes (HT_ENOMEM: some of them).
int ht_scratch_each(ht_ctx* ctx, const std::vector<ScratchWant>& want);
// Releases the slots that have grown since it was made (a by-source list that was made meanwhile stays).
struct ScratchMark {
  ht_ctx* ctx;
  size_t was[HT_N_SCRATCH];
  explicit ScratchMark(ht_ctx* c);
  void undo();
};

// Memory that only makes calls faster (all chunks at once, by-source lists, rows kept between passes) must not be what a call is
// refused for.  Passes that can do with less ask ht_may_spend first, and fall back when they are refused memory; a call that is refused
// all the same is made again once everything the context can do without was given back (scratch slots, by-source lists), with `lean`
// set.  From then on nothing is spent until there is more room than was left by that call.
bool ht_may_spend(ht_ctx* ctx);
bool ht_caller_captures(ht_ctx* ctx);   // the owner of the context's stream records what is launched there: nothing may be allocated
bool ht_give_back(ht_ctx* ctx);   // false: there was nothing to give back
int64_t ht_held(const ht_ctx* ctx);   // bytes that ht_give_back would free
// `changed`: the call has begun to change what the caller handed in, and cannot be made again.
template <class F>
int ht_with_room(ht_ctx* ctx, F&& call, const bool* changed = nullptr) {
  if (!ctx->recorded) ctx->recorded = ht_caller_captures(ctx);
  int rc = call();
  if (rc != HT_ENOMEM || (changed && *changed) || !ht_give_back(ctx)) return rc;
  ctx->lean = true;
  rc = call();
  ctx->lean = false;
  if (rc == HT_OK) ctx->tight_room = ht_room(ctx);
  return rc;
}
// Grow-only pinned host scratch.
int ht_host_scratch(ht_ctx* ctx, int slot, size_t bytes, void** out);

template <typename T>
struct DevArr {
  T* p = nullptr;
  size_t n = 0;
  ht_ctx* ctx = nullptr;
  bool owned = true;   // false: a view into a block that another DevArr owns
  DevArr() = default;
  DevArr(const DevArr&) = delete;
  DevArr& operator=(const DevArr&) = delete;
  DevArr(DevArr&& o) noexcept : p(o.p), n(o.n), ctx(o.ctx), owned(o.owned) { o.p = nullptr; o.n = 0; }
  DevArr& operator=(DevArr&& o) noexcept {
    if (this != &o) {
      release();
      p = o.p; n = o.n; ctx = o.ctx; owned = o.owned;
      o.p = nullptr; o.n = 0;
    }
    return *this;
  }
  ~DevArr() { release(); }
  int alloc(ht_ctx* c, size_t count) {
    release();
    ctx = c;
    n = count;
    owned = true;
    if (count == 0) return HT_OK;
    return ht_dev_alloc(c, (void**)&p, count * sizeof(T));
  }
  void release() {
    if (p && owned) ht_dev_free(ctx, p, n * sizeof(T));
    p = nullptr;
    n = 0;
  }
  size_t bytes() const { return n * sizeof(T); }
};

// Arrays of one lifetime carved out of one device allocation: an allocation and its release cost tens of
// microseconds each whatever their size, and ht_partition makes dozens.  add() every array first, then
// alloc(), then take() them in the same order; every array starts on a 256-byte boundary.
struct DevBlock {
  DevArr<char> mem;
  size_t planned = 0, taken = 0;
  static size_t pad(size_t b) { return (b + 255) & ~(size_t)255; }
  template <typename T>
  void add(size_t count) { planned += pad(count * sizeof(T)); }
  int alloc(ht_ctx* c) { taken = 0; return mem.alloc(c, planned > 0 ? planned : 1); }
  // the same in a scratch slot of the context, which stays its owner
  int alloc_in(ht_ctx* c, int slot) {
    void* p = nullptr;
    const int rc = ht_scratch(c, slot, planned > 0 ? planned : 1, &p);
    if (rc != HT_OK) return rc;
    mem.release();
    mem.p = (char*)p;
    mem.n = planned;
    mem.ctx = c;
    mem.owned = false;
    taken = 0;
    return HT_OK;
  }
  template <typename T>
  void take(DevArr<T>& a, size_t count) {
    a.release();
    a.ctx = mem.ctx;
    a.owned = false;
    a.n = count;
    a.p = (T*)(mem.p + taken);
    taken += pad(count * sizeof(T));
  }
  void release() { mem.release(); planned = taken = 0; }
};

static inline int64_t ceil_div64(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- primitives (ht_prims.hip) -------------------------------------------------------
// Exclusive prefix sum of n values into out[0..n); out[n] = total when want_total.
// Rates the epoch planner prices its choices with (measured on MI355X: host link beside compute,
// rows gathered per second by the aggregation kernel, in bytes).
constexpr double HT_LINK_BYTES_PER_S = 45e9;
constexpr double HT_GATHER_BYTES_PER_S = 15e12;

// Destination rows from which the dense work of neighbouring chunks is no longer merged.
constexpr int64_t HT_DENSE_MERGE_ROWS = 32768;

// Row pitch (in floats) of a library-allocated [rows x d] matrix: a multiple of 4 (16-byte
// vectors); in HBM, rows start on 128-byte cache lines when that costs at most 3 % more memory,
// so a feature slab never shares a line with the slab of another XCD; in pinned host memory rows
// start on 64-byte boundaries: a row read over the link then splits into whole 64-byte requests
// (rows at a 400-byte pitch were gathered at 22 GB/s beside a D2H copy that fell to 29 GB/s; at a
// 448-byte pitch 26-34 GB/s beside 46-50 GB/s).
inline int64_t ht_row_pitch(int32_t d, bool device) {
  const int64_t p4 = ((int64_t)d + 3) & ~(int64_t)3, p16 = ((int64_t)d + 15) & ~(int64_t)15, p32 = ((int64_t)d + 31) & ~(int64_t)31;
  if (!device) return p16;
  return p32 * 100 <= p4 * 103 ? p32 : p4;
}

int ht_scan_i32(ht_ctx* ctx, const int32_t* in, int64_t* out, int64_t n, bool want_total);
int ht_scan_i64(ht_ctx* ctx, const int64_t* in, int64_t* out, int64_t n, bool want_total);
// Stable LSD radix sort of 64-bit keys on bits [bit_lo, bit_hi).  keys and tmp
// have n entries; returns in *sorted which of the two holds the result.
int ht_radix_sort_u64(ht_ctx* ctx, uint64_t* keys, uint64_t* tmp, int64_t n, int bit_lo, int bit_hi,
                      uint64_t** sorted);
// Edges as keys (destination << bits) | source, a self-loop per vertex behind them where n > E; an id outside [0, V) raises the flag and becomes 0, so that
// nothing later leaves its array.
struct EdgeKeys {
  const int32_t *src, *dst;
  int64_t E, V;
  int bits;
  int64_t* flag;
  __device__ __forceinline__ void load(int64_t i, uint32_t* u, uint32_t* v) const { *u = *v = (uint32_t)(i - E); if (i < E) *u = (uint32_t)src[i], *v = (uint32_t)dst[i]; }
  __device__ __forceinline__ bool valid(uint32_t u, uint32_t v) const { return u < (uint64_t)V && v < (uint64_t)V; }
  __device__ __forceinline__ uint64_t key(uint32_t u, uint32_t v) const { return valid(u, v) ? (uint64_t)v << bits | u : 0ull; }
};
// The n keys of these edges in ascending order, in keys or tmp; the first pass makes them on the way (64 M edges: 250 us less than making them first).
int ht_radix_sort_edges(ht_ctx* ctx, const EdgeKeys& edges, uint64_t* keys, uint64_t* tmp, int64_t n, uint64_t** sorted);
// Bitmap helpers: words are uint64, bit b of word w is element 64*w + b.
// pref[w] = number of set bits before word w; pref[nw] = total.
int ht_bitmap_prefix(ht_ctx* ctx, const uint64_t* bm, int64_t nw, int32_t* cnt_tmp, int64_t* pref);

// ---- graph -------------------------------------------------------------------------------
// Work items of one aggregation direction: a row with at most HT_SEG entries is one item; a longer row is cut into items
// of HT_SEG entries whose partial sums are added in item order by a second kernel.  Rows are destinations (forward) or
// positions of the N arena (backward); rows, entries and partial sums are numbered over the whole graph, and a chunk's
// items are a contiguous range of the list, so a launch can take one chunk or all of them.
struct __attribute__((aligned(16))) WorkItem {
  uint32_t row;    // (positions of the N arena: up to 2^32 of them)
  uint32_t e0;     // first entry (stored edges, or distinct pairs when duplicates are merged)
  int32_t len;     // entries (<= HT_SEG)
  int32_t part;    // -1: the row's only item; else index of its partial sum
};
struct __attribute__((aligned(16))) CutRow {   // a row with several items
  uint32_t row;
  int32_t part0, nseg;
  uint32_t item0;              // its first item, in row order
};
struct GraphItems {
  DevArr<WorkItem> items;
  DevArr<CutRow> cuts;
  int64_t n_items = 0, n_part = 0, n_cut = 0;
};
struct ItemRange {             // a chunk's share
  int64_t it0 = 0, n_items = 0, part0 = 0, n_part = 0, cut0 = 0, n_cut = 0;
};

struct ChunkMeta {
  int32_t id = 0;              // position in vertex order
  int64_t dst0 = 0, dst1 = 0;  // destination range
  int64_t e0 = 0, nnz = 0;     // edge range in the global CSC arrays
  int64_t ue0 = 0, nu = 0;     // range of distinct (destination, source) pairs in the merged arrays (= e0, nnz when not merged)
  int64_t nsrc = 0;            // |N_j|
  int64_t nbr_off = 0;         // offset of N_j in the nbr / slot arenas (chunks in vertex order)
  int64_t sptr_off = 0;        // offset of sptr_j in the sptr arena (nbr_off + id)
  int64_t n_reuse = 0, n_load = 0, n_leave = 0;
  int64_t reuse_off = 0, load_off = 0, leave_off = 0;
  ItemRange fwd, bwd;
};

// The whole graph's entries grouped by source (destinations ascending), for backward passes that read grad a of all
// destinations at once.  Built at the first such pass that has memory for it; the others go chunk by chunk.
struct SourceRows {
  bool ok = false;
  DevBlock blk;
  DevArr<int32_t> idx;         // destination of each entry
  DevArr<float> w;             // multiplicity * s[destination] (merged graphs; others look s up)
  DevArr<float> mult;          // multiplicity (merged graphs, made for the first GAT backward pass)
  DevArr<int64_t> ptr;         // [V + 1] first entry of every source
  GraphItems items;            // rows = vertices
};

// How passes that are made over a graph again and again (training passes with everything in HBM) take one direction's entries: made at
// the first such pass that has memory for it, kept with the graph, given back with the by-source list (ht_dense.hip).
//
// Shorter work items over the same entries: the items in flight at one time read a narrower range of rows, more of which L2 keeps.
struct ShortItems {
  bool ok = false;
  int64_t refused = -1;          // there was no memory for it with this much room
  DevBlock mem;
  GraphItems items;              // rows = destinations, or sources
};
// Tiles of DENSE_ROWS x DENSE_COLS multiplicities, rows and columns in order of their number of entries, and work items over the entries in
// no tile.
constexpr int DENSE_ROWS = 256, DENSE_COLS = 64;
constexpr int DENSE_SEG = 64;    // tiles that one block multiplies at most
struct DenseSeg {
  int32_t tile0, n;              // consecutive tiles of one row block
};
struct DenseSide {
  bool ok = false;
  int64_t taken = -1;            // entries that the graph's dense tiles hold (-1: not counted yet)
  int64_t refused = -1;
  DevBlock tiles, rest;
  DevArr<uint8_t> cells;         // the tiles' multiplicities
  DevArr<int32_t> tile_cg;       // column group of each tile
  DevArr<DenseSeg> segs;
  DevArr<int32_t> seg0;          // first segment of each row block, then their number
  DevArr<int32_t> pos;           // [V] row block * DENSE_ROWS + row in it (-1: the row is in none)
  DevArr<int32_t> cols;          // [n_cols] vertex of each column (-1: none)
  DevArr<int32_t> idx;           // entries in no tile ...
  DevArr<float> w;               // ... and their weights
  GraphItems items;              // rows in row blocks are all cut rows (in `rest`)
  int64_t n_tiles = 0, n_segs = 0, n_cols = 0, n_rest = 0;
};
struct GraphPlan {
  ShortItems fine;
  DenseSide dense;
  int64_t bytes() const {
    return (int64_t)(fine.mem.mem.bytes() + dense.tiles.mem.bytes() + dense.rest.mem.bytes());
  }
  void release() {               // what was counted stays known
    const int64_t taken = dense.taken;
    *this = GraphPlan();
    dense.taken = taken;
  }
};
// Vertices in order of their number of entries, as destinations [0] and as sources [1]: both directions' tiles are made of the two.  Made with
// the first direction's, given back with the second's.
struct DegreeRanks {
  bool ok = false;
  DevBlock mem;
  DevArr<int32_t> order[2];      // the first vertices, in row blocks of DENSE_ROWS (-1 behind the last)
  DevArr<int32_t> rank[2];       // [V]
};
// What a pass takes of it.
struct PassPlan {
  const GraphItems* items = nullptr;   // null: the graph's own items
  const DenseSide* dense = nullptr;    // null: all entries by these items
  int64_t parts() const { return items ? items->n_part + (dense ? dense->n_segs * DENSE_ROWS : 0) : 0; }   // of the items, then of the segments
};

struct ht_graph {
  ht_ctx* ctx = nullptr;
  uint64_t serial = 0;         // unique per ht_partition call in this process: tells graphs at one address apart
  int64_t V = 0, Ep = 0;
  int32_t n = 0;
  int32_t add_self_loops = 1;
  bool single_leave = false;   // schedule-aware buffer that loads (and so releases) every row once per pass
  DevArr<int64_t> indptr;      // [V+1]
  DevArr<int32_t> col;         // [E'] global source ids
  DevArr<float> s;             // [V] D^-1/2
  std::vector<int64_t> bounds; // [n+1] host, in vertex-id order
  std::vector<int32_t> order;  // [n] schedule position -> chunk id (identity unless chunks were reorganised)
  std::vector<ChunkMeta> chunks;
  DevArr<int32_t> nbr;         // [v_ori] N_j lists
  DevArr<int32_t> col_local;   // [E']
  DevArr<int32_t> col_slot;    // [E'] buffer position of each edge's source
  DevArr<int64_t> sptr;        // [v_ori + n] per-chunk offsets, rebased to 0
  DevArr<int32_t> sdst;        // [E'] local destinations grouped by local source
  DevArr<int32_t> slot;        // [v_ori] buffer position of N_j[i]
  DevArr<int32_t> gslot;       // [v_ori] slot | (1<<31 when N_j[i] is newly loaded)
  DevArr<int32_t> reuse;       // [v_ori - v_load]
  DevArr<int32_t> load;        // [v_load]
  DevArr<int32_t> load_slot;   // [v_load]
  DevArr<int32_t> leave;       // [v_load] rows leaving after each chunk (everything still buffered after the last)
  DevArr<int32_t> leave_slot;  // [v_load]
  // Duplicate edges merged for the aggregation kernels (built when at least 5 % of the edges repeat
  // a pair): one entry per distinct pair, its multiplicity folded into the weight.  The arrays above
  // stay the canonical ones (export, parity).
  bool merged = false;
  int64_t n_unique = 0;
  DevArr<int64_t> uindptr;     // [V+1] row offsets in distinct-pair space
  DevArr<int32_t> ucol;        // [n_unique] source of each distinct pair, CSC order
  DevArr<int32_t> ucol_slot;   // [n_unique] its buffer position
  DevArr<float> uw_fwd;        // [n_unique] multiplicity * s[source]
  DevArr<float> umult;         // [n_unique] multiplicity (for rows already scaled in the buffer)
  DevArr<int64_t> usptr;       // [v_ori + n] per-chunk by-source offsets in distinct-pair space
  DevArr<int32_t> usdst;       // [n_unique] local destination of each distinct pair, by-source order
  DevArr<float> uw_bwd;        // [n_unique] multiplicity * s[destination]
  DevArr<float> umult_bwd;     // [n_unique] multiplicity, by-source order
  GraphItems fwd_items, bwd_items;
  std::vector<int32_t> pos;    // [n] chunk id -> schedule position (inverse of order)
  // Destination rows whose part of grad W is summed together: runs of chunks adjacent in schedule and in vertex order, closed
  // at HT_DENSE_MERGE_ROWS rows; {first row, last row + 1} each, in schedule order.
  std::vector<int64_t> dense_groups;
  DevArr<int64_t> d_dense_groups;
  mutable SourceRows by_src;
  mutable GraphPlan plan_fwd, plan_bwd;
  mutable DegreeRanks ranks;
  mutable int64_t tile_estimate = -1;   // entries that dense tiles should hold, by the vertices' numbers of entries alone (-1: not looked at)
  DevBlock blk_csc, blk_pairs, blk_chunks;   // the allocations behind the CSC, the distinct-pair arrays, and the per-chunk arenas with the work items
  int64_t v_ori = 0, v_ru = 0, v_load = 0;  // v_load: rows actually loaded per pass with this buffer
  int64_t max_nsrc = 0, max_ndst = 0, max_nnz = 0, max_fpart = 0, max_bpart = 0;
  int64_t cache_rows = 0;
  int32_t cache_policy = 0;    // HT_CACHE_*
  double partition_ms = 0.0;
  mutable std::vector<int32_t> leave_host;  // host copy of `leave`, made on first use by the CPU-side adds
  int64_t hbm_bytes() const;
};

// Makes g->by_src if it is not there (HT_ENOMEM: it may not have, or there is no memory for it).  The slot is overwritten on the way.
int ht_graph_by_source(ht_ctx* ctx, const ht_graph* g, int slot);
// Bytes that it takes, and that making it takes of the slot (0: it is there).
void ht_graph_by_source_bytes(const ht_graph* g, int64_t* list, size_t* slot);
// Partial sums of a by-source list over so many entries, at most.
int64_t ht_by_source_parts_bound(int64_t entries);
// Makes g->by_src.mult of a merged graph whose by_src is there (HT_ENOMEM: no memory for it).
int ht_graph_by_source_mult(ht_ctx* ctx, const ht_graph* g);

// Distinct entries (entries, where duplicates are not merged) of every source, into cnt[V].  lists: scratch memory of 2 (g->n + 1) words.
int ht_graph_source_counts(ht_ctx* ctx, const ht_graph* g, int64_t* lists, int32_t* cnt);
// Work items over rows 0 .. V - 1 with entries ptr[r] .. ptr[r + 1] of idx (values below V); rows with pos[r] >= 0 (pos may be null) become cut
// rows whatever their length.  The slot is overwritten on the way.  out's arrays are taken out of `mem`, or are there already, of the sizes that
// ht_row_items_bound and ht_row_cuts_bound say (null).
int ht_graph_row_items(ht_ctx* ctx, int64_t V, const int64_t* ptr, int64_t n_ent, const int32_t* idx, const int32_t* pos, int seg, int slot,
                       DevBlock* mem, GraphItems* out);
inline int64_t ht_row_items_bound(int64_t rows, int64_t entries, int seg) { return rows + entries / seg + 1; }
// (rows that are cut because they are longer than an item, and `forced` ones)
inline int64_t ht_row_cuts_bound(int64_t entries, int seg, int64_t forced) { return entries / seg + 1 + forced; }
// Rows of a direction's list: first entries of its rows.
inline const int64_t* ht_row_ptr(const ht_graph* g, bool fwd) { return !fwd ? g->by_src.ptr.p : g->merged ? g->uindptr.p : g->indptr.p; }
inline int64_t ht_entries(const ht_graph* g) { return g->merged ? g->n_unique : g->Ep; }
// What a pass over rows of d columns, src_ld floats apart, should take, made if it is not there and may be.  (Backward: by_src is there.)
int ht_pass_plan(ht_ctx* ctx, const ht_graph* g, bool fwd, int32_t d, int64_t src_ld, PassPlan* out);
// The segments' sums of s_u src[u] into partial: DENSE_ROWS rows of pitch out_ld each.
int ht_dense_launch(ht_ctx* ctx, hipStream_t st, const DenseSide& D, const float* src, int64_t ld, const float* s, int32_t d, float* partial,
                    int64_t out_ld);

// Column units (k_spmm_unit): lanes, each with a float4, that own one item's part of a row.
constexpr int UNIT_LANES = 16;
// Rows go in column units where those are whole cache lines (a line that two units share is fetched twice: 2 M vertices, 30 M edges, 200
// columns in rows of 800 bytes 13.5 -> 15.9 ms a layer) or there is one unit, and where the rows that are read are more than the caches
// hold (116 k rows of 132: no difference; 60 k of 132: 86 us a pass, 70 expected of the slab kernel; 1 M of 64: 950 -> 870).
inline bool ht_unit_shape(int64_t src_rows, int64_t src_ld, int nvec, bool aligned) {
  return (((src_ld & 31) == 0 && aligned) || nvec <= UNIT_LANES) && src_rows * src_ld * 4 >= ((int64_t)64 << 20);
}

// ---- compute kernels' host launchers -----------------------------------------------------
// Aggregation over work items (ht_spmm.hip).  One wave (or a lane group of it)
// owns an item; sums are taken in edge order, partial sums in item order.
struct SpmmArgs {
  // items
  const WorkItem* items;
  int64_t n_items;
  int64_t n_edges;        // entries covered by the items (for launch heuristics)
  const CutRow* cuts;
  int64_t n_fix;
  int64_t part0 = 0;      // number of the first partial sum (row 0 of `partial`)
  int64_t row0 = 0;       // row that is row 0 of `out` (when out_idx is null)
  // edges
  const int32_t* idx;     // per entry: row of `src` to read
  const float* ew;        // per-edge weight table indexed by idx (nullable: weight 1)
  const float* w_edge = nullptr;  // per-entry weights in entry order, the first one for entry w0 (takes precedence over ew)
  int64_t w0 = 0;
  const float* src;       // source matrix
  int64_t src_ld;
  int32_t d;              // valid columns
  // output
  float* out;             // output matrix
  int64_t out_ld;
  const int32_t* out_idx; // row r -> output row (nullable: r - row0); bit 31 set => overwrite even when accumulating
  const float* post;      // per-row factor
  const int32_t* post_idx;// row r -> index into post (nullable: r)
  int32_t accumulate;     // 1: out += value
  float* partial;         // [n_part x out_ld] workspace
  int relu = 0;           // clamp the finished row at 0 (only without accumulate)
  int max_slabs = 0;      // cap on the number of feature slabs (0 = by width)
  bool units = false;     // items are short and in order of length: column units may be used
  int64_t src_rows = 0;   // rows of src (for that choice)
  // the dense part's sums, from partial sum dense_part on (null: there is none)
  const int32_t* dense_pos = nullptr;
  const int32_t* dense_seg0 = nullptr;
  int64_t dense_part = 0;
  // optional timing of the two kernels (null: not timed)
  struct Timer* tm = nullptr;
  double* t_items = nullptr;
  double* t_fix = nullptr;
};
int ht_spmm_launch(ht_ctx* ctx, hipStream_t st, const SpmmArgs& a);
// A launch of 2^32 threads or more is not rejected, its excess is silently dropped.  Kernels that take a wave per work item, or
// a block of 4 waves per cut row, therefore go in launches of at most this many waves (2^31 threads; a graph of 70 M vertices
// has more items than one launch can hold).
constexpr int64_t HT_LAUNCH_WAVES = (int64_t)1 << 25;
template <class F>
int ht_in_launches(int64_t n, int64_t most, F&& launch) {   // launch(first, count)
  for (int64_t i = 0; i < n; i += most) {
    const int rc = launch(i, (n - i) < most ? (n - i) : most);
    if (rc != HT_OK) return rc;
  }
  return HT_OK;
}
// How an aggregation is spread over the XCDs (d, n_items, n_edges, src, src_ld and max_slabs of `a` are read): P launches of
// S slabs of nvs float4 columns, eps entries per step of a wave.
struct SlabShape {
  int S, P, nvs, eps;
  bool contig;               // each XCD of a slab takes a contiguous part of the items (else they are interleaved)
  int64_t launch_items() const { return HT_LAUNCH_WAVES / S; }
  // blocks of 4 waves for one launch over n items; grp_per_part: groups of 4 items per part, 0 where they are interleaved
  unsigned grid(int64_t n, int64_t* grp_per_part) const {
    const int64_t parts = 8 / S, gpp = ((n + 3) / 4 + parts - 1) / parts;
    *grp_per_part = contig ? gpp : 0;
    return (unsigned)(gpp * 8);
  }
};
int ht_slab_shape(ht_ctx* ctx, const SpmmArgs& a, SlabShape* out);
// Only the second kernel: the cut rows = their partial rows added in item order (d, out*, partial, cuts, part0 are read).
int ht_spmm_fix_launch(ht_ctx* ctx, hipStream_t st, const SpmmArgs& a);

// Row gather / scatter (ht_spmm.hip)
// dst[dst_idx[k]] = scale[src_idx[k]] * src[src_idx[k]]   (scale nullable)
int ht_gather_rows(ht_ctx* ctx, hipStream_t st, const float* src, int64_t src_ld, const int32_t* src_idx,
                   float* dst, int64_t dst_ld, const int32_t* dst_idx, int64_t n_rows, int32_t d,
                   const float* scale, int max_blocks = 0);
// Contiguous copy by a kernel with a small grid; src/dst may be device or GPU-addressable host memory.
int ht_copy_link(ht_ctx* ctx, hipStream_t st, void* dst, const void* src, size_t bytes, int blocks);
// dst[dst_idx[k]] += src[src_idx[k]]  (dst_idx unique inside one call)
int ht_add_rows(ht_ctx* ctx, hipStream_t st, const float* src, int64_t src_ld, const int32_t* src_idx,
                float* dst, int64_t dst_ld, const int32_t* dst_idx, int64_t n_rows, int32_t d);

// Dense transform (ht_gemm.hip)
// Bytes of the packed copy of a [K x N] W that the NN kernels read (in the context's scratch).
inline int64_t ht_packed_w_bytes(int64_t K, int64_t N) { return ((K + 15) & ~(int64_t)15) * ((N + 127) & ~(int64_t)127) * 4; }
// C[M x N] = A[M x K] B[K x N], optional ReLU, C rows pitch ldc.  B is row-major dense [K x N].
int ht_gemm_nn(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, float* C, int64_t ldc,
               int64_t M, int32_t K, int32_t N, int relu);
// C[M x K] = A[M x N] B[K x N]^T
int ht_gemm_nt(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, float* C, int64_t ldc,
               int64_t M, int32_t N, int32_t K, int accumulate);
// C[K x N] (+)= A[M x K]^T B[M x N]; fixed-order reduction over M slices.
// `later` (C of width 4: with its columns, which are written instead of C): the sum may be left to ht_step; *left = it was.
struct TnLater {
  float* column[2] = {nullptr, nullptr};
  bool left = false;
};
// `mask`: B's values count where mask.ref (as many rows and columns) is positive, and are 0 elsewhere; with mask.to (which may be mask.ref) what counts
// is also written there, rows up to their next multiple of 4.  Only products for which ht_gemm_tn_writes holds take a mask.to.
struct ReluMask {
  const float* ref = nullptr;
  int64_t ld = 0;
  float* to = nullptr;
  int64_t to_ld = 0;
};
bool ht_gemm_tn_writes(int64_t rows, int32_t K, int32_t N);
int ht_gemm_tn(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, int64_t ldb, float* C,
               int64_t M, int32_t K, int32_t N, int accumulate, TnLater* later = nullptr, ReluMask mask = ReluMask());
// Products may leave their sums to ht_step from here on, where all of them together take little memory; `bytes`: their partial tiles.
int ht_defer_products(ht_ctx* ctx, const std::vector<size_t>& bytes);
// Adds up what was left (before something else needs it, or after an error: `drop`).
int ht_flush_products(ht_ctx* ctx, hipStream_t st, bool drop = false);

// Bytes of the partial tiles (slot HT_S_TNPART) of an ht_gemm_tn call over M rows.
size_t ht_gemm_tn_bytes(int64_t M, int32_t K, int32_t N);
// The scratch memory of an ht_gemm_tn_groups call.
void ht_gemm_groups_wants(int32_t K, int32_t N, const std::vector<int64_t>& groups, std::vector<ScratchWant>* want);
// C[K x N] = sum over the row groups [groups[2g], groups[2g+1]) of A^T B, added group by group (d_groups: the same on the device).
int ht_gemm_tn_groups(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int32_t K,
                      int32_t N, const std::vector<int64_t>& groups, const int64_t* d_groups, TnLater* later = nullptr, ReluMask mask = ReluMask());
// Partial tiles of such a call, all groups together.
size_t ht_gemm_groups_bytes(int32_t K, int32_t N, const std::vector<int64_t>& groups);

// Aggregate + transform of one chunk in one kernel, the aggregate kept in LDS (ht_fused.hip)
int ht_agg_update_fused(ht_ctx* ctx, hipStream_t st, const ht_graph* g, const ChunkMeta& c, const float* H_in, int64_t in_ld,
                        int32_t d_in, const float* W, int32_t d_out, int relu, float* H_out, int64_t out_ld);

// Elementwise / loss (ht_elem.hip)
// dz = dh * [ref > 0]
int ht_relu_mask(ht_ctx* ctx, hipStream_t st, const float* dh, int64_t ld_dh, const float* ref, int64_t ld_ref,
                 float* dz, int64_t ld_dz, int64_t rows, int32_t cols);
// The loss as the sums of its blocks; ht_step adds them up.
struct LossParts {
  const double* part;
  int n_part;
  const unsigned long long* count;   // labelled vertices per block
  int n_count;
};
int ht_softmax_ce(ht_ctx* ctx, hipStream_t st, const float* logits, int64_t ld, const int32_t* labels, int64_t V,
                  int32_t C, float* grad, int64_t ld_g, LossParts* loss);
// W -= lr dW for every item
struct ht_sgd_item {
  float* W;
  const float* dW;
  int64_t n;
};
constexpr int HT_SGD_MAX = 3 * HT_MAX_LAYERS;   // items per launch
// The end of an epoch: what products have left is added up, W -= lr dW, and the loss goes to *loss (memory of the host that the GPU can
// write, as it sees it).
int ht_step(ht_ctx* ctx, hipStream_t st, const std::vector<ht_sgd_item>& items, float lr, const LossParts& parts, float* loss);
int ht_fill_words(ht_ctx* ctx, hipStream_t st, void* p, size_t bytes, uint32_t value);
inline int ht_fill_zero(ht_ctx* ctx, hipStream_t st, void* p, size_t bytes) { return ht_fill_words(ctx, st, p, bytes, 0u); }

// stats helpers: HIP-event pairs around phases, each on the stream that runs the phase
struct Timer {
  ht_ctx* ctx;
  hipStream_t st;  // default stream for begin()/end()
  bool on;
  struct Ent {
    hipEvent_t a, b;
    hipStream_t s;
    double* dst;
  };
  std::vector<Ent> ev;
  const double *only_lo = nullptr, *only_hi = nullptr;   // when set: time only accumulators inside [only_lo, only_hi)
  Timer(ht_ctx* c, hipStream_t s, bool enabled) : ctx(c), st(s), on(enabled) {}
  int last = -1;   // id of the pair opened by the last begin() (-1: that phase is not timed)
  void begin(double* acc) { last = begin_on(acc, st); }
  void end() { end_id(last); last = -1; }
  int begin_on(double* acc, hipStream_t s);  // returns an id for end_id (-1 when timing is off)
  void end_id(int id);
  int resolve();  // after the streams are synchronised
};
hipEvent_t ht_event(ht_ctx* ctx);
