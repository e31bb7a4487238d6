// ht_partition: edge list -> CSC by destination -> contiguous chunks -> per
// chunk dedup remap (unique sorted sources, local indices), by-source grouping
// for the backward pass, reuse / load split between adjacent chunks, in-place
// buffer positions, aggregation work items.  All on the GPU.
//
// Sec. 4.1 (chunks = destination ranges with all in-edges), Sec. 5.1 step 2
// (N_j ^ N_{j-1} reused, N_j \ N_{j-1} loaded), Sec. 5.3 (V_ori, V_+ru),
// Sec. 6 (same buffer position for duplicated vertices of adjacent chunks;
// loaded rows take freed positions; topology rewritten to buffer positions).
//
// Every step runs over all chunks in one launch: the chunks' arrays lie behind
// each other in vertex order, so an edge, a word of a neighbour bitmap or a
// local source finds its chunk by a search in the n + 1 offsets (once per block,
// then forward).  Only the buffer positions are made chunk by chunk, because
// the positions a chunk's loads take are those the chunks before it left free.
// With one set of launches per chunk a 10,000-vertex graph of 4 chunks took 380
// launches and 2.2 ms with a first layer, now 0.85 ms; a graph of 2.45 M vertices,
// 62 M edges and 16 chunks 1,606 launches and 27.1 ms, now 16.2 ms (MI355X).
#include <algorithm>
#include <atomic>
#include <cstdlib>

#include "ht_internal.h"

namespace {

constexpr int TB = 256;
constexpr int ETILE = 2048;      // entries of a sorted list one block handles
constexpr int RTILE = 1024;      // rows one block cuts into work items
inline unsigned nblk(int64_t n, int tb = TB) { return (unsigned)((n + tb - 1) / tb); }
// Blocks per launch of the kernels that take a block per tile of every chunk's bitmap: n V / 64 threads in all, and a launch of
// 2^32 threads or more silently drops its excess (from n V = 2^38 on: 268 M vertices in 1,024 chunks).
constexpr int64_t TILE_LAUNCH = HT_LAUNCH_WAVES * 64 / TB;

// ---- block-level helpers

// last k in [0, n) with off[k] <= x (off ascending, off[0] <= x): the range that x lies in, empty ranges skipped
__device__ __forceinline__ int find_range(const int64_t* __restrict__ off, int n, int64_t x) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint64_t lanes_below(int lane) { return lane == 0 ? 0ull : (~0ull >> (64 - lane)); }

// Exclusive sum over the 256 threads of a block, *total = sum of all.
__device__ __forceinline__ uint64_t block_excl(uint64_t x, uint64_t* total) {
  __shared__ uint64_t part[TB / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  __syncthreads();   // a previous use of part
  if (lane == 63) part[wave] = inc;
  __syncthreads();
  uint64_t before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < TB / 64; ++w) {
    if (w < wave) before += part[w];
    tot += part[w];
  }
  *total = tot;
  return before + inc - x;
}

// ---- edges -> CSC

// From the sorted keys: sources, row offsets, and the number of distinct keys of each tile.
__global__ void __launch_bounds__(TB) k_csc(const uint64_t* __restrict__ keys, int64_t n, int bitsV, int64_t V,
                                            int32_t* __restrict__ col, int64_t* __restrict__ indptr,
                                            int32_t* __restrict__ ucount) {
  const uint64_t mask = ((uint64_t)1 << bitsV) - 1;
  uint32_t uniq = 0;
#pragma unroll
  for (int r = 0; r < ETILE / TB; ++r) {
    const int64_t i = (int64_t)blockIdx.x * ETILE + r * TB + threadIdx.x;
    if (i >= n) break;
    const uint64_t k = keys[i];
    const uint64_t kp = i > 0 ? keys[i - 1] : ~k;
    col[i] = (int32_t)(k & mask);
    uniq += k != kp;
    const int64_t row = (int64_t)(k >> bitsV), rp = i > 0 ? (int64_t)(kp >> bitsV) : -1;
    for (int64_t q = rp + 1; q <= row; ++q) indptr[q] = i;
    if (i == n - 1)
      for (int64_t q = row + 1; q <= V; ++q) indptr[q] = n;
  }
  uint64_t tot;
  block_excl(uniq, &tot);
  if (threadIdx.x == 0) ucount[blockIdx.x] = (int32_t)tot;
}

// Positions of the first entry of every run of equal keys: upos[rank] = i, upos[nU] = n.  A wave takes 512
// consecutive entries, so ranks follow the order of the list.  base[t] = runs before tile t.
struct RunRanks {
  uint64_t m[ETILE / TB];
  int64_t off;     // rank of the wave's first run
  int64_t first;   // the wave's first entry
  __device__ __forceinline__ void find(const uint64_t* __restrict__ keys, int64_t n, const int64_t* __restrict__ base) {
    __shared__ int32_t wtot[TB / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    first = (int64_t)blockIdx.x * ETILE + wave * (ETILE / 4);
    int32_t tot = 0;
#pragma unroll
    for (int r = 0; r < ETILE / TB; ++r) {
      const int64_t i = first + r * 64 + lane;
      const bool start = i < n && (i == 0 || keys[i] != keys[i - 1]);
      m[r] = __ballot(start);
      tot += __popcll(m[r]);
    }
    if (lane == 0) wtot[wave] = tot;
    __syncthreads();
    off = base[blockIdx.x];
    for (int w = 0; w < wave; ++w) off += wtot[w];
  }
};

__global__ void __launch_bounds__(TB) k_runs_fwd(const uint64_t* __restrict__ keys, int64_t n, int bitsV, int64_t V,
                                                 const int64_t* __restrict__ base, int64_t nU, uint32_t* __restrict__ upos,
                                                 int64_t* __restrict__ uindptr) {
  RunRanks R;
  R.find(keys, n, base);
  const int lane = threadIdx.x & 63;
  const uint64_t lt = lanes_below(lane);
#pragma unroll
  for (int r = 0; r < ETILE / TB; ++r) {
    const int64_t i = R.first + r * 64 + lane;
    if (i < n) {
      const int64_t rank = R.off + __popcll(R.m[r] & lt);
      const int64_t row = (int64_t)(keys[i] >> bitsV), rp = i > 0 ? (int64_t)(keys[i - 1] >> bitsV) : -1;
      if ((R.m[r] >> lane) & 1) upos[rank] = (uint32_t)i;
      for (int64_t q = rp + 1; q <= row; ++q) uindptr[q] = rank;
      if (i == n - 1) {
        for (int64_t q = row + 1; q <= V; ++q) uindptr[q] = nU;
        upos[nU] = (uint32_t)n;
      }
    }
    R.off += __popcll(R.m[r]);
  }
}

// distinct pairs in CSC order: source, weight multiplicity * s[source] (rows read in place), multiplicity (rows pre-scaled in the buffer)
__global__ void k_merge_fwd(const uint32_t* __restrict__ upos, int64_t nU, const int32_t* __restrict__ col,
                            const float* __restrict__ s, int32_t* __restrict__ ucol, float* __restrict__ uw,
                            float* __restrict__ umult) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= nU) return;
  const uint32_t e = upos[u];
  const float m = (float)(upos[u + 1] - e);
  const int32_t c = col[e];
  ucol[u] = c;
  uw[u] = m * s[c];
  umult[u] = m;
}

__global__ void k_norm(const int64_t* __restrict__ indptr, int64_t V, float* __restrict__ s) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  const int64_t D = indptr[v + 1] - indptr[v];
  s[v] = D > 0 ? (float)(1.0 / sqrt((double)D)) : 0.f;
}

// Chunk boundaries b[0..n] and their edge offsets.  Edges: b[j] = min{ v in [0, V] : indptr[v] >= ceil(j Ep / n) };
// vertices: b[j] = floor(j V / n).  (j Ep < 2^31 2^32)
__global__ void k_bounds(const int64_t* __restrict__ indptr, int64_t V, int64_t Ep, int32_t n, int mode, int64_t* __restrict__ b,
                         int64_t* __restrict__ eoff) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j > n) return;
  int64_t v;
  if (j == 0) v = 0;
  else if (j == n) v = V;
  else if (mode == HT_BALANCE_VERTICES) v = (int64_t)((uint64_t)j * (uint64_t)V / (uint64_t)n);
  else {
    const int64_t t = (int64_t)(((uint64_t)j * (uint64_t)Ep + (uint64_t)n - 1) / (uint64_t)n);
    int64_t lo = 0, hi = V;   // indptr[V] >= t always
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (indptr[mid] >= t) hi = mid; else lo = mid + 1;
    }
    v = lo;
  }
  b[j] = v;
  eoff[j] = indptr[v];
}

// out[i] = a[at[i]] for a handful of positions
__global__ void k_gather_i64(const int64_t* __restrict__ a, const int64_t* __restrict__ at, int64_t n, int64_t* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = a[at[i]];
}
// out[i] = a[i * stride]
__global__ void k_gather_stride(const int64_t* __restrict__ a, int64_t stride, int64_t n, int64_t* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = a[i * stride];
}

// ---- neighbour bitmaps: row k holds N_k, bit u of it is in word u / 64; rows are padded to whole tiles of 256 words

// The set of sources of a chunk, N_k, as a bitmap.  Marking bits directly needs an atomic OR per entry, and the
// XCDs' L2s only agree on a word through device-scope accesses, which travel to the memory side: with a plain
// test first, then a device-scope test, then the atomic, a 14 M-entry chunk took 258 us (346 without the plain
// test) and a 9.8 M-entry chunk of a 23 M-vertex graph 467 us.  So entries mark a byte per vertex with plain
// stores instead (every writer stores the same 1, the caches merge bytes on write-back, nothing has to be
// coherent before the kernel ends), and a second kernel packs 64 bytes into a word and clears them for the next
// chunks.  A repeated source follows its first copy (sources ascend inside a destination) and is skipped; a byte
// seen set (a cached view can only lag behind) is not stored again.
// Entries [e0, e0 + cnt) of chunks k0, k0 + 1, ...: row k - k0 of `seen`.
__global__ void __launch_bounds__(TB) k_mark_bytes(const int32_t* __restrict__ col, int64_t e0, int64_t cnt,
                                                   const int64_t* __restrict__ eoff, int n, int k0, uint8_t* seen,
                                                   int64_t row_bytes) {
  int k = find_range(eoff, n, e0 + (int64_t)blockIdx.x * ETILE);
  int64_t end = eoff[k + 1], beg = eoff[k];
  // (every entry is a chain of loads: its source, then its byte; eight of them at a time: 64 M entries 520 -> 500 us)
  constexpr int R = ETILE / TB;
  uint8_t* at[R];
  uint32_t u[R], before[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t t = (int64_t)blockIdx.x * ETILE + r * TB + threadIdx.x;
    u[r] = t < cnt ? (uint32_t)col[e0 + t] : 0u;
    before[r] = t < cnt && e0 + t > 0 ? (uint32_t)col[e0 + t - 1] : 0u;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t t = (int64_t)blockIdx.x * ETILE + r * TB + threadIdx.x, e = e0 + t;
    at[r] = nullptr;
    if (t >= cnt) continue;
    while (e >= end) {
      ++k;
      beg = end;
      end = eoff[k + 1];
    }
    if (e == beg || before[r] != u[r]) at[r] = seen + (int64_t)(k - k0) * row_bytes + u[r];
  }
  uint8_t was[R];
#pragma unroll
  for (int r = 0; r < R; ++r) was[r] = at[r] ? *at[r] : 1;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (!was[r]) *at[r] = 1;
}
// bm[w] = bit b set iff seen[64 w + b]; the bytes (0 or 1 each) are cleared, a tile's set bits are counted.  Eight bytes
// become eight bits by one multiplication: byte k sits at bit 8k and the factor's term 2^(56 - 7k) moves it to bit
// 56 + k; no two (byte, term) pairs meet in one bit, so nothing carries.  A block per tile of 256 words.
__global__ void __launch_bounds__(TB) k_pack_seen(uint8_t* seen, uint64_t* __restrict__ bm, int32_t* __restrict__ tile_cnt) {
  const int64_t w = (int64_t)blockIdx.x * TB + threadIdx.x;
  ulonglong2* p = reinterpret_cast<ulonglong2*>(seen + w * 64);
  uint64_t bits = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const ulonglong2 v = p[q];
    bits |= ((v.x * 0x0102040810204080ull) >> 56) << (16 * q);
    bits |= ((v.y * 0x0102040810204080ull) >> 56) << (16 * q + 8);
    if (v.x | v.y) p[q] = make_ulonglong2(0ull, 0ull);
  }
  bm[w] = bits;
  uint64_t tot;
  block_excl((uint64_t)__popcll(bits), &tot);
  if (threadIdx.x == 0) tile_cnt[blockIdx.x] = (int32_t)tot;
}

constexpr int64_t SEEN_BYTES = (int64_t)256 << 20;   // byte maps of as many chunks at once as stay in the last-level cache

// words of a row of the chunks' bitmaps
inline int64_t bm_words(int64_t V) { return ceil_div64(ceil_div64(V, 64), TB) * TB; }
// chunks marked at once
inline int64_t mark_group(int64_t nwp, int32_t n) { return std::max<int64_t>(1, std::min<int64_t>(n, SEEN_BYTES / (nwp * 64))); }

// The neighbour bitmaps of all n chunks (chunk k: entries eoff[k] .. eoff[k + 1] of col) and the set bits of each of
// their tiles; seen: grp rows of nwp * 64 zero bytes.
int mark_chunks(ht_ctx* ctx, hipStream_t st, const int32_t* col, const int64_t* h_eoff, const int64_t* d_eoff, int32_t n,
                int64_t nwp, int64_t grp, uint8_t* seen, uint64_t* bm, int32_t* tile_cnt) {
  const int64_t tiles = nwp / TB;
  for (int64_t k0 = 0; k0 < n; k0 += grp) {
    const int64_t k1 = std::min<int64_t>(n, k0 + grp), cnt = h_eoff[k1] - h_eoff[k0];
    if (cnt > 0) {
      k_mark_bytes<<<nblk(cnt, ETILE), TB, 0, st>>>(col, h_eoff[k0], cnt, d_eoff, n, (int)k0, seen, nwp * 64);
      HT_LAUNCH_CHECK(ctx);
    }
    k_pack_seen<<<(unsigned)((k1 - k0) * tiles), TB, 0, st>>>(seen, bm + k0 * nwp, tile_cnt + k0 * tiles);
    HT_LAUNCH_CHECK(ctx);
  }
  return HT_OK;
}

// ... and of chunk k alone
int mark_chunk(ht_ctx* ctx, hipStream_t st, const int32_t* col, const int64_t* h_eoff, const int64_t* d_eoff, int32_t n, int k,
               int64_t nwp, uint8_t* seen, uint64_t* bm, int32_t* tile_cnt) {
  const int64_t cnt = h_eoff[k + 1] - h_eoff[k];
  if (cnt > 0) {
    k_mark_bytes<<<nblk(cnt, ETILE), TB, 0, st>>>(col, h_eoff[k], cnt, d_eoff, n, k, seen, nwp * 64);
    HT_LAUNCH_CHECK(ctx);
  }
  k_pack_seen<<<(unsigned)(nwp / TB), TB, 0, st>>>(seen, bm, tile_cnt);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}

// p0 + base[t] = set bits before tile t: every word's prefix and the list of set bits (vertex ids, rows behind each other)
// (tile0: the launch's first tile)
__global__ void __launch_bounds__(TB) k_expand_rows(const uint64_t* __restrict__ bm, int64_t nwp, const int64_t* __restrict__ base,
                                                    uint32_t* __restrict__ wpref, int32_t* __restrict__ out, int64_t tile0, int64_t p0) {
  const int64_t tile = tile0 + blockIdx.x, w = tile * TB + threadIdx.x;
  uint64_t bits = bm[w], tot;
  int64_t p = p0 + base[tile] + (int64_t)block_excl((uint64_t)__popcll(bits), &tot);
  if (wpref) wpref[w] = (uint32_t)p;
  const int32_t u0 = (int32_t)((w % nwp) * 64);
  while (bits) {
    out[p++] = u0 + __ffsll((unsigned long long)bits) - 1;
    bits &= bits - 1;
  }
}

// ---- reuse / load / leave lists

// What chunk position j reuses, loads and releases, as words: adjacent reuse (Sec. 5.1) compares the chunk's bitmap with
// those of its neighbours in the schedule; a schedule-aware buffer brings the rows that are resident before chunk j
// (pbm row j, released rows taken out) and the rows that leave after it (ebm row j + 1).
struct ListRows {
  const uint64_t* bm;      // neighbour bitmaps, row = chunk id (or position mod 3)
  const int32_t* order;    // schedule position -> chunk id; nullable: bm holds the rows of positions j0 - 1, j0 and j0 + 1 alone
  const uint64_t* pbm;     // row = position from j0 on; nullable: adjacent reuse
  const uint64_t* ebm;
  int64_t nwp;
  int32_t n;
  int32_t j0, nj;          // the launch's positions
  __device__ __forceinline__ uint64_t word(int j, int64_t w) const { return bm[(int64_t)(order ? order[j] : j % 3) * nwp + w]; }
  __device__ __forceinline__ void words(int j, int64_t w, uint64_t* reuse, uint64_t* load, uint64_t* leave) const {
    const uint64_t cur = word(j, w);
    uint64_t prev, out;
    if (pbm) {
      prev = pbm[(int64_t)(j - j0) * nwp + w];
      out = ebm[(int64_t)(j + 1) * nwp + w];
    } else {
      prev = j > 0 ? word(j - 1, w) : 0ull;
      out = j + 1 < n ? (cur & ~word(j + 1, w)) : cur;
    }
    *reuse = cur & prev;
    *load = cur & ~prev;
    *leave = out;
  }
};

// cnt[0 / 1 / 2][j, tile]: members of a tile of the reuse / load / leave words of position j0 + j
__global__ void __launch_bounds__(TB) k_list_counts(ListRows R, int64_t tiles, int32_t* __restrict__ cnt, int64_t tile0) {
  const int64_t tile = tile0 + blockIdx.x, j = tile / tiles, t = tile % tiles;
  uint64_t a, b, c, tot;
  R.words(R.j0 + (int)j, t * TB + threadIdx.x, &a, &b, &c);
  // three counts of at most 2^14 each travel in one sum
  block_excl((uint64_t)__popcll(a) | ((uint64_t)__popcll(b) << 20) | ((uint64_t)__popcll(c) << 40), &tot);
  if (threadIdx.x < 3) cnt[(int64_t)threadIdx.x * R.nj * tiles + tile] = (int32_t)((tot >> (20 * threadIdx.x)) & 0xFFFFF);
}

__device__ __forceinline__ void put_bits(uint64_t bits, int32_t u0, int32_t* __restrict__ out) {
  while (bits) {
    *out++ = u0 + __ffsll((unsigned long long)bits) - 1;
    bits &= bits - 1;
  }
}

// the three lists, positions behind each other; base: exclusive prefix over cnt
__global__ void __launch_bounds__(TB) k_list_expand(ListRows R, int64_t tiles, const int64_t* __restrict__ base,
                                                    int32_t* __restrict__ reuse, int32_t* __restrict__ load,
                                                    int32_t* __restrict__ leave, int64_t tile0) {
  const int64_t tile = tile0 + blockIdx.x, j = tile / tiles, t = tile % tiles, nt = (int64_t)R.nj * tiles;
  uint64_t a, b, c, tot;
  R.words(R.j0 + (int)j, t * TB + threadIdx.x, &a, &b, &c);
  const uint64_t off = block_excl((uint64_t)__popcll(a) | ((uint64_t)__popcll(b) << 20) | ((uint64_t)__popcll(c) << 40), &tot);
  const int32_t u0 = (int32_t)((t * TB + threadIdx.x) * 64);
  put_bits(a, u0, reuse + base[tile] + (int64_t)(off & 0xFFFFF));
  put_bits(b, u0, load + (base[nt + tile] - base[nt]) + (int64_t)((off >> 20) & 0xFFFFF));
  put_bits(c, u0, leave + (base[2 * nt + tile] - base[2 * nt]) + (int64_t)((off >> 40) & 0xFFFFF));
}

// out[0 .. 3]: members of one chunk's N, reuse, load and leave lists, from the prefix sums over their tiles
__global__ void k_put_counts(const int64_t* __restrict__ tbase, const int64_t* __restrict__ lbase, int64_t tiles, int64_t* __restrict__ out) {
  const int w = threadIdx.x;
  if (w < 4) out[w] = w == 0 ? tbase[tiles] : lbase[w * tiles] - lbase[(w - 1) * tiles];
}

// Sum of up to three per-thread counts over the grid into totals[0..2]: waves by shuffles, the block's four waves
// through LDS, one atomic add per block and total (with one add per wave the adds of a 23 M-bit bitmap, all to the
// same three words, took 180 us).  Launch with a bounded grid; the callers stride.
__device__ __forceinline__ void block_add2(unsigned long long a, unsigned long long b, unsigned long long* __restrict__ totals, int ntot) {
  __shared__ unsigned long long part[4][2];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_down(a, o, 64);
    b += __shfl_down(b, o, 64);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    part[wave][0] = a;
    part[wave][1] = b;
  }
  __syncthreads();
  if ((int)threadIdx.x < ntot) {
    unsigned long long t = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += part[w][threadIdx.x];
    if (t) atomicAdd(&totals[threadIdx.x], t);
  }
}
constexpr int POPC_GRID = 256;
inline unsigned popc_grid(int64_t nw) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(nblk(nw), POPC_GRID)); }

// ---- row-buffer schedule with a known future (release for room, farthest next use first)
__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
// nxt[i] = position of the next chunk after j that needs N_j[i] (n: none); chunks are visited last to first
__global__ void k_next_use(const int32_t* __restrict__ nbr, int64_t n, int32_t* __restrict__ last, int32_t j,
                           int32_t* __restrict__ nxt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t u = nbr[i];
  nxt[i] = last[u];
  last[u] = j;
}
__global__ void k_set_nu(const int32_t* __restrict__ nbr, int64_t n, const int32_t* __restrict__ nxt,
                         int32_t* __restrict__ nu) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) nu[nbr[i]] = nxt[i];
}
// totals[0] += |R u cur|, totals[1] += |R ^ cur|
__global__ void __launch_bounds__(256) k_popc_union(const uint64_t* __restrict__ R, const uint64_t* __restrict__ cur,
                                                    int64_t nw, unsigned long long* __restrict__ totals) {
  unsigned long long a = 0, b = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw; i += (int64_t)gridDim.x * blockDim.x) {
    a += __popcll(R[i] | cur[i]);
    b += __popcll(R[i] & cur[i]);
  }
  block_add2(a, b, totals, 2);
}
// totals[0] += members of the union of the n rows
__global__ void __launch_bounds__(256) k_popc_all(const uint64_t* __restrict__ bm, int64_t nwp, int32_t n,
                                                  unsigned long long* __restrict__ totals) {
  unsigned long long a = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nwp; i += (int64_t)gridDim.x * blockDim.x) {
    uint64_t w = 0;
    for (int32_t k = 0; k < n; ++k) w |= bm[(int64_t)k * nwp + i];
    a += __popcll(w);
  }
  block_add2(a, 0, totals, 1);
}
// hist[nu[u]] += 1 for every u in the candidate set (integer counts: order does not matter).
// nbins <= HIST_LDS_BINS: counted per block in LDS first, so the few global bins see one add per block.
constexpr int HIST_LDS_BINS = 4096;
__global__ void k_hist_nu(const uint64_t* __restrict__ cand, int64_t nw, const int32_t* __restrict__ nu, int nbins,
                          unsigned int* __restrict__ hist) {
  __shared__ unsigned int h[HIST_LDS_BINS];
  const bool local = nbins <= HIST_LDS_BINS;
  if (local) {
    for (int b = threadIdx.x; b < nbins; b += blockDim.x) h[b] = 0;
    __syncthreads();
  }
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw; i += (int64_t)gridDim.x * blockDim.x) {
    uint64_t w = cand[i];
    while (w) {
      const int b = __ffsll((long long)w) - 1;
      w &= w - 1;
      const int32_t x = nu[i * 64 + b];
      if (local) atomicAdd(&h[x], 1u);
      else atomicAdd(&hist[x], 1u);
    }
  }
  if (local) {
    __syncthreads();
    for (int b = threadIdx.x; b < nbins; b += blockDim.x)
      if (h[b]) atomicAdd(&hist[b], h[b]);
  }
}
// gt = candidates whose next use lies beyond t, eq = candidates whose next use is t
__global__ void k_select_nu(const uint64_t* __restrict__ cand, int64_t nw, const int32_t* __restrict__ nu, int32_t t,
                            uint64_t* __restrict__ gt, uint64_t* __restrict__ eq) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nw) return;
  uint64_t w = cand[i], g = 0, e = 0;
  while (w) {
    const int b = __ffsll((long long)w) - 1;
    w &= w - 1;
    const int32_t x = nu[i * 64 + b];
    if (x > t) g |= 1ull << b;
    else if (x == t) e |= 1ull << b;
  }
  gt[i] |= g;      // the row may already hold the rows that left after their last use
  eq[i] = e;
}
// rows of N_j that no later chunk needs: set in bm, counted into *count
__global__ void k_mark_dead(const int32_t* __restrict__ nbr, int64_t n, const int32_t* __restrict__ nxt, int32_t never,
                            uint32_t* bm32, unsigned long long* __restrict__ count) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool dead = i < n && nxt[i] == never;
  if (dead) {
    const uint32_t u = (uint32_t)nbr[i];
    atomicOr(&bm32[u >> 5], 1u << (u & 31));
  }
  const unsigned long long m = __ballot(dead);
  if ((threadIdx.x & 63) == 0 && m) atomicAdd(count, (unsigned long long)__popcll(m));
}
// out |= the m members of eq with the smallest ids (pref = exclusive prefix of eq's per-word popcounts)
__global__ void k_take_first(const uint64_t* __restrict__ eq, const int64_t* __restrict__ pref, int64_t nw, int64_t m,
                             uint64_t* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nw) return;
  int64_t room = m - pref[i];
  if (room <= 0) return;
  uint64_t w = eq[i], keep = 0;
  while (w && room > 0) {
    const uint64_t low = w & (~w + 1);
    keep |= low;
    w ^= low;
    --room;
  }
  out[i] |= keep;
}

// out[k] += popc(bms[k] & last) for every candidate bitmap k (grid.y = k)
__global__ void k_overlap(const uint64_t* __restrict__ bms, int64_t nw, const uint64_t* __restrict__ last,
                          unsigned long long* __restrict__ out) {
  const int k = blockIdx.y;
  const uint64_t* bm = bms + (int64_t)k * nw;
  unsigned long long a = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw; i += (int64_t)gridDim.x * blockDim.x)
    a += __popcll(bm[i] & last[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a += __shfl_down(a, o, 64);
  if ((threadIdx.x & 63) == 0 && a) atomicAdd(&out[k], a);
}

__global__ void k_bm_or(uint64_t* __restrict__ acc, const uint64_t* __restrict__ x, int64_t nw) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nw) acc[i] |= x[i];
}
// out = a & ~b (out may be a)
__global__ void k_bm_minus(const uint64_t* a, const uint64_t* __restrict__ b, int64_t nw, uint64_t* out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nw) out[i] = a[i] & ~b[i];
}

// ---- buffer positions (Sec. 6), chunk by chunk

// every position free: ones, the last word cut to C bits
__global__ void k_free_init(uint64_t* __restrict__ bm, int64_t nwC, int64_t C) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nwC) bm[i] = (i == nwC - 1 && (C & 63)) ? (~0ull >> (64 - (C & 63))) : ~0ull;
}
__global__ void __launch_bounds__(TB) k_free_count(const uint64_t* __restrict__ bm, int64_t nwC, int32_t* __restrict__ tile_cnt) {
  const int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x;
  uint64_t tot;
  block_excl(i < nwC ? (uint64_t)__popcll(bm[i]) : 0ull, &tot);
  if (threadIdx.x == 0) tile_cnt[blockIdx.x] = (int32_t)tot;
}
// The loaded rows take the lowest free positions: free position number r goes to load[r].  A block hands out one tile of
// 256 words; the free positions before it are the sum over the tiles before (tile_cnt), or over the words before when
// there are few.  in -> out: blocks must not see each other's positions taken.
__global__ void __launch_bounds__(TB) k_assign(const uint64_t* __restrict__ in, uint64_t* __restrict__ out, int64_t nwC,
                                               const int32_t* __restrict__ tile_cnt, const int32_t* __restrict__ load,
                                               int64_t n_load, int32_t* __restrict__ vslot, int32_t* __restrict__ load_slot) {
  const int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x;
  uint64_t before = 0, tot;
  if (tile_cnt)
    for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += TB) before += (uint64_t)tile_cnt[t];
  else
    for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x * TB; t += TB) before += (uint64_t)__popcll(in[t]);
  block_excl(before, &before);
  uint64_t w = i < nwC ? in[i] : 0ull;
  int64_t r = (int64_t)(before + block_excl((uint64_t)__popcll(w), &tot));
  if (i >= nwC) return;
  while (w && r < n_load) {
    const int b = __ffsll((unsigned long long)w) - 1;
    const int32_t sl = (int32_t)(i * 64 + b);
    vslot[load[r]] = sl;
    load_slot[r] = sl;
    w &= w - 1;
    ++r;
  }
  out[i] = w;
}
// Positions of the members of N_j (with bit 31 where a member was not resident before), and of the rows that leave after
// chunk j, which become free.
__global__ void k_lookup_evict(const int32_t* __restrict__ nbr, int64_t nsrc, const int32_t* __restrict__ vslot,
                               const uint64_t* __restrict__ prev_bm, int32_t* __restrict__ slot, int32_t* __restrict__ gslot,
                               const int32_t* __restrict__ leave, int64_t n_leave, uint32_t* freebm32,
                               int32_t* __restrict__ leave_slot) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nsrc) {
    const uint32_t u = (uint32_t)nbr[i];
    const int32_t sl = vslot[u];
    slot[i] = sl;
    const bool was = prev_bm && ((prev_bm[u >> 6] >> (u & 63)) & 1ull);
    gslot[i] = was ? sl : (int32_t)((uint32_t)sl | 0x80000000u);
    return;
  }
  i -= nsrc;
  if (i >= n_leave) return;
  const int32_t sl = vslot[leave[i]];
  leave_slot[i] = sl;
  atomicOr(&freebm32[(uint32_t)sl >> 5], 1u << (sl & 31));
}

// ---- topology in local indices

// For the edges [e0, e1) in CSC order (bm, wpref: from chunk k0's row on): the position of its source in N_k, its buffer position, and the sort key
// (position of (k, source) in the N arena, local destination) of the by-source grouping.
__global__ void __launch_bounds__(TB) k_remap(const uint64_t* __restrict__ csc_keys, int64_t e0, int64_t e1, int k0, int bitsV,
                                              const int64_t* __restrict__ eoff, const int64_t* __restrict__ bounds,
                                              const int64_t* __restrict__ noff, int n, const uint64_t* __restrict__ bm,
                                              int64_t nwp, const uint32_t* __restrict__ wpref, const int32_t* __restrict__ slot,
                                              int32_t* __restrict__ col_local, int32_t* __restrict__ col_slot,
                                              uint64_t* __restrict__ keys) {
  int k = find_range(eoff, n, e0 + (int64_t)blockIdx.x * ETILE);
  int64_t end = eoff[k + 1];
  const uint64_t mask = ((uint64_t)1 << bitsV) - 1;
  // (every entry is a chain of loads: its key, its word of the bitmap and the count before it, its buffer position; RB of them at a time: 64 M
  // entries 901 -> 805 us, three scattered loads an entry)
  constexpr int RB = 4;
#pragma unroll 1
  for (int r0 = 0; r0 < ETILE / TB; r0 += RB) {
    uint64_t key[RB], word[RB];
    uint32_t p[RB];
    int ck[RB];
    int32_t sl[RB];
    const int64_t first = e0 + (int64_t)blockIdx.x * ETILE + r0 * TB + threadIdx.x;
#pragma unroll
    for (int r = 0; r < RB; ++r) key[r] = csc_keys[first + r * TB < e1 ? first + r * TB : e1 - 1];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int64_t e = first + r * TB;
      while (e < e1 && e >= end) end = eoff[++k + 1];
      ck[r] = k;
      // (behind the last entry: that one again, nothing is written)
      const int64_t w = (int64_t)(k - k0) * nwp + (int64_t)((uint32_t)(key[r] & mask) >> 6);
      word[r] = bm[w];
      p[r] = wpref[w];
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const uint32_t b = (uint32_t)(key[r] & mask) & 63;
      p[r] += (uint32_t)__popcll(b ? word[r] & (~0ull >> (64 - b)) : 0ull);
      sl[r] = first + r * TB < e1 ? slot[p[r]] : 0;
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int64_t e = first + r * TB;
      if (e >= e1) break;
      col_local[e] = (int32_t)((int64_t)p[r] - noff[ck[r]]);
      col_slot[e] = sl[r];
      keys[e] = ((uint64_t)p[r] << 32) | (uint64_t)((int64_t)(key[r] >> bitsV) - bounds[ck[r]]);
    }
  }
}

// From the keys sorted by arena position: local destinations, offsets of every local source inside its chunk
// (chunk k's nsrc + 1 offsets start at arena position + k), distinct keys per tile (nullable).
__global__ void __launch_bounds__(TB) k_by_source(const uint64_t* __restrict__ keys, int64_t n_edges,
                                                  const int64_t* __restrict__ eoff, int n, int32_t* __restrict__ sdst,
                                                  int64_t* __restrict__ sptr, int32_t* __restrict__ ucount) {
  int k = find_range(eoff, n, (int64_t)blockIdx.x * ETILE);
  int64_t end = eoff[k + 1], beg = eoff[k];
  uint32_t uniq = 0;
#pragma unroll
  for (int r = 0; r < ETILE / TB; ++r) {
    const int64_t i = (int64_t)blockIdx.x * ETILE + r * TB + threadIdx.x;
    if (i >= n_edges) break;
    while (i >= end) {
      ++k;
      beg = end;
      end = eoff[k + 1];
    }
    const uint64_t key = keys[i], kp = i > 0 ? keys[i - 1] : ~key;
    sdst[i] = (int32_t)(key & 0xFFFFFFFFull);
    if ((key >> 32) != (kp >> 32)) sptr[(int64_t)(key >> 32) + k] = i - beg;
    uniq += key != kp;
  }
  if (!ucount) return;
  uint64_t tot;
  block_excl(uniq, &tot);
  if (threadIdx.x == 0) ucount[blockIdx.x] = (int32_t)tot;
}
// the closing offset of every chunk: its number of entries
__global__ void k_sptr_ends(const int64_t* __restrict__ noff, const int64_t* __restrict__ eoff, int n, int64_t* __restrict__ sptr) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) sptr[noff[k + 1] + k] = eoff[k + 1] - eoff[k];
}
// the same for the distinct (source, destination) pairs
__global__ void __launch_bounds__(TB) k_runs_bwd(const uint64_t* __restrict__ keys, int64_t n_edges,
                                                 const int64_t* __restrict__ base, int64_t nU, const int64_t* __restrict__ eoff,
                                                 const int64_t* __restrict__ ueoff, int n, uint32_t* __restrict__ upos,
                                                 int64_t* __restrict__ usptr) {
  RunRanks R;
  R.find(keys, n_edges, base);
  const int lane = threadIdx.x & 63;
  const uint64_t lt = lanes_below(lane);
  int k = find_range(eoff, n, (int64_t)blockIdx.x * ETILE);
  int64_t end = eoff[k + 1];
#pragma unroll
  for (int r = 0; r < ETILE / TB; ++r) {
    const int64_t i = R.first + r * 64 + lane;
    if (i < n_edges) {
      while (i >= end) end = eoff[++k + 1];
      const int64_t rank = R.off + __popcll(R.m[r] & lt);
      if ((R.m[r] >> lane) & 1) {
        upos[rank] = (uint32_t)i;
        if (i == 0 || (keys[i] >> 32) != (keys[i - 1] >> 32)) usptr[(int64_t)(keys[i] >> 32) + k] = rank - ueoff[k];
      }
      if (i == n_edges - 1) upos[nU] = (uint32_t)n_edges;
    }
    R.off += __popcll(R.m[r]);
  }
}
// by-source distinct pairs: local destination, weight multiplicity * s[destination], multiplicity
__global__ void __launch_bounds__(TB) k_merge_bwd(const uint32_t* __restrict__ upos, int64_t nU, const uint64_t* __restrict__ keys,
                                                  const int64_t* __restrict__ ueoff, const int64_t* __restrict__ bounds, int n,
                                                  const float* __restrict__ s, int32_t* __restrict__ usdst,
                                                  float* __restrict__ uw, float* __restrict__ umult) {
  int k = find_range(ueoff, n, (int64_t)blockIdx.x * ETILE);
  int64_t end = ueoff[k + 1];
#pragma unroll
  for (int r = 0; r < ETILE / TB; ++r) {
    const int64_t u = (int64_t)blockIdx.x * ETILE + r * TB + threadIdx.x;
    if (u >= nU) break;
    while (u >= end) end = ueoff[++k + 1];
    const uint32_t t = upos[u];
    const float m = (float)(upos[u + 1] - t);
    const int32_t d = (int32_t)(keys[t] & 0xFFFFFFFFull);
    usdst[u] = d;
    uw[u] = m * s[bounds[k] + d];
    umult[u] = m;
  }
}
__global__ void k_gather_i32(const int32_t* __restrict__ table, const uint32_t* __restrict__ at, int64_t n, int32_t* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = table[at[i]];
}

// ---- work items

// The rows of one direction: destinations (entries ptr[r] .. ptr[r + 1]), or positions of the N arena, whose offsets are
// relative to their chunk (chunk k's entries start at eoff[k], its offsets at arena position + k).
struct RowSet {
  const int64_t* ptr;
  const int64_t* first;    // [n + 1] first row of every chunk
  const int64_t* eoff;     // nullptr: destinations
  int n;
  const int32_t* pos = nullptr;   // rows with pos[r] >= 0 are cut rows however short they are (and without an item where they are empty)
  __device__ __forceinline__ void get(int64_t r, int k, int64_t* e0, int64_t* len) const {
    const int64_t* p = ptr + r + (eoff ? k : 0);
    *e0 = p[0] + (eoff ? eoff[k] : 0);
    *len = p[1] - p[0];
  }
  __device__ __forceinline__ bool forced(int64_t r) const { return pos && pos[r] >= 0; }
  // items of row r
  __device__ __forceinline__ uint64_t items(int64_t len, int seg, bool forced) const {
    return len > seg ? (uint64_t)((len + seg - 1) / seg) : forced && len == 0 ? 0 : 1;
  }
};

// items, items of cut rows, cut rows of every tile of RTILE rows
__global__ void __launch_bounds__(TB) k_items_count(RowSet R, int64_t nrows, int seg, int64_t tiles, int32_t* __restrict__ cnt) {
  int k = find_range(R.first, R.n, (int64_t)blockIdx.x * RTILE);
  int64_t end = R.first[k + 1];
  uint64_t items = 0, parts = 0, cuts = 0;
#pragma unroll
  for (int q = 0; q < RTILE / TB; ++q) {
    const int64_t r = (int64_t)blockIdx.x * RTILE + q * TB + threadIdx.x;
    if (r >= nrows) break;
    while (r >= end) end = R.first[++k + 1];
    int64_t e0, len;
    R.get(r, k, &e0, &len);
    const bool forced = R.forced(r);
    const uint64_t m = R.items(len, seg, forced);
    items += m;
    parts += m > 1 || forced ? m : 0;
    cuts += m > 1 || forced;
  }
  uint64_t t1, t2;
  block_excl(items | (cuts << 40), &t1);
  block_excl(parts, &t2);
  if (threadIdx.x == 0) {
    cnt[blockIdx.x] = (int32_t)(t1 & 0xFFFFFFFFFFull);
    cnt[tiles + blockIdx.x] = (int32_t)t2;
    cnt[2 * tiles + blockIdx.x] = (int32_t)(t1 >> 40);
  }
}

// The items in row order, their dispatch keys, the cut rows, and where every chunk's share starts (starts[0 / 1 / 2][k]).
// Dispatch order: chunk by chunk, inside a chunk by the first row an item reads (entries of a row are sorted by that
// index), so items in flight together read neighbouring rows.  fbits: bits of the key left for that row; a wider index
// is rounded down (the order is about locality only).  The items of rows cut into more than FILL_ALONE are left to k_items_fill_cut: a
// thread that wrote a hub's thousands one after the other held up the whole launch (116 k vertices, 57 M edges by source: 491 us,
// the two launches 33).
constexpr int FILL_ALONE = 4;
struct ItemOut {
  int seg, fbits, fshift, classes;   // classes: bits of the key in front of that row for the item's length, longest first
  const int32_t* idx;
  WorkItem* item;
  uint64_t* keys;
  __device__ __forceinline__ void put(uint32_t row, int k, int64_t e0, int64_t len, int64_t i0, int64_t p0, int64_t j) const {   // p0 < 0: not cut
    const int64_t b = e0 + j * seg, rem = len - j * seg;
    WorkItem w;
    w.row = row;
    w.e0 = (uint32_t)b;
    w.len = (int32_t)(rem < seg ? rem : seg);
    w.part = p0 >= 0 ? (int32_t)(p0 + j) : -1;
    item[i0 + j] = w;
    if (keys) {
      const uint32_t f = w.len > 0 ? (uint32_t)idx[b] >> fshift : 0u;
      const uint32_t c = classes ? (uint32_t)(((int64_t)(seg - w.len) << classes) / (seg + 1)) : 0u;
      keys[i0 + j] = ((((((uint64_t)k << classes) | c) << fbits) | f) << 32) | (uint64_t)(uint32_t)(i0 + j);
    }
  }
};
__global__ void __launch_bounds__(TB) k_items_fill(RowSet R, int64_t nrows, int64_t tiles, const int64_t* __restrict__ base, ItemOut out,
                                                   CutRow* __restrict__ cut, int64_t* __restrict__ starts) {
  const int seg = out.seg;
  int k = find_range(R.first, R.n, (int64_t)blockIdx.x * RTILE);
  int64_t end = R.first[k + 1];
  const int n1 = R.n + 1;
  int64_t at_i = base[blockIdx.x], at_p = base[tiles + blockIdx.x] - base[tiles], at_c = base[2 * tiles + blockIdx.x] - base[2 * tiles];
  for (int q = 0; q < RTILE / TB; ++q) {
    const int64_t r = (int64_t)blockIdx.x * RTILE + q * TB + threadIdx.x;
    int64_t e0 = 0, len = 0;
    uint64_t m = 0;
    bool is_cut = false;
    if (r < nrows) {
      while (r >= end) end = R.first[++k + 1];
      R.get(r, k, &e0, &len);
      const bool forced = R.forced(r);
      m = R.items(len, seg, forced);
      is_cut = m > 1 || forced;
    }
    uint64_t t1, t2;
    const uint64_t x = block_excl(m | ((uint64_t)is_cut << 40), &t1);
    const uint64_t y = block_excl(is_cut ? m : 0, &t2);
    const int64_t i0 = at_i + (int64_t)(x & 0xFFFFFFFFFFull), p0 = at_p + (int64_t)y, c0 = at_c + (int64_t)(x >> 40);
    if (r < nrows) {
      for (int kk = k; kk >= 0 && R.first[kk] == r; --kk) {   // chunks that start at this row (empty ones before it too)
        starts[kk] = i0;
        starts[n1 + kk] = p0;
        starts[2 * n1 + kk] = c0;
      }
      if (m <= FILL_ALONE)
        for (int64_t j = 0; j < (int64_t)m; ++j) out.put((uint32_t)r, k, e0, len, i0, is_cut ? p0 : -1, j);
      if (is_cut) {
        CutRow c;
        c.row = (uint32_t)r;
        c.part0 = (int32_t)p0;
        c.nseg = (int32_t)m;
        c.item0 = (uint32_t)i0;
        cut[c0] = c;
      }
    }
    at_i += (int64_t)(t1 & 0xFFFFFFFFFFull);
    at_p += (int64_t)t2;
    at_c += (int64_t)(t1 >> 40);
  }
}

// the items of the rows that k_items_fill left out, a wave per cut row
__global__ void __launch_bounds__(TB) k_items_fill_cut(RowSet R, const CutRow* __restrict__ cut, int64_t n_cut, ItemOut out) {
  const int64_t f = (int64_t)blockIdx.x * (TB / 64) + (threadIdx.x >> 6);
  if (f >= n_cut) return;
  const CutRow c = cut[f];
  if (c.nseg <= FILL_ALONE) return;
  const int k = find_range(R.first, R.n, c.row);
  int64_t e0, len;
  R.get(c.row, k, &e0, &len);
  for (int32_t j = threadIdx.x & 63; j < c.nseg; j += 64) out.put(c.row, k, e0, len, c.item0, c.part0, j);
}

// (in: from item i0 on)
__global__ void k_items_permute(const uint64_t* __restrict__ keys, int64_t n, const WorkItem* __restrict__ in, uint32_t i0, WorkItem* __restrict__ out) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) out[t] = in[(uint32_t)(keys[t] & 0xFFFFFFFFull) - i0];
}

// ---- entries of the whole graph grouped by source

// members of the N arena: entries per vertex (added over the chunks)
__global__ void k_src_counts(const int32_t* __restrict__ nbr, RowSet R, int64_t nrows, int32_t* __restrict__ cnt) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nrows) return;
  int64_t e0, len;
  R.get(p, find_range(R.first, R.n, p), &e0, &len);
  atomicAdd(&cnt[nbr[p]], (int32_t)len);
}
// off[p] = where the entries of (chunk, source) p go; chunk by chunk in vertex order, so that a source's destinations ascend
__global__ void k_src_offsets(const int32_t* __restrict__ nbr, RowSet R, int k, int64_t p0, int64_t n, int64_t* __restrict__ cur,
                              int64_t* __restrict__ off) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int64_t e0, len;
  R.get(p0 + i, k, &e0, &len);
  const int32_t u = nbr[p0 + i];
  off[p0 + i] = cur[u] - e0;   // entry e of the chunk's list goes to off + e
  cur[u] += len;
}
// SRC_LANES lanes per backward work item copy its entries: destination in vertex ids, weight.  What bounds it is the chain of loads
// before an item's first entry, so the more items in flight the better (most have a few dozen entries; 116 k vertices, 57 M edges in 7
// chunks: 234 us, a wave per item 351).
constexpr int SRC_LANES = 16;
__global__ void __launch_bounds__(TB) k_src_copy(const WorkItem* __restrict__ items, int64_t n_items, const int64_t* __restrict__ first,
                                                 const int64_t* __restrict__ bounds, int n, const int64_t* __restrict__ off,
                                                 const int32_t* __restrict__ sdst, const float* __restrict__ w,
                                                 int32_t* __restrict__ idx, float* __restrict__ w_out) {
  const int64_t t = (int64_t)blockIdx.x * (TB / SRC_LANES) + threadIdx.x / SRC_LANES;
  if (t >= n_items) return;
  const WorkItem it = items[t];
  const int64_t to = off[it.row] + it.e0;
  const int32_t d0 = (int32_t)bounds[find_range(first, n, it.row)];
  for (int32_t i0 = threadIdx.x % SRC_LANES; i0 < it.len; i0 += 4 * SRC_LANES) {
    int32_t d[4];
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t i = i0 + q * SRC_LANES;
      const int64_t e = (int64_t)it.e0 + (i < it.len ? i : i0);
      d[q] = sdst[e];
      if (w) v[q] = w[e];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t i = i0 + q * SRC_LANES;
      if (i >= it.len) break;
      idx[to + i] = d0 + d[q];
      if (w) w_out[to + i] = v[q];
    }
  }
}

// The multiplicity out of w = multiplicity * s[destination]: both roundings together are off by less than 2^-23 of it, so
// rounding to a whole number gives it back exactly below 2^22 (and its fp32 neighbour above).
__global__ void __launch_bounds__(TB) k_src_mult(const float* __restrict__ w, const int32_t* __restrict__ idx, const float* __restrict__ s,
                                                 int64_t n, float* __restrict__ mult) {
  for (int64_t e = (int64_t)blockIdx.x * TB + threadIdx.x; e < n; e += (int64_t)gridDim.x * TB) mult[e] = rintf(w[e] / s[idx[e]]);
}

int bits_for(int64_t n) {  // bits needed for values 0..n-1 (at least 1)
  int b = 1;
  while (((int64_t)1 << b) < n) ++b;
  return b;
}

// One direction's work items over a set of rows: counted, then filled and put into dispatch order.
struct ItemBuild {
  RowSet rows;
  int64_t nrows = 0, tiles = 0;
  int64_t range = 0;           // values of the entries' row index are below this
  int seg = 0, classes = 0;
  const int64_t* h_first = nullptr;   // host copy of rows.first
  const int32_t* idx = nullptr;
  int32_t* cnt = nullptr;      // [3 * tiles]
  int64_t* base = nullptr;     // [3 * tiles + 1]
  int64_t* starts = nullptr;   // [3 * (rows.n + 1)]
  GraphItems* out = nullptr;
};

// Items a list of `rows` rows with `entries` entries can make: ceil(len / seg) per row, at least one.
inline int64_t item_bound(int64_t rows, int64_t entries, int seg) { return ht_row_items_bound(rows, entries, seg); }
inline int64_t cut_bound(int64_t entries, int seg) { return ht_row_cuts_bound(entries, seg, 0); }

// h_tot (pinned, 3 words): the totals' prefix sums, valid once the stream is synchronised
int count_items(ht_ctx* ctx, const ItemBuild& b, int64_t* h_tot) {
  if (b.nrows == 0) return HT_OK;
  k_items_count<<<(unsigned)b.tiles, TB, 0, ctx->stream>>>(b.rows, b.nrows, b.seg, b.tiles, b.cnt);
  HT_LAUNCH_CHECK(ctx);
  HT_TRY(ht_scan_i32(ctx, b.cnt, b.base, 3 * b.tiles, true));
  void* d_tot = nullptr;     // (one launch that writes to the host: a copy each took longer)
  HT_HIP(ctx, hipHostGetDevicePointer(&d_tot, h_tot, 0));
  k_gather_stride<<<1, TB, 0, ctx->stream>>>(b.base + b.tiles, b.tiles, 3, (int64_t*)d_tot);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}

// Items go into dispatch order however few they are and however few rows they read: row order (the sort is six launches a direction) was faster to make and slower to
// use.  Partition and one layer of 10,000 vertices, 100,000 edges, 40 columns 495 us sorted, 430 in row order; but in row order neighbouring rows, which in many graphs
// are alike in length, fall to the same CUs and XCDs: us of an aggregation sorted | in row order, 8,000 vertices, 40 edges a row, 128 columns 29.8 | 39.2, 256
// columns 51 | 70; 10 a row 25.6 | 31.7, 46 | 56; 4,000 vertices, 10 a row, 256 columns 39 | 43; an epoch of 10,000 vertices, 100,000 edges, 64-32-8 111 | 117.
// made: room for n_made items in row order, before they are permuted; keysA, keysB: nkeys words each.  Where made does not hold all
// items, they are put in order range by range (the order is by range first in any case; h_starts: pinned, rows.n + 1 words).
int fill_items(ht_ctx* ctx, const ItemBuild& b, const int64_t* h_tot, WorkItem* made, size_t n_made, uint64_t* keysA, uint64_t* keysB,
               size_t nkeys, bool order, int64_t* h_starts = nullptr) {
  if (b.nrows == 0) return HT_OK;
  const int64_t ni = h_tot[0], np = h_tot[1] - h_tot[0], nc = h_tot[2] - h_tot[1];
  if (ni > (int64_t)b.out->items.n || nc > (int64_t)b.out->cuts.n || ni > (int64_t)nkeys)
    return ht_set_err(ctx, HT_ESTATE, "work items: %lld items and %lld cut rows, more than was planned for", (long long)ni, (long long)nc);
  b.out->n_items = ni;
  b.out->n_part = np;
  b.out->n_cut = nc;
  const bool sorted_items = order && ni > 1, at_once = ni <= (int64_t)n_made;
  const int kbits = b.rows.n > 1 ? bits_for(b.rows.n) : 0, vbits = bits_for(b.range);
  const int fbits = std::min(vbits, 32 - kbits - b.classes), fshift = vbits - fbits;
  const ItemOut to{b.seg, fbits, fshift, b.classes, b.idx, sorted_items && at_once ? made : b.out->items.p, sorted_items ? keysA : nullptr};
  k_items_fill<<<(unsigned)b.tiles, TB, 0, ctx->stream>>>(b.rows, b.nrows, b.tiles, b.base, to, b.out->cuts.p, b.starts);
  HT_LAUNCH_CHECK(ctx);
  if (np > FILL_ALONE)
    HT_TRY(ht_in_launches(nc, HT_LAUNCH_WAVES, [&](int64_t i, int64_t m) {
      k_items_fill_cut<<<nblk(m, TB / 64), TB, 0, ctx->stream>>>(b.rows, b.out->cuts.p + i, m, to);
      HT_LAUNCH_CHECK(ctx);
      return (int)HT_OK;
    }));
  if (!sorted_items) return HT_OK;
  auto sort_range = [&](int64_t i0, int64_t n, const WorkItem* from, int bits) -> int {
    uint64_t* sorted = nullptr;
    HT_TRY(ht_radix_sort_u64(ctx, keysA + i0, keysB + i0, n, 32, 32 + bits, &sorted));
    k_items_permute<<<nblk(n), TB, 0, ctx->stream>>>(sorted, n, from, (uint32_t)i0, b.out->items.p + i0);
    HT_LAUNCH_CHECK(ctx);
    return HT_OK;
  };
  if (at_once) return sort_range(0, ni, made, kbits + b.classes + fbits);
  HT_HIP(ctx, hipMemcpyAsync(h_starts, b.starts, ((size_t)b.rows.n + 1) * 8, hipMemcpyDeviceToHost, ctx->stream));
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  // (a range behind the last row has no start of its own)
  const std::vector<int64_t> starts(h_starts, h_starts + b.rows.n);
  int64_t end = ni;
  for (int k = b.rows.n - 1; k >= 0; --k) {
    if (b.h_first[k] >= b.nrows) continue;
    const int64_t i0 = starts[k], n = end - i0;
    end = i0;
    if (n <= 1) continue;
    if (n > (int64_t)n_made) return ht_set_err(ctx, HT_ESTATE, "work items: a chunk has %lld, more than was planned for", (long long)n);
    HT_HIP(ctx, hipMemcpyAsync(made, b.out->items.p + i0, (size_t)n * sizeof(WorkItem), hipMemcpyDeviceToDevice, ctx->stream));
    HT_TRY(sort_range(i0, n, made, b.classes + fbits));
  }
  return HT_OK;
}

struct ItemSwitches {          // experiments
  int seg_fwd = HT_SEG, seg_bwd = HT_SEG / 2;   // measured best at 233 k vertices / 115 M edges
  bool order = true;
  ItemSwitches() {
    if (const char* v = getenv("HT_SEG_FWD")) seg_fwd = std::max(64, atoi(v));
    if (const char* v = getenv("HT_SEG_BWD")) seg_bwd = std::max(64, atoi(v));
    if (const char* v = getenv("HT_ITEM_ORDER")) order = atoi(v) != 0;
  }
};

// Bytes of bitmaps and word prefixes up to which all chunks' rows are held at once.  Beyond (n V / 8 bytes of bitmaps alone: many
// chunks of many vertices), and where all rows do not fit a sixteenth of the free memory, a few rows are marked at a time.
constexpr int64_t ROWS_BYTES = (int64_t)3 << 30, ROWS_SMALL = (int64_t)256 << 20;

// lean: as little temporary memory as the steps can do with (three bitmap rows, one byte map, work items ordered chunk by chunk),
// where the memory for all chunks at once was refused; the graph is the same.
int partition_impl(ht_ctx* ctx, int64_t V, int64_t E, const int32_t* src_in, const int32_t* dst_in, int32_t n,
                   const ht_part_opts* opts, bool lean, ht_graph* g) {
  hipStream_t st = ctx->stream;
  const int self_loops = opts ? (opts->add_self_loops != 0) : 1;
  const int mode = opts ? opts->balance_mode : HT_BALANCE_EDGES;
  const int ptr_loc = opts ? opts->ptr_loc : HT_PTR_DEVICE;
  const int64_t Ep = E + (self_loops ? V : 0);
  // the per-edge kernels take one thread per stored edge, and a launch holds fewer than 2^32 threads; entry positions are 32-bit
  if (Ep >= ((int64_t)1 << 32) - 4096)
    return ht_set_err(ctx, HT_EINVAL, "ht_partition: %lld stored edges; fewer than 2^32 are supported", (long long)Ep);
  g->ctx = ctx;
  g->V = V;
  g->Ep = Ep;
  g->n = n;
  g->add_self_loops = self_loops;
  const size_t n1 = (size_t)n + 1;
  const int bitsV = bits_for(V);
  const int64_t nwp = bm_words(V), T = nwp / TB;   // words and tiles of a bitmap row
  const int64_t etiles = ceil_div64(std::max<int64_t>(Ep, 1), ETILE);
  const ItemSwitches sw;
  const int seg_fwd = sw.seg_fwd, seg_bwd = sw.seg_bwd;

  // pinned host memory for what is read back (a flag and a few counts, then lists of n + 1 offsets) and for the chunk order
  int64_t* hp = nullptr;
  {
    void* p = nullptr;
    HT_TRY(ht_host_scratch(ctx, HT_HS_READBACK, (8 + 9 * n1) * 8, &p));
    hp = (int64_t*)p;
  }
  int64_t* hl = hp + 8;

  // ---- edge list on the device
  DevArr<int32_t> src_copy, dst_copy;
  const int32_t* src = src_in;
  const int32_t* dst = dst_in;
  if (ptr_loc == HT_PTR_HOST && E > 0) {
    HT_TRY(src_copy.alloc(ctx, E));
    HT_TRY(dst_copy.alloc(ctx, E));
    HT_HIP(ctx, hipMemcpyAsync(src_copy.p, src_in, E * 4, hipMemcpyHostToDevice, st));
    HT_HIP(ctx, hipMemcpyAsync(dst_copy.p, dst_in, E * 4, hipMemcpyHostToDevice, st));
    src = src_copy.p;
    dst = dst_copy.p;
  }

  // ---- temporaries of the whole call, one allocation
  bool by_chunk = lean;
  {
    const int64_t need = (int64_t)n * nwp * 12;
    if (need > ROWS_BYTES) by_chunk = true;
    else if (need > ROWS_SMALL) {
      size_t free_b = 0, total_b = 0;
      HT_HIP(ctx, hipMemGetInfo(&free_b, &total_b));
      if (need > (int64_t)(free_b / 16)) by_chunk = true;
    }
    if (const char* v = getenv("HT_PART_BY_CHUNK")) by_chunk = by_chunk || atoi(v) != 0;   // for tests
  }
  const int64_t grp = by_chunk ? 1 : mark_group(nwp, n);
  const int64_t nrow = by_chunk ? 3 : n, nlist = by_chunk ? 1 : n;   // bitmap rows held; positions listed at once
  const size_t nkeys = (size_t)std::max<int64_t>(std::max(Ep, item_bound(V, Ep, std::min(seg_fwd, seg_bwd))), 1) + 64;
  DevBlock tmp;
  DevArr<uint64_t> keysA, keysB, allbm;
  DevArr<int32_t> ucount, tile_cnt, list_cnt, d_order;
  DevArr<int64_t> ubase, tbase, lbase, lists;   // lists: see L_* below
  DevArr<uint8_t> seen;
  DevArr<uint32_t> wpref;
  enum { L_FLAG, L_BOUNDS, L_EOFF, L_UEOFF, L_NOFF, L_REUSE, L_LOAD, L_LEAVE, L_COUNT };
  tmp.add<uint64_t>(nkeys);
  tmp.add<uint64_t>(nkeys);
  tmp.add<uint64_t>((size_t)nrow * nwp);
  tmp.add<int32_t>((size_t)etiles);
  tmp.add<int32_t>((size_t)nlist * T);
  tmp.add<int32_t>((size_t)3 * nlist * T);
  tmp.add<int32_t>((size_t)n);
  tmp.add<int64_t>((size_t)etiles + 1);
  tmp.add<int64_t>((size_t)nlist * T + 1);
  tmp.add<int64_t>((size_t)3 * nlist * T + 1);
  tmp.add<int64_t>(n1 * L_COUNT);
  tmp.add<uint8_t>((size_t)grp * nwp * 64);
  tmp.add<uint32_t>((size_t)nlist * nwp);
  HT_TRY(tmp.alloc(ctx));
  tmp.take(keysA, nkeys);
  tmp.take(keysB, nkeys);
  tmp.take(allbm, (size_t)nrow * nwp);
  tmp.take(ucount, (size_t)etiles);
  tmp.take(tile_cnt, (size_t)nlist * T);
  tmp.take(list_cnt, (size_t)3 * nlist * T);
  tmp.take(d_order, (size_t)n);
  tmp.take(ubase, (size_t)etiles + 1);
  tmp.take(tbase, (size_t)nlist * T + 1);
  tmp.take(lbase, (size_t)3 * nlist * T + 1);
  tmp.take(lists, n1 * L_COUNT);
  tmp.take(seen, (size_t)grp * nwp * 64);
  tmp.take(wpref, (size_t)nlist * nwp);
  auto list = [&](int which) { return lists.p + (size_t)which * n1; };
  HT_TRY(ht_fill_zero(ctx, st, list(L_FLAG), 8));
  HT_TRY(ht_fill_zero(ctx, st, seen.p, seen.bytes()));

  // ---- CSC by (destination, source), chunk boundaries
  {
    DevBlock& b = g->blk_csc;
    b.add<int64_t>((size_t)V + 1);
    b.add<int32_t>((size_t)std::max<int64_t>(Ep, 1));
    b.add<float>((size_t)V);
    HT_TRY(b.alloc(ctx));
    b.take(g->indptr, (size_t)V + 1);
    b.take(g->col, (size_t)std::max<int64_t>(Ep, 1));
    b.take(g->s, (size_t)V);
  }
  uint64_t* csc = keysA.p;
  if (Ep > 0) {
    HT_TRY(ht_radix_sort_edges(ctx, EdgeKeys{src, dst, E, V, bitsV, list(L_FLAG)}, keysA.p, keysB.p, Ep, &csc));
    k_csc<<<(unsigned)etiles, TB, 0, st>>>(csc, Ep, bitsV, V, g->col.p, g->indptr.p, ucount.p);
    HT_LAUNCH_CHECK(ctx);
    HT_TRY(ht_scan_i32(ctx, ucount.p, ubase.p, etiles, true));
  } else {
    HT_TRY(ht_fill_zero(ctx, st, g->indptr.p, (size_t)(V + 1) * 8));
    HT_TRY(ht_fill_zero(ctx, st, ubase.p, (size_t)(etiles + 1) * 8));
  }
  uint64_t* other = csc == keysA.p ? keysB.p : keysA.p;
  k_norm<<<nblk(V), TB, 0, st>>>(g->indptr.p, V, g->s.p);
  HT_LAUNCH_CHECK(ctx);
  k_bounds<<<nblk(n + 1), TB, 0, st>>>(g->indptr.p, V, Ep, n, mode, list(L_BOUNDS), list(L_EOFF));
  HT_LAUNCH_CHECK(ctx);
  HT_HIP(ctx, hipMemcpyAsync(&hp[0], list(L_FLAG), 8, hipMemcpyDeviceToHost, st));
  HT_HIP(ctx, hipMemcpyAsync(&hp[1], ubase.p + etiles, 8, hipMemcpyDeviceToHost, st));
  HT_HIP(ctx, hipMemcpyAsync(hl, list(L_BOUNDS), 2 * n1 * 8, hipMemcpyDeviceToHost, st));
  HT_HIP(ctx, hipStreamSynchronize(st));
  if (hp[0]) return ht_set_err(ctx, HT_EINVAL, "ht_partition: a vertex id is outside [0, V)");
  src_copy.release();
  dst_copy.release();
  g->bounds.assign(hl, hl + n1);
  const std::vector<int64_t> eoff(hl + n1, hl + 2 * n1);
  const int64_t nU = hp[1];

  // ---- duplicate edges: one entry per distinct (destination, source) pair when that pays.  Merged arrays cost 16 B per
  // distinct pair: worth it from about 5 % duplicates.
  const char* mg_env = getenv("HT_MERGE_DUPS");
  DevArr<uint32_t> upos;
  g->merged = !(mg_env && atoi(mg_env) == 0) && Ep > 0 && (double)nU <= 0.95 * (double)Ep;
  if (g->merged) {
    g->n_unique = nU;
    HT_TRY(upos.alloc(ctx, (size_t)nU + 1));
    DevBlock& b = g->blk_pairs;
    b.add<int64_t>((size_t)V + 1);
    for (int k = 0; k < 7; ++k) b.add<int32_t>((size_t)nU);
    HT_TRY(b.alloc(ctx));
    b.take(g->uindptr, (size_t)V + 1);
    b.take(g->ucol, (size_t)nU);
    b.take(g->ucol_slot, (size_t)nU);
    b.take(g->uw_fwd, (size_t)nU);
    b.take(g->umult, (size_t)nU);
    b.take(g->usdst, (size_t)nU);
    b.take(g->uw_bwd, (size_t)nU);
    b.take(g->umult_bwd, (size_t)nU);
    k_runs_fwd<<<(unsigned)etiles, TB, 0, st>>>(csc, Ep, bitsV, V, ubase.p, nU, upos.p, g->uindptr.p);
    HT_LAUNCH_CHECK(ctx);
    k_merge_fwd<<<nblk(nU), TB, 0, st>>>(upos.p, nU, g->col.p, g->s.p, g->ucol.p, g->uw_fwd.p, g->umult.p);
    HT_LAUNCH_CHECK(ctx);
    k_gather_i64<<<nblk((int64_t)n1), TB, 0, st>>>(g->uindptr.p, list(L_BOUNDS), (int64_t)n1, list(L_UEOFF));
    HT_LAUNCH_CHECK(ctx);
  }

  // ---- neighbour sets of the chunks as bitmaps (bit u of row k: u is in N_k; k = chunk id in vertex order)
  if (!by_chunk) {
    HT_TRY(mark_chunks(ctx, st, g->col.p, eoff.data(), list(L_EOFF), n, nwp, grp, seen.p, allbm.p, tile_cnt.p));
    HT_TRY(ht_scan_i32(ctx, tile_cnt.p, tbase.p, (int64_t)n * T, true));
    k_gather_stride<<<nblk((int64_t)n1), TB, 0, st>>>(tbase.p, T, (int64_t)n1, list(L_NOFF));
    HT_LAUNCH_CHECK(ctx);
  }
  // chunk by chunk: the row of schedule position j, marked into one of three
  auto mark_row = [&](int j, int32_t* cnt) -> int {
    return mark_chunk(ctx, st, g->col.p, eoff.data(), list(L_EOFF), n, g->order[j], nwp, seen.p, allbm.p + (j % 3) * nwp, cnt);
  };
  auto row_of = [&](int j) { return allbm.p + (size_t)(by_chunk ? j % 3 : g->order[j]) * nwp; };

  // a buffer with room for every distinct source is the schedule-aware buffer at that size
  const bool keep_all = opts && opts->cache_rows == -1;
  const bool far_first = (opts && opts->cache_policy == HT_CACHE_FARTHEST) || keep_all;

  // ---- chunk reorganisation (Alg. 4, phase 2; one GPU, so a batch is one chunk): the first chunk
  // stays first, then the unplaced chunk whose neighbour set overlaps most with the chunk placed last
  // comes next (ties: smallest id).
  g->order.resize(n);
  for (int j = 0; j < n; ++j) g->order[j] = j;
  if (opts && opts->reorder_chunks && n > 2) {
    DevArr<unsigned long long> ov;
    HT_TRY(ov.alloc(ctx, n));
    DevArr<uint64_t> rows_tmp;      // (the greedy steps compare every chunk with every other)
    const uint64_t* bms = allbm.p;
    if (by_chunk) {
      DevArr<int32_t> cnt_tmp;
      HT_TRY(rows_tmp.alloc(ctx, (size_t)n * nwp));
      HT_TRY(cnt_tmp.alloc(ctx, (size_t)n * T));
      HT_TRY(mark_chunks(ctx, st, g->col.p, eoff.data(), list(L_EOFF), n, nwp, grp, seen.p, rows_tmp.p, cnt_tmp.p));
      HT_HIP(ctx, hipStreamSynchronize(st));
      bms = rows_tmp.p;
    }
    std::vector<unsigned long long> hov(n);
    std::vector<char> placed(n, 0);
    placed[0] = 1;
    const unsigned gx = (unsigned)std::min<int64_t>(T, 64);
    for (int j = 1; j < n; ++j) {
      HT_TRY(ht_fill_zero(ctx, st, ov.p, (size_t)n * 8));
      k_overlap<<<dim3(gx, n), TB, 0, st>>>(bms, nwp, bms + (size_t)g->order[j - 1] * nwp, ov.p);
      HT_LAUNCH_CHECK(ctx);
      HT_HIP(ctx, hipMemcpyAsync(hov.data(), ov.p, (size_t)n * 8, hipMemcpyDeviceToHost, st));
      HT_HIP(ctx, hipStreamSynchronize(st));
      int best = -1;
      for (int k = 0; k < n; ++k)
        if (!placed[k] && (best < 0 || hov[k] > hov[best])) best = k;
      g->order[j] = best;
      placed[best] = 1;
    }
  }
  std::copy(g->order.begin(), g->order.end(), (int32_t*)(hl + 8 * n1));
  HT_HIP(ctx, hipMemcpyAsync(d_order.p, hl + 8 * n1, (size_t)n * 4, hipMemcpyHostToDevice, st));

  // ---- reuse / load / leave lists: counted here for the adjacent rule; the schedule-aware buffer is simulated first
  ListRows rows{allbm.p, by_chunk ? nullptr : d_order.p, nullptr, nullptr, nwp, n, 0, (int32_t)nlist};
  auto count_lists = [&]() -> int {
    HT_TRY(ht_in_launches((int64_t)rows.nj * T, TILE_LAUNCH, [&](int64_t t, int64_t m) {
      k_list_counts<<<(unsigned)m, TB, 0, st>>>(rows, T, list_cnt.p, t);
      HT_LAUNCH_CHECK(ctx);
      return (int)HT_OK;
    }));
    return ht_scan_i32(ctx, list_cnt.p, lbase.p, (int64_t)3 * rows.nj * T, true);
  };
  auto list_starts = [&]() -> int {
    for (int w = 0; w < 3; ++w) {
      k_gather_stride<<<nblk((int64_t)n1), TB, 0, st>>>(lbase.p + (int64_t)w * n * T, T, (int64_t)n1, list(L_REUSE + w));
      HT_LAUNCH_CHECK(ctx);
    }
    return HT_OK;
  };
  auto expand_lists = [&](int32_t* reuse, int32_t* load, int32_t* leave) -> int {
    return ht_in_launches((int64_t)rows.nj * T, TILE_LAUNCH, [&](int64_t t, int64_t m) {
      k_list_expand<<<(unsigned)m, TB, 0, st>>>(rows, T, lbase.p, reuse, load, leave, t);
      HT_LAUNCH_CHECK(ctx);
      return (int)HT_OK;
    });
  };
  std::vector<int64_t> ueoff, noff;
  std::vector<int64_t> offs[3];   // starts of every schedule position's reuse / load / leave list
  int64_t n_distinct = 0;         // |N_0 u ... u N_{n-1}| (schedule-aware buffer)
  if (!by_chunk) {
    DevArr<unsigned long long> distinct;
    if (far_first) {
      HT_TRY(distinct.alloc(ctx, 1));
      HT_TRY(ht_fill_zero(ctx, st, distinct.p, 8));
      k_popc_all<<<popc_grid(nwp), TB, 0, st>>>(allbm.p, nwp, n, distinct.p);
      HT_LAUNCH_CHECK(ctx);
      HT_HIP(ctx, hipMemcpyAsync(&hp[2], distinct.p, 8, hipMemcpyDeviceToHost, st));
    }
    // (the adjacent rule's loads are also V_+ru, which every schedule reports)
    HT_TRY(count_lists());
    HT_TRY(list_starts());
    HT_HIP(ctx, hipMemcpyAsync(hl, list(L_UEOFF), (size_t)(L_COUNT - L_UEOFF) * n1 * 8, hipMemcpyDeviceToHost, st));
    HT_HIP(ctx, hipStreamSynchronize(st));
    ueoff.assign(hl, hl + n1);
    noff.assign(hl + n1, hl + 2 * n1);
    if (far_first) n_distinct = hp[2];
  } else {
    DevArr<int64_t> counts;   // |N|, reuse, load, leave of every position
    DevArr<uint64_t> all;     // N_0 u N_1 u ...
    DevArr<unsigned long long> distinct;
    HT_TRY(counts.alloc(ctx, (size_t)4 * n));
    if (far_first) {
      HT_TRY(all.alloc(ctx, (size_t)nwp));
      HT_TRY(distinct.alloc(ctx, 1));
      HT_TRY(ht_fill_zero(ctx, st, all.p, all.bytes()));
      HT_TRY(ht_fill_zero(ctx, st, distinct.p, 8));
    }
    for (int j = 0; j < n; ++j) {
      if (j == 0) HT_TRY(mark_row(0, tile_cnt.p));
      HT_TRY(ht_scan_i32(ctx, tile_cnt.p, tbase.p, T, true));       // (tile_cnt: row j's)
      if (j + 1 < n) HT_TRY(mark_row(j + 1, tile_cnt.p));
      rows.j0 = j;
      HT_TRY(count_lists());
      k_put_counts<<<1, 64, 0, st>>>(tbase.p, lbase.p, T, counts.p + 4 * j);
      HT_LAUNCH_CHECK(ctx);
      if (far_first) {
        k_bm_or<<<nblk(nwp), TB, 0, st>>>(all.p, row_of(j), nwp);
        HT_LAUNCH_CHECK(ctx);
      }
    }
    if (far_first) {
      k_popc_all<<<popc_grid(nwp), TB, 0, st>>>(all.p, nwp, 1, distinct.p);
      HT_LAUNCH_CHECK(ctx);
      HT_HIP(ctx, hipMemcpyAsync(&hp[2], distinct.p, 8, hipMemcpyDeviceToHost, st));
    }
    std::vector<int64_t> h4((size_t)4 * n);
    HT_HIP(ctx, hipMemcpyAsync(h4.data(), counts.p, (size_t)4 * n * 8, hipMemcpyDeviceToHost, st));
    HT_HIP(ctx, hipMemcpyAsync(hl, list(L_UEOFF), n1 * 8, hipMemcpyDeviceToHost, st));
    HT_HIP(ctx, hipStreamSynchronize(st));
    ueoff.assign(hl, hl + n1);
    noff.assign(n1, 0);
    for (int j = 0; j < n; ++j) noff[g->order[j] + 1] = h4[(size_t)4 * j];
    for (int k = 0; k < n; ++k) noff[k + 1] += noff[k];
    for (int w = 0; w < 3; ++w) {
      offs[w].assign(n1, 0);
      for (int j = 0; j < n; ++j) offs[w][j + 1] = offs[w][j] + h4[(size_t)4 * j + 1 + w];
    }
    std::copy(noff.begin(), noff.end(), hl);
    HT_HIP(ctx, hipMemcpyAsync(list(L_NOFF), hl, n1 * 8, hipMemcpyHostToDevice, st));
    HT_HIP(ctx, hipStreamSynchronize(st));
    if (far_first) n_distinct = hp[2];
  }
  auto take_offsets = [&](const int64_t* h) {
    for (int w = 0; w < 3; ++w) {
      offs[w].assign(h + (size_t)w * n1, h + (size_t)(w + 1) * n1);
      const int64_t b0 = offs[w][0];
      for (int64_t& x : offs[w]) x -= b0;
    }
  };
  if (!by_chunk) take_offsets(hl + (size_t)(L_REUSE - L_UEOFF) * n1);
  g->v_ori = noff[n];
  g->v_ru = offs[1][n];
  g->pos.resize(n);
  for (int j = 0; j < n; ++j) g->pos[g->order[j]] = j;
  g->chunks.clear();
  g->chunks.resize(n);
  for (int j = 0; j < n; ++j) {
    ChunkMeta& c = g->chunks[j];
    const int k = g->order[j];
    c.id = k;
    c.dst0 = g->bounds[k];
    c.dst1 = g->bounds[k + 1];
    c.e0 = eoff[k];
    c.nnz = eoff[k + 1] - eoff[k];
    c.ue0 = g->merged ? ueoff[k] : c.e0;
    c.nu = g->merged ? ueoff[k + 1] - ueoff[k] : c.nnz;
    c.nbr_off = noff[k];
    c.nsrc = noff[k + 1] - noff[k];
    c.sptr_off = noff[k] + k;
    g->max_ndst = std::max(g->max_ndst, c.dst1 - c.dst0);
    g->max_nnz = std::max(g->max_nnz, c.nnz);
    g->max_nsrc = std::max(g->max_nsrc, c.nsrc);
  }
  for (int j = 0; j < n;) {
    int k = j;
    while (k + 1 < n && g->chunks[k + 1].dst1 > g->chunks[k + 1].dst0 && g->chunks[k + 1].dst0 == g->chunks[k].dst1 &&
           g->chunks[k].dst1 - g->chunks[j].dst0 < HT_DENSE_MERGE_ROWS && g->chunks[j].dst1 > g->chunks[j].dst0)
      ++k;
    if (g->chunks[k].dst1 > g->chunks[j].dst0) {
      g->dense_groups.push_back(g->chunks[j].dst0);
      g->dense_groups.push_back(g->chunks[k].dst1);
    }
    j = k + 1;
  }
  int64_t C = opts ? opts->cache_rows : 0;
  if (keep_all) C = n_distinct;
  if (C <= 0) C = g->max_nsrc;
  if (C < g->max_nsrc)
    return ht_set_err(ctx, HT_EINVAL, "ht_partition: cache_rows %lld < max_j |N_j| = %lld", (long long)C,
                      (long long)g->max_nsrc);
  const size_t vo = (size_t)std::max<int64_t>(g->v_ori, 1);
  HT_TRY(g->nbr.alloc(ctx, vo));
  if (!by_chunk)
    HT_TRY(ht_in_launches((int64_t)n * T, TILE_LAUNCH, [&](int64_t t, int64_t m) {
      k_expand_rows<<<(unsigned)m, TB, 0, st>>>(allbm.p, nwp, tbase.p, wpref.p, g->nbr.p, t, 0);
      HT_LAUNCH_CHECK(ctx);
      return (int)HT_OK;
    }));
  // chunk by chunk: row j's word prefixes and its list, from its tile counts
  auto expand_row = [&](int j) -> int {
    HT_TRY(ht_scan_i32(ctx, tile_cnt.p, tbase.p, T, true));
    k_expand_rows<<<(unsigned)T, TB, 0, st>>>(row_of(j), nwp, tbase.p, wpref.p, g->nbr.p, 0, noff[g->order[j]]);
    HT_LAUNCH_CHECK(ctx);
    return HT_OK;
  };

  // ---- schedule of a buffer that knows the future: a row leaves after its last use, or for room with the farthest next
  // use first.  Simulated chunk by chunk on bitmaps; kept for the lists: the rows resident before every chunk (Pbm), the
  // rows released before it (Ebm row j; row n: what is still resident at the end).
  DevArr<uint64_t> Pbm, Ebm;
  if (far_first) {
    DevBlock fb;
    DevArr<int32_t> nxt, last, nu, cnt1;
    DevArr<unsigned int> hist;
    DevArr<unsigned long long> tot2;
    DevArr<int64_t> pref1;
    DevArr<uint64_t> eqbm, bmT, bmR;
    fb.add<int32_t>(vo); fb.add<int32_t>((size_t)V); fb.add<int32_t>((size_t)V); fb.add<int32_t>((size_t)nwp);
    fb.add<unsigned int>(n1); fb.add<unsigned long long>((size_t)n + 2); fb.add<int64_t>((size_t)nwp + 1);
    for (int k = 0; k < 3; ++k) fb.add<uint64_t>((size_t)nwp);
    HT_TRY(fb.alloc(ctx));
    fb.take(nxt, vo); fb.take(last, (size_t)V); fb.take(nu, (size_t)V); fb.take(cnt1, (size_t)nwp);
    fb.take(hist, n1); fb.take(tot2, (size_t)n + 2); fb.take(pref1, (size_t)nwp + 1);
    fb.take(eqbm, (size_t)nwp); fb.take(bmT, (size_t)nwp); fb.take(bmR, (size_t)nwp);
    unsigned long long* dead_cnt = tot2.p + 2;
    HT_TRY(Pbm.alloc(ctx, (size_t)nlist * nwp));
    HT_TRY(Ebm.alloc(ctx, n1 * (size_t)nwp));
    HT_TRY(ht_fill_zero(ctx, st, dead_cnt, (size_t)n * 8));
    HT_TRY(ht_fill_zero(ctx, st, Ebm.p, Ebm.bytes()));
    HT_TRY(ht_fill_zero(ctx, st, bmR.p, bmR.bytes()));
    k_fill_i32<<<nblk(V), TB, 0, st>>>(last.p, V, n);
    HT_LAUNCH_CHECK(ctx);
    k_fill_i32<<<nblk(V), TB, 0, st>>>(nu.p, V, n);
    HT_LAUNCH_CHECK(ctx);
    // next uses, last chunk first
    for (int j = n - 1; j >= 0; --j) {
      const ChunkMeta& c = g->chunks[j];
      if (by_chunk) {
        HT_TRY(mark_row(j, tile_cnt.p));
        HT_TRY(expand_row(j));
      }
      if (c.nsrc > 0) {
        k_next_use<<<nblk(c.nsrc), TB, 0, st>>>(g->nbr.p + c.nbr_off, c.nsrc, last.p, j, nxt.p + c.nbr_off);
        HT_LAUNCH_CHECK(ctx);
      }
    }
    // forward simulation: bmR = resident rows
    std::vector<unsigned int> hh(n1);
    std::vector<int64_t> n_reuse((size_t)n), n_leave((size_t)n, 0);
    for (int j = 0; j < n; ++j) {
      const ChunkMeta& c = g->chunks[j];
      const uint64_t* bmj = row_of(j);   // N_j
      if (by_chunk) HT_TRY(mark_row(j, tile_cnt.p));
      HT_TRY(ht_fill_zero(ctx, st, tot2.p, 16));
      k_popc_union<<<popc_grid(nwp), TB, 0, st>>>(bmR.p, bmj, nwp, tot2.p);
      HT_LAUNCH_CHECK(ctx);
      unsigned long long t2[2];
      HT_HIP(ctx, hipMemcpyAsync(t2, tot2.p, 16, hipMemcpyDeviceToHost, st));
      HT_HIP(ctx, hipStreamSynchronize(st));
      const int64_t over = (int64_t)t2[0] - C;
      n_reuse[j] = (int64_t)t2[1];
      if (over > 0) {
        n_leave[j - 1] += over;     // j > 0 here: nothing is resident before the first chunk
        uint64_t* Ej = Ebm.p + (size_t)j * nwp;
        k_bm_minus<<<nblk(nwp), TB, 0, st>>>(bmR.p, bmj, nwp, bmT.p);   // candidates: resident, not needed now
        HT_LAUNCH_CHECK(ctx);
        HT_TRY(ht_fill_zero(ctx, st, hist.p, n1 * 4));
        k_hist_nu<<<(unsigned)std::min<int64_t>(nblk(nwp), 2048), TB, 0, st>>>(bmT.p, nwp, nu.p, n + 1, hist.p);
        HT_LAUNCH_CHECK(ctx);
        HT_HIP(ctx, hipMemcpyAsync(hh.data(), hist.p, n1 * 4, hipMemcpyDeviceToHost, st));
        HT_HIP(ctx, hipStreamSynchronize(st));
        int32_t t = n;
        int64_t cum = 0, m = 0;
        for (; t >= 0; --t) {
          if (cum + (int64_t)hh[t] >= over) {
            m = over - cum;
            break;
          }
          cum += hh[t];
        }
        if (t < 0) return ht_set_err(ctx, HT_ESTATE, "ht_partition: buffer schedule ran out of rows to release");
        k_select_nu<<<nblk(nwp), TB, 0, st>>>(bmT.p, nwp, nu.p, t, Ej, eqbm.p);
        HT_LAUNCH_CHECK(ctx);
        HT_TRY(ht_bitmap_prefix(ctx, eqbm.p, nwp, cnt1.p, pref1.p));
        k_take_first<<<nblk(nwp), TB, 0, st>>>(eqbm.p, pref1.p, nwp, m, Ej);
        HT_LAUNCH_CHECK(ctx);
        k_bm_minus<<<nblk(nwp), TB, 0, st>>>(bmR.p, Ej, nwp, bmR.p);
        HT_LAUNCH_CHECK(ctx);
      }
      if (!by_chunk) HT_HIP(ctx, hipMemcpyAsync(Pbm.p + (size_t)j * nwp, bmR.p, (size_t)nwp * 8, hipMemcpyDeviceToDevice, st));
      k_bm_or<<<nblk(nwp), TB, 0, st>>>(bmR.p, bmj, nwp);
      HT_LAUNCH_CHECK(ctx);
      if (c.nsrc > 0) {
        k_set_nu<<<nblk(c.nsrc), TB, 0, st>>>(g->nbr.p + c.nbr_off, c.nsrc, nxt.p + c.nbr_off, nu.p);
        HT_LAUNCH_CHECK(ctx);
        if (j + 1 < n) {   // rows that no later chunk needs leave now (after the last chunk everything does)
          uint64_t* E1 = Ebm.p + (size_t)(j + 1) * nwp;
          k_mark_dead<<<nblk(c.nsrc), TB, 0, st>>>(g->nbr.p + c.nbr_off, c.nsrc, nxt.p + c.nbr_off, n, (uint32_t*)E1,
                                                   dead_cnt + j);
          HT_LAUNCH_CHECK(ctx);
          k_bm_minus<<<nblk(nwp), TB, 0, st>>>(bmR.p, E1, nwp, bmR.p);
          HT_LAUNCH_CHECK(ctx);
        }
      }
    }
    HT_HIP(ctx, hipMemcpyAsync(Ebm.p + (size_t)n * nwp, bmR.p, (size_t)nwp * 8, hipMemcpyDeviceToDevice, st));
    rows.pbm = Pbm.p;
    rows.ebm = Ebm.p;
    if (!by_chunk) {
      HT_TRY(count_lists());
      HT_TRY(list_starts());
      HT_HIP(ctx, hipMemcpyAsync(hl, list(L_REUSE), 3 * n1 * 8, hipMemcpyDeviceToHost, st));
      HT_HIP(ctx, hipStreamSynchronize(st));
      take_offsets(hl);
    } else {   // counted on the way
      HT_TRY(ht_fill_zero(ctx, st, tot2.p, 16));
      k_popc_union<<<popc_grid(nwp), TB, 0, st>>>(bmR.p, bmR.p, nwp, tot2.p);
      HT_LAUNCH_CHECK(ctx);
      std::vector<unsigned long long> dead((size_t)n + 2);
      HT_HIP(ctx, hipMemcpyAsync(dead.data(), tot2.p, dead.size() * 8, hipMemcpyDeviceToHost, st));
      HT_HIP(ctx, hipStreamSynchronize(st));
      for (int j = 0; j + 1 < n; ++j) n_leave[j] += (int64_t)dead[j + 2];
      n_leave[n - 1] = (int64_t)dead[0];      // what is still resident leaves at the end of a pass
      for (int j = 0; j < n; ++j) {
        offs[0][j + 1] = offs[0][j] + n_reuse[j];
        offs[1][j + 1] = offs[1][j] + g->chunks[j].nsrc - n_reuse[j];
        offs[2][j + 1] = offs[2][j] + n_leave[j];
      }
    }
  }
  g->v_load = offs[1][n];
  for (int j = 0; j < n; ++j) {
    ChunkMeta& c = g->chunks[j];
    c.reuse_off = offs[0][j];
    c.load_off = offs[1][j];
    c.leave_off = offs[2][j];
    c.n_reuse = offs[0][j + 1] - c.reuse_off;
    c.n_load = offs[1][j + 1] - c.load_off;
    c.n_leave = offs[2][j + 1] - c.leave_off;
  }
  if (C < 1) C = 1;
  g->cache_rows = C;
  g->cache_policy = far_first ? HT_CACHE_FARTHEST : HT_CACHE_ADJACENT;
  g->single_leave = far_first && g->v_load == n_distinct;

  // ---- arenas
  const size_t vr = (size_t)std::max<int64_t>(g->v_load, 1);
  const size_t ep = (size_t)std::max<int64_t>(Ep, 1);
  const size_t n_reused = (size_t)std::max<int64_t>(g->v_ori - g->v_load, 1);
  const int64_t n_ent = g->merged ? nU : Ep;
  const int64_t fb_items = item_bound(V, n_ent, seg_fwd), bb_items = item_bound(g->v_ori, n_ent, seg_bwd);
  {
    DevBlock& b = g->blk_chunks;
    b.add<int32_t>(vo); b.add<int32_t>(vo); b.add<int64_t>(vo + n); b.add<int32_t>(n_reused);
    for (int k = 0; k < 4; ++k) b.add<int32_t>(vr);
    for (int k = 0; k < 3; ++k) b.add<int32_t>(ep);
    if (g->merged) b.add<int64_t>(vo + n);
    b.add<int64_t>(g->dense_groups.size());
    b.add<WorkItem>((size_t)fb_items); b.add<CutRow>((size_t)cut_bound(n_ent, seg_fwd));
    b.add<WorkItem>((size_t)bb_items); b.add<CutRow>((size_t)cut_bound(n_ent, seg_bwd));
    HT_TRY(b.alloc(ctx));
    b.take(g->slot, vo);
    b.take(g->gslot, vo);
    b.take(g->sptr, vo + n);
    b.take(g->reuse, n_reused);
    b.take(g->load, vr);
    b.take(g->load_slot, vr);
    b.take(g->leave, vr);
    b.take(g->leave_slot, vr);
    b.take(g->col_local, ep);
    b.take(g->col_slot, ep);
    b.take(g->sdst, ep);
    if (g->merged) b.take(g->usptr, vo + n);
    b.take(g->d_dense_groups, g->dense_groups.size());
    b.take(g->fwd_items.items, (size_t)fb_items);
    b.take(g->fwd_items.cuts, (size_t)cut_bound(n_ent, seg_fwd));
    b.take(g->bwd_items.items, (size_t)bb_items);
    b.take(g->bwd_items.cuts, (size_t)cut_bound(n_ent, seg_bwd));
  }
  const int64_t nwC = ceil_div64(C, 64), tC = ceil_div64(nwC, TB);
  ItemBuild ib[2];
  ib[0].nrows = V;
  ib[0].seg = seg_fwd;
  ib[0].rows = RowSet{g->merged ? g->uindptr.p : g->indptr.p, list(L_BOUNDS), nullptr, n};
  ib[0].idx = g->merged ? g->ucol.p : g->col.p;   // forward items are ordered by buffer-independent source id
  ib[0].range = V;
  ib[0].out = &g->fwd_items;
  ib[1].nrows = g->v_ori;
  ib[1].seg = seg_bwd;
  ib[1].rows = RowSet{g->merged ? g->usptr.p : g->sptr.p, list(L_NOFF), list(g->merged ? L_UEOFF : L_EOFF), n};
  ib[1].idx = g->merged ? g->usdst.p : g->sdst.p;   // backward items by local destination
  ib[1].range = g->max_ndst;
  ib[1].out = &g->bwd_items;
  ib[0].h_first = g->bounds.data();
  ib[1].h_first = noff.data();
  int64_t n_made = std::max(fb_items, bb_items);     // items put in order at once
  if (lean) {
    n_made = 1;
    for (const ChunkMeta& c : g->chunks)
      n_made = std::max(n_made, std::max(item_bound(c.dst1 - c.dst0, c.nu, seg_fwd), item_bound(c.nsrc, c.nu, seg_bwd)));
  }
  DevBlock tmp2;
  DevArr<int32_t> vslot, free_cnt, icnt[2];
  DevArr<uint64_t> freebm;
  DevArr<int64_t> ibase[2], istarts;
  DevArr<WorkItem> made;
  for (ItemBuild& b : ib) b.tiles = ceil_div64(b.nrows, RTILE);
  tmp2.add<int32_t>((size_t)V);
  tmp2.add<int32_t>((size_t)tC);
  tmp2.add<uint64_t>((size_t)2 * nwC);
  for (const ItemBuild& b : ib) { tmp2.add<int32_t>((size_t)3 * b.tiles); tmp2.add<int64_t>((size_t)3 * b.tiles + 1); }
  tmp2.add<int64_t>(6 * n1);
  tmp2.add<WorkItem>((size_t)n_made);
  HT_TRY(tmp2.alloc(ctx));
  tmp2.take(vslot, (size_t)V);
  tmp2.take(free_cnt, (size_t)tC);
  tmp2.take(freebm, (size_t)2 * nwC);
  for (int d = 0; d < 2; ++d) {
    tmp2.take(icnt[d], (size_t)3 * ib[d].tiles);
    tmp2.take(ibase[d], (size_t)3 * ib[d].tiles + 1);
    ib[d].cnt = icnt[d].p;
    ib[d].base = ibase[d].p;
  }
  tmp2.take(istarts, 6 * n1);
  tmp2.take(made, (size_t)n_made);
  ib[0].starts = istarts.p;
  ib[1].starts = istarts.p + 3 * n1;

  HT_HIP(ctx, hipMemcpyAsync(g->d_dense_groups.p, g->dense_groups.data(), g->dense_groups.size() * 8, hipMemcpyHostToDevice, st));

  // ---- the lists, then the buffer positions, chunk by chunk
  uint64_t* free_now = freebm.p;
  uint64_t* free_next = freebm.p + nwC;
  k_free_init<<<nblk(nwC), TB, 0, st>>>(free_now, nwC, C);
  HT_LAUNCH_CHECK(ctx);
  auto positions = [&](int j) -> int {
    const ChunkMeta& c = g->chunks[j];
    if (c.n_load > 0) {
      const bool counted = nwC > 16 * TB;   // few words: every block adds up those before it by itself
      if (counted) {
        k_free_count<<<(unsigned)tC, TB, 0, st>>>(free_now, nwC, free_cnt.p);
        HT_LAUNCH_CHECK(ctx);
      }
      k_assign<<<(unsigned)tC, TB, 0, st>>>(free_now, free_next, nwC, counted ? free_cnt.p : nullptr, g->load.p + c.load_off,
                                            c.n_load, vslot.p, g->load_slot.p + c.load_off);
      HT_LAUNCH_CHECK(ctx);
      std::swap(free_now, free_next);
    }
    if (c.nsrc + c.n_leave > 0) {
      const uint64_t* prev = far_first ? Pbm.p + (size_t)(by_chunk ? 0 : j) * nwp : j > 0 ? row_of(j - 1) : nullptr;
      k_lookup_evict<<<nblk(c.nsrc + c.n_leave), TB, 0, st>>>(g->nbr.p + c.nbr_off, c.nsrc, vslot.p, prev, g->slot.p + c.nbr_off,
                                                             g->gslot.p + c.nbr_off, g->leave.p + c.leave_off, c.n_leave,
                                                             (uint32_t*)free_now, g->leave_slot.p + c.leave_off);
      HT_LAUNCH_CHECK(ctx);
    }
    return HT_OK;
  };
  // edges [e0, e1), the first of them of chunk k0, whose bitmap row is bm
  auto remap = [&](int64_t e0, int64_t e1, int k0, const uint64_t* bm) -> int {
    if (e1 <= e0) return HT_OK;
    k_remap<<<nblk(e1 - e0, ETILE), TB, 0, st>>>(csc, e0, e1, k0, bitsV, list(L_EOFF), list(L_BOUNDS), list(L_NOFF), n, bm, nwp, wpref.p,
                                                 g->slot.p, g->col_local.p, g->col_slot.p, other);
    HT_LAUNCH_CHECK(ctx);
    return HT_OK;
  };
  if (!by_chunk) {
    HT_TRY(expand_lists(g->reuse.p, g->load.p, g->leave.p));
    for (int j = 0; j < n; ++j) HT_TRY(positions(j));
    HT_TRY(remap(0, Ep, 0, allbm.p));
  } else {
    if (far_first) HT_TRY(ht_fill_zero(ctx, st, Pbm.p, Pbm.bytes()));
    for (int j = 0; j < n; ++j) {
      const ChunkMeta& c = g->chunks[j];
      if (j == 0 || far_first) HT_TRY(mark_row(j, tile_cnt.p));
      HT_TRY(expand_row(j));                                        // (tile_cnt: row j's)
      if (far_first) {   // Pbm: the rows resident before chunk j
        k_bm_minus<<<nblk(nwp), TB, 0, st>>>(Pbm.p, Ebm.p + (size_t)j * nwp, nwp, Pbm.p);
        HT_LAUNCH_CHECK(ctx);
      } else if (j + 1 < n) HT_TRY(mark_row(j + 1, tile_cnt.p));
      rows.j0 = j;
      HT_TRY(count_lists());
      HT_TRY(expand_lists(g->reuse.p + c.reuse_off, g->load.p + c.load_off, g->leave.p + c.leave_off));
      HT_TRY(positions(j));
      HT_TRY(remap(c.e0, c.e0 + c.nnz, c.id, row_of(j)));
      if (far_first) {
        k_bm_or<<<nblk(nwp), TB, 0, st>>>(Pbm.p, row_of(j), nwp);
        HT_LAUNCH_CHECK(ctx);
      }
    }
  }

  // ---- topology in local indices, the edges grouped by source
  k_sptr_ends<<<nblk(n), TB, 0, st>>>(list(L_NOFF), list(L_EOFF), n, g->sptr.p);
  HT_LAUNCH_CHECK(ctx);
  if (g->merged) {
    k_sptr_ends<<<nblk(n), TB, 0, st>>>(list(L_NOFF), list(L_UEOFF), n, g->usptr.p);
    HT_LAUNCH_CHECK(ctx);
  }
  if (Ep > 0) {
    if (g->merged) {   // buffer positions of the distinct forward pairs
      k_gather_i32<<<nblk(nU), TB, 0, st>>>(g->col_slot.p, upos.p, nU, g->ucol_slot.p);
      HT_LAUNCH_CHECK(ctx);
    }
    uint64_t* by_src = nullptr;
    HT_TRY(ht_radix_sort_u64(ctx, other, csc, Ep, 32, 32 + bits_for(g->v_ori), &by_src));
    k_by_source<<<(unsigned)etiles, TB, 0, st>>>(by_src, Ep, list(L_EOFF), n, g->sdst.p, g->sptr.p, g->merged ? ucount.p : nullptr);
    HT_LAUNCH_CHECK(ctx);
    if (g->merged) {
      HT_TRY(ht_scan_i32(ctx, ucount.p, ubase.p, etiles, true));
      k_runs_bwd<<<(unsigned)etiles, TB, 0, st>>>(by_src, Ep, ubase.p, nU, list(L_EOFF), list(L_UEOFF), n, upos.p, g->usptr.p);
      HT_LAUNCH_CHECK(ctx);
      k_merge_bwd<<<nblk(nU, ETILE), TB, 0, st>>>(upos.p, nU, by_src, list(L_UEOFF), list(L_BOUNDS), n, g->s.p, g->usdst.p,
                                                  g->uw_bwd.p, g->umult_bwd.p);
      HT_LAUNCH_CHECK(ctx);
    }
  }

  // ---- work items of both directions
  for (int d = 0; d < 2; ++d) HT_TRY(count_items(ctx, ib[d], hp + 3 * d));
  HT_HIP(ctx, hipStreamSynchronize(st));
  for (int d = 0; d < 2; ++d) HT_TRY(fill_items(ctx, ib[d], hp + 3 * d, made.p, (size_t)n_made, keysA.p, keysB.p, nkeys, sw.order, hl));
  HT_HIP(ctx, hipMemcpyAsync(hl, istarts.p, 6 * n1 * 8, hipMemcpyDeviceToHost, st));
  HT_HIP(ctx, hipStreamSynchronize(st));
  for (int d = 0; d < 2; ++d) {
    const int64_t tot[3] = {ib[d].out->n_items, ib[d].out->n_part, ib[d].out->n_cut};
    const std::vector<int64_t>& first = d == 0 ? g->bounds : noff;
    // start of chunk k's share (chunks that start behind the last row have none)
    auto at = [&](int w, int k) { return k < n && first[k] < ib[d].nrows ? hl[(size_t)(3 * d + w) * n1 + k] : tot[w]; };
    for (int j = 0; j < n; ++j) {
      ChunkMeta& c = g->chunks[j];
      ItemRange& r = d == 0 ? c.fwd : c.bwd;
      r.it0 = at(0, c.id);
      r.n_items = at(0, c.id + 1) - r.it0;
      r.part0 = at(1, c.id);
      r.n_part = at(1, c.id + 1) - r.part0;
      r.cut0 = at(2, c.id);
      r.n_cut = at(2, c.id + 1) - r.cut0;
      int64_t& mx = d == 0 ? g->max_fpart : g->max_bpart;
      mx = std::max(mx, r.n_part);
    }
  }
  return HT_OK;
}

template <typename T>
int d2h(ht_ctx* ctx, T* dst, const T* src, int64_t n) {
  if (!dst || n <= 0) return HT_OK;
  HT_HIP(ctx, hipMemcpy(dst, src, (size_t)n * sizeof(T), hipMemcpyDeviceToHost));
  return HT_OK;
}

}  // namespace

namespace {

// The list costs 4 or 8 bytes per entry; it is copied together from the chunks' by-source lists.
void plan_by_source(const ht_graph* g, DevBlock* kept, DevBlock* tmp) {
  const ItemSwitches sw;
  const int64_t V = g->V, n_ent = g->merged ? g->n_unique : g->Ep, bound = item_bound(V, n_ent, sw.seg_bwd);
  const size_t n1 = (size_t)g->n + 1, tiles = (size_t)ceil_div64(V, RTILE);
  kept->add<int32_t>((size_t)std::max<int64_t>(n_ent, 1));
  if (g->merged) kept->add<float>((size_t)n_ent);
  kept->add<WorkItem>((size_t)bound);
  kept->add<CutRow>((size_t)cut_bound(n_ent, sw.seg_bwd));
  kept->add<int64_t>((size_t)V + 1);
  tmp->add<int32_t>((size_t)V);
  tmp->add<int32_t>(3 * tiles);
  tmp->add<int64_t>((size_t)std::max<int64_t>(g->v_ori, 1));
  tmp->add<int64_t>(3 * n1 + 2);
  tmp->add<int64_t>(3 * tiles + 1);
  tmp->add<int64_t>(6);
  tmp->add<WorkItem>((size_t)bound);
  tmp->add<uint64_t>((size_t)bound);
  tmp->add<uint64_t>((size_t)bound);
}

// A destroyed graph's list memory is kept for the next graph up to this size.
constexpr size_t LIST_KEPT_BYTES = (size_t)1 << 30;

int build_by_source(ht_ctx* ctx, const ht_graph* g, int slot) {
  hipStream_t st = ctx->stream;
  SourceRows& S = g->by_src;
  const ItemSwitches sw;
  const int64_t V = g->V, n_ent = g->merged ? g->n_unique : g->Ep, vo = g->v_ori;
  const size_t n1 = (size_t)g->n + 1;
  const int64_t bound = item_bound(V, n_ent, sw.seg_bwd), cuts = cut_bound(n_ent, sw.seg_bwd);
  DevBlock tmp;
  plan_by_source(g, &S.blk, &tmp);
  // The list of one graph at a time is kept in a slot of the context, where the next graph finds the memory after this one was
  // destroyed (13 MiB from the device: 320 us, more than the rest of the list's making)
  if (!ctx->list_owner) {
    HT_TRY(S.blk.alloc_in(ctx, HT_S_LIST));
    ctx->list_owner = g;
  } else {
    HT_TRY(S.blk.alloc(ctx));
  }
  S.blk.take(S.idx, (size_t)std::max<int64_t>(n_ent, 1));
  if (g->merged) S.blk.take(S.w, (size_t)n_ent);
  S.blk.take(S.items.items, (size_t)bound);
  S.blk.take(S.items.cuts, (size_t)cuts);
  S.blk.take(S.ptr, (size_t)V + 1);
  ItemBuild b;
  b.nrows = V;
  b.tiles = ceil_div64(V, RTILE);
  b.seg = sw.seg_bwd;
  b.idx = S.idx.p;
  b.range = V;
  b.out = &S.items;
  DevArr<int32_t> cnt, icnt;
  DevArr<int64_t> off, lists, ibase, istarts;
  DevArr<int64_t>& ptr = S.ptr;
  DevArr<WorkItem> made;
  DevArr<uint64_t> keysA, keysB;
  HT_TRY(tmp.alloc_in(ctx, slot));   // (an allocation of its own and its release took as long as the rest of this together)
  tmp.take(cnt, (size_t)V);
  tmp.take(icnt, (size_t)3 * b.tiles);
  tmp.take(off, (size_t)std::max<int64_t>(vo, 1));
  tmp.take(lists, 3 * n1 + 2);
  tmp.take(ibase, (size_t)3 * b.tiles + 1);
  tmp.take(istarts, 6);
  tmp.take(made, (size_t)bound);
  tmp.take(keysA, (size_t)bound);
  tmp.take(keysB, (size_t)bound);
  b.cnt = icnt.p;
  b.base = ibase.p;
  b.starts = istarts.p;
  // the chunks' first arena positions, first entries and first destinations, in vertex order; then {0, V} for the one range
  int64_t* hp = nullptr;
  {
    void* p = nullptr;
    HT_TRY(ht_host_scratch(ctx, HT_HS_READBACK, (8 + 3 * n1 + 2) * 8, &p));
    hp = (int64_t*)p;
  }
  int64_t* hl = hp + 8;
  for (int k = 0; k < g->n; ++k) {
    const ChunkMeta& c = g->chunks[g->pos[k]];
    hl[k] = c.nbr_off;
    hl[n1 + k] = c.ue0;
    hl[2 * n1 + k] = c.dst0;
  }
  hl[g->n] = vo;
  hl[n1 + g->n] = n_ent;
  hl[2 * n1 + g->n] = V;
  hl[3 * n1] = 0;
  hl[3 * n1 + 1] = V;
  HT_HIP(ctx, hipMemcpyAsync(lists.p, hl, (3 * n1 + 2) * 8, hipMemcpyHostToDevice, st));
  const RowSet arena{g->merged ? g->usptr.p : g->sptr.p, lists.p, lists.p + n1, g->n};
  // ptr[u + 1] runs from where u's entries start to where they end while the chunks take their places, and is then the start of u + 1
  HT_TRY(ht_fill_zero(ctx, st, cnt.p, (size_t)V * 4));
  HT_TRY(ht_fill_zero(ctx, st, ptr.p, 8));
  if (vo > 0) {
    k_src_counts<<<nblk(vo), TB, 0, st>>>(g->nbr.p, arena, vo, cnt.p);
    HT_LAUNCH_CHECK(ctx);
  }
  HT_TRY(ht_scan_i32(ctx, cnt.p, ptr.p + 1, V, false));
  for (int k = 0; k < g->n; ++k) {
    const ChunkMeta& c = g->chunks[g->pos[k]];
    if (c.nsrc == 0) continue;
    k_src_offsets<<<nblk(c.nsrc), TB, 0, st>>>(g->nbr.p, arena, k, c.nbr_off, c.nsrc, ptr.p + 1, off.p);
    HT_LAUNCH_CHECK(ctx);
  }
  const int64_t ni = g->bwd_items.n_items;
  if (ni > 0) {
    HT_TRY(ht_in_launches(ni, HT_LAUNCH_WAVES * 64 / SRC_LANES, [&](int64_t i, int64_t m) {
      k_src_copy<<<nblk(m, TB / SRC_LANES), TB, 0, st>>>(g->bwd_items.items.p + i, m, lists.p, lists.p + 2 * n1, g->n, off.p,
                                                 g->merged ? g->usdst.p : g->sdst.p, g->merged ? g->uw_bwd.p : nullptr, S.idx.p, S.w.p);
      HT_LAUNCH_CHECK(ctx);
      return (int)HT_OK;
    }));
  }
  b.rows = RowSet{ptr.p, lists.p + 3 * n1, nullptr, 1};
  HT_TRY(count_items(ctx, b, hp));
  HT_HIP(ctx, hipStreamSynchronize(st));
  return fill_items(ctx, b, hp, made.p, (size_t)bound, keysA.p, keysB.p, (size_t)bound, sw.order);
}

}  // namespace

int64_t ht_by_source_parts_bound(int64_t entries) { return 2 * entries / ItemSwitches().seg_bwd + 1; }   // (a cut row has more than one item's)

void ht_graph_by_source_bytes(const ht_graph* g, int64_t* list, size_t* slot) {
  DevBlock kept, tmp;
  if (!g->by_src.ok) plan_by_source(g, &kept, &tmp);
  // (in its slot, which may hold some of it)
  *list = g->by_src.ok ? 0 : (int64_t)(kept.planned + kept.planned / 8);
  if (!g->ctx->list_owner) *list = std::max<int64_t>(0, *list - (int64_t)g->ctx->scratch_bytes[HT_S_LIST]);
  *slot = tmp.planned;
}

int ht_graph_by_source(ht_ctx* ctx, const ht_graph* g, int slot) {
  SourceRows& S = g->by_src;
  if (S.ok) return HT_OK;
  if (ctx->no_grow || !ht_may_spend(ctx)) return HT_ENOMEM;
  const int rc = build_by_source(ctx, g, slot);
  S.ok = rc == HT_OK;
  if (!S.ok) {
    (void)hipStreamSynchronize(ctx->stream);
    S = SourceRows();
    if (ctx->list_owner == g) ctx->list_owner = nullptr;
    if (rc == HT_ENOMEM) ctx->tight_room = ht_room(ctx);
  }
  return rc;
}

int ht_graph_by_source_mult(ht_ctx* ctx, const ht_graph* g) {
  SourceRows& S = g->by_src;
  if (!g->merged || S.mult.p) return HT_OK;
  HT_TRY(S.mult.alloc(ctx, (size_t)g->n_unique));
  if (g->n_unique > 0) {
    k_src_mult<<<(unsigned)std::min<int64_t>((g->n_unique + TB - 1) / TB, 1 << 16), TB, 0, ctx->stream>>>(S.w.p, S.idx.p, g->s.p, g->n_unique, S.mult.p);
    HT_LAUNCH_CHECK(ctx);
  }
  return HT_OK;
}

int ht_graph_source_counts(ht_ctx* ctx, const ht_graph* g, int64_t* lists, int32_t* cnt) {
  const size_t n1 = (size_t)g->n + 1;
  void* p = nullptr;
  HT_TRY(ht_host_scratch(ctx, HT_HS_READBACK, 2 * n1 * 8, &p));
  int64_t* hl = (int64_t*)p;
  for (int k = 0; k < g->n; ++k) {
    const ChunkMeta& c = g->chunks[g->pos[k]];
    hl[k] = c.nbr_off;
    hl[n1 + k] = c.ue0;
  }
  hl[g->n] = g->v_ori;
  hl[n1 + g->n] = g->merged ? g->n_unique : g->Ep;
  HT_HIP(ctx, hipMemcpyAsync(lists, hl, 2 * n1 * 8, hipMemcpyHostToDevice, ctx->stream));
  HT_TRY(ht_fill_zero(ctx, ctx->stream, cnt, (size_t)g->V * 4));
  if (g->v_ori > 0) {
    const RowSet arena{g->merged ? g->usptr.p : g->sptr.p, lists, lists + n1, g->n};
    k_src_counts<<<nblk(g->v_ori), TB, 0, ctx->stream>>>(g->nbr.p, arena, g->v_ori, cnt);
    HT_LAUNCH_CHECK(ctx);
  }
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));   // (the pinned copy of the lists is used again)
  return HT_OK;
}

int ht_graph_row_items(ht_ctx* ctx, int64_t V, const int64_t* ptr, int64_t n_ent, const int32_t* idx, const int32_t* pos, int seg, int slot,
                       DevBlock* mem, GraphItems* out) {
  const ItemSwitches sw;
  ItemBuild b;
  b.nrows = V;
  b.tiles = ceil_div64(V, RTILE);
  b.seg = seg;
  b.classes = 3;   // (items of like length in a wave: k_spmm_unit works on several; 2.45 M vertices, 62 M edges 52.0 -> 51.0 ms an epoch)
  b.idx = idx;
  b.range = V;
  b.out = out;
  const int64_t bound = item_bound(V, n_ent, b.seg);
  DevBlock tmp;
  DevArr<int32_t> cnt;
  DevArr<int64_t> base, starts, first;
  DevArr<WorkItem> made;
  DevArr<uint64_t> keysA, keysB;
  tmp.add<int32_t>((size_t)(3 * b.tiles));
  tmp.add<int64_t>((size_t)(3 * b.tiles + 1));
  tmp.add<int64_t>(6);
  tmp.add<int64_t>(2);
  tmp.add<WorkItem>((size_t)bound);
  tmp.add<uint64_t>((size_t)bound);
  tmp.add<uint64_t>((size_t)bound);
  HT_TRY(tmp.alloc_in(ctx, slot));
  tmp.take(cnt, (size_t)(3 * b.tiles));
  tmp.take(base, (size_t)(3 * b.tiles + 1));
  tmp.take(starts, 6);
  tmp.take(first, 2);
  tmp.take(made, (size_t)bound);
  tmp.take(keysA, (size_t)bound);
  tmp.take(keysB, (size_t)bound);
  b.cnt = cnt.p;
  b.base = base.p;
  b.starts = starts.p;
  void* p = nullptr;
  HT_TRY(ht_host_scratch(ctx, HT_HS_READBACK, 8 * 8, &p));
  int64_t* h = (int64_t*)p;
  h[4] = 0;
  h[5] = V;
  HT_HIP(ctx, hipMemcpyAsync(first.p, h + 4, 16, hipMemcpyHostToDevice, ctx->stream));
  b.rows = RowSet{ptr, first.p, nullptr, 1, pos};
  HT_TRY(count_items(ctx, b, h));
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  const size_t ni = (size_t)std::max<int64_t>(h[0], 1), nc = (size_t)std::max<int64_t>(h[2] - h[1], 1);
  if (mem) {
    mem->add<WorkItem>(ni);
    mem->add<CutRow>(nc);
    HT_TRY(mem->alloc(ctx));
    mem->take(out->items, ni);
    mem->take(out->cuts, nc);
  } else if (out->items.n < ni || out->cuts.n < nc) {
    return ht_set_err(ctx, HT_ESTATE, "work items: %zu and %zu cut rows, more than was planned for", ni, nc);
  }
  return fill_items(ctx, b, h, made.p, (size_t)bound, keysA.p, keysB.p, (size_t)bound, sw.order);
}

int64_t ht_graph::hbm_bytes() const {
  int64_t b = indptr.bytes() + col.bytes() + s.bytes() + nbr.bytes() + col_local.bytes() + col_slot.bytes() +
              sptr.bytes() + sdst.bytes() + slot.bytes() + gslot.bytes() + reuse.bytes() + load.bytes() +
              load_slot.bytes() + leave.bytes() + leave_slot.bytes() + uindptr.bytes() + ucol.bytes() +
              ucol_slot.bytes() + uw_fwd.bytes() + umult.bytes() + usdst.bytes() + uw_bwd.bytes() + umult_bwd.bytes() + usptr.bytes();
  b += (int64_t)(by_src.blk.mem.bytes() + by_src.mult.bytes()) + plan_fwd.bytes() + plan_bwd.bytes() + (int64_t)ranks.mem.mem.bytes();
  for (const GraphItems* i : {&fwd_items, &bwd_items}) b += i->n_items * (int64_t)sizeof(WorkItem) + i->n_cut * (int64_t)sizeof(CutRow);
  return b;
}

extern "C" {

int ht_partition(ht_ctx* ctx, int64_t V, int64_t E, const int32_t* src, const int32_t* dst, int32_t n_chunks,
                 const ht_part_opts* opts, ht_graph** out) {
  if (!ctx) return HT_EINVAL;
  if (!out) return ht_set_err(ctx, HT_EINVAL, "ht_partition: out is null");
  *out = nullptr;
  if (V <= 0 || V >= ((int64_t)1 << 31)) return ht_set_err(ctx, HT_EINVAL, "ht_partition: V must be in [1, 2^31)");
  if (E < 0 || (E > 0 && (!src || !dst))) return ht_set_err(ctx, HT_EINVAL, "ht_partition: bad edge list");
  if (n_chunks < 1) return ht_set_err(ctx, HT_EINVAL, "ht_partition: n_chunks must be >= 1");
  if (opts && (opts->reorder_chunks < 0 || opts->reorder_chunks > 1 || opts->balance_mode < 0 || opts->balance_mode > 1 || opts->ptr_loc < 0 || opts->ptr_loc > 1 ||
               opts->cache_rows < -1 || opts->cache_policy < 0 || opts->cache_policy > 1))
    return ht_set_err(ctx, HT_EINVAL, "ht_partition: bad options");
  HT_HIP(ctx, hipSetDevice(ctx->device));
  auto t0 = std::chrono::steady_clock::now();
  static std::atomic<uint64_t> next_serial{1};
  ht_graph* g = new (std::nothrow) ht_graph();
  if (g) g->serial = next_serial.fetch_add(1);
  if (!g) return ht_set_err(ctx, HT_ENOMEM, "ht_partition: host allocation failed");
  const bool held = ht_held(ctx) > 0;
  int rc = partition_impl(ctx, V, E, src, dst, n_chunks, opts, false, g);
  for (int again = held ? 0 : 1; rc == HT_ENOMEM && again < 2; ++again) {   // with what earlier calls hold given back, then with less memory
    (void)hipStreamSynchronize(ctx->stream);
    (void)ht_give_back(ctx);
    const uint64_t serial = g->serial;
    delete g;
    g = new (std::nothrow) ht_graph();
    if (!g) return ht_set_err(ctx, HT_ENOMEM, "ht_partition: host allocation failed");
    g->serial = serial;
    rc = partition_impl(ctx, V, E, src, dst, n_chunks, opts, again > 0, g);
  }
  if (rc != HT_OK) {
    (void)hipStreamSynchronize(ctx->stream);
    delete g;
    return rc;
  }
  ctx->graphs.push_back(g);
  g->partition_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  *out = g;
  return HT_OK;
}

int ht_graph_destroy(ht_graph* g) {
  if (!g) return HT_EINVAL;
  if (!g->ctx) {
    ht_free_orphan(g);
    return HT_OK;
  }
  ht_ctx* ctx = g->ctx;
  (void)hipStreamSynchronize(ctx->stream);
  ctx->graphs.erase(std::remove(ctx->graphs.begin(), ctx->graphs.end(), g), ctx->graphs.end());
  if (ctx->list_owner == g) {
    ctx->list_owner = nullptr;
    if (ctx->scratch_bytes[HT_S_LIST] > LIST_KEPT_BYTES) (void)ht_scratch_release(ctx, HT_S_LIST);
  }
  delete g;
  ht_kept_trim(ctx);
  return HT_OK;
}

int ht_graph_info_get(const ht_graph* g, ht_graph_info* out) {
  if (!g || !out) return HT_EINVAL;
  out->V = g->V;
  out->E_stored = g->Ep;
  out->n_chunks = g->n;
  out->reserved = 0;
  out->v_ori = g->v_ori;
  out->v_ru = g->v_ru;
  out->v_load = g->v_load;
  out->alpha = g->V > 0 ? (double)g->v_ori / (double)g->V : 0.0;
  out->max_nsrc = g->max_nsrc;
  out->max_ndst = g->max_ndst;
  out->max_nnz = g->max_nnz;
  out->cache_rows = g->cache_rows;
  out->hbm_bytes = g->hbm_bytes();
  out->partition_ms = g->partition_ms;
  return HT_OK;
}

int ht_graph_chunk_info(const ht_graph* g, int32_t j, ht_chunk_info* out) {
  if (!g || !out || j < 0 || j >= g->n) return HT_EINVAL;
  const ChunkMeta& c = g->chunks[j];
  out->dst_begin = c.dst0;
  out->dst_end = c.dst1;
  out->nnz = c.nnz;
  out->n_src = c.nsrc;
  out->n_reuse = c.n_reuse;
  out->n_load = c.n_load;
  out->n_leave = c.n_leave;
  return HT_OK;
}

int ht_graph_export_chunk(const ht_graph* g, int32_t j, ht_chunk_host* out) {
  if (!g || !out || j < 0 || j >= g->n) return HT_EINVAL;
  ht_ctx* ctx = g->ctx;
  const ChunkMeta& c = g->chunks[j];
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  const int64_t nd = c.dst1 - c.dst0;
  if (out->indptr) {
    HT_TRY(d2h(ctx, out->indptr, g->indptr.p + c.dst0, nd + 1));
    for (int64_t i = 0; i <= nd; ++i) out->indptr[i] -= c.e0;
  }
  HT_TRY(d2h(ctx, out->col, g->col.p + c.e0, c.nnz));
  HT_TRY(d2h(ctx, out->nbr, g->nbr.p + c.nbr_off, c.nsrc));
  HT_TRY(d2h(ctx, out->col_local, g->col_local.p + c.e0, c.nnz));
  HT_TRY(d2h(ctx, out->sptr, g->sptr.p + c.sptr_off, c.nsrc + 1));
  HT_TRY(d2h(ctx, out->sdst, g->sdst.p + c.e0, c.nnz));
  HT_TRY(d2h(ctx, out->reuse, g->reuse.p + c.reuse_off, c.n_reuse));
  HT_TRY(d2h(ctx, out->load, g->load.p + c.load_off, c.n_load));
  HT_TRY(d2h(ctx, out->slot, g->slot.p + c.nbr_off, c.nsrc));
  HT_TRY(d2h(ctx, out->leave, g->leave.p + c.leave_off, c.n_leave));
  return HT_OK;
}

int ht_graph_export_csc(const ht_graph* g, int64_t* indptr, int32_t* col, float* s, int64_t* bounds) {
  if (!g) return HT_EINVAL;
  ht_ctx* ctx = g->ctx;
  HT_HIP(ctx, hipStreamSynchronize(ctx->stream));
  HT_TRY(d2h(ctx, indptr, g->indptr.p, g->V + 1));
  HT_TRY(d2h(ctx, col, g->col.p, g->Ep));
  HT_TRY(d2h(ctx, s, g->s.p, g->V));
  if (bounds)
    for (int j = 0; j <= g->n; ++j) bounds[j] = g->bounds[j];
  return HT_OK;
}

int ht_graph_chunk_order(const ht_graph* g, int32_t* order) {
  if (!g || !order) return HT_EINVAL;
  for (int j = 0; j < g->n; ++j) order[j] = g->order[j];
  return HT_OK;
}

// Alg. 4 on neighbour bitmaps: one |V|-bit map per subgraph and one per batch union; every greedy
// step is one launch that counts the common members of all candidates with the current union.
static int reorganize_impl(ht_ctx* ctx, const ht_graph* g, int32_t m, int32_t* layout, int64_t* before, int64_t* after) {
  if (!ctx) return HT_EINVAL;
  if (!g || !layout) return ht_set_err(ctx, HT_EINVAL, "ht_graph_reorganize: null argument");
  if (g->ctx != ctx) return ht_set_err(ctx, HT_ESTATE, "graph belongs to another context");
  if (m < 1 || g->n % m != 0)
    return ht_set_err(ctx, HT_EINVAL, "ht_graph_reorganize: %d chunks do not split into %d partitions", g->n, m);
  for (int j = 0; j < g->n; ++j)
    if (g->order[j] != j)
      return ht_set_err(ctx, HT_ESTATE, "ht_graph_reorganize: the graph's chunks must be in vertex-id order (reorder_chunks = 0)");
  const int n = g->n / m, mn = g->n;
  const int64_t nw = bm_words(g->V);
  hipStream_t st = ctx->stream;
  DevArr<uint64_t> bms, U;
  HT_TRY(bms.alloc(ctx, (size_t)mn * nw));
  HT_TRY(U.alloc(ctx, (size_t)n * nw));
  {
    DevArr<uint8_t> seen;
    DevArr<int32_t> tile_cnt;
    DevArr<int64_t> d_eoff;
    std::vector<int64_t> eoff;
    for (const ChunkMeta& ch : g->chunks) eoff.push_back(ch.e0);
    eoff.push_back(g->Ep);
    int64_t grp = mark_group(nw, mn);
    int rc = seen.alloc(ctx, (size_t)grp * nw * 64);
    if (rc == HT_ENOMEM && grp > 1) {
      grp = 1;
      rc = seen.alloc(ctx, (size_t)nw * 64);
    }
    HT_TRY(rc);
    HT_TRY(tile_cnt.alloc(ctx, (size_t)mn * (nw / TB)));
    HT_TRY(d_eoff.alloc(ctx, eoff.size()));
    HT_HIP(ctx, hipMemcpyAsync(d_eoff.p, eoff.data(), eoff.size() * 8, hipMemcpyHostToDevice, st));
    HT_TRY(ht_fill_zero(ctx, st, seen.p, seen.bytes()));
    HT_TRY(mark_chunks(ctx, st, g->col.p, eoff.data(), d_eoff.p, mn, nw, grp, seen.p, bms.p, tile_cnt.p));
    HT_HIP(ctx, hipStreamSynchronize(st));
  }
  DevArr<unsigned long long> cnt;
  HT_TRY(cnt.alloc(ctx, (size_t)2 * n));
  std::vector<unsigned long long> hcnt((size_t)2 * n);
  const unsigned gx = (unsigned)std::min<int64_t>(ceil_div64(nw, TB), 64);
  // hcnt[k] = |cand_k ^ with| for the ncand bitmaps that start at cand
  auto common = [&](const uint64_t* cand, int ncand, const uint64_t* with) -> int {
    HT_HIP(ctx, hipMemsetAsync(cnt.p, 0, (size_t)ncand * 8, st));
    k_overlap<<<dim3(gx, ncand), TB, 0, st>>>(cand, nw, with, cnt.p);
    HT_LAUNCH_CHECK(ctx);
    HT_HIP(ctx, hipMemcpyAsync(hcnt.data(), cnt.p, (size_t)ncand * 8, hipMemcpyDeviceToHost, st));
    HT_HIP(ctx, hipStreamSynchronize(st));
    return HT_OK;
  };
  // V_ori, V_+p2p, V_+ru (Sec. 5.3) of a layout; uses U for the batch unions
  auto volumes = [&](const std::vector<int32_t>& lay, int64_t* out) -> int {
    HT_HIP(ctx, hipMemsetAsync(U.p, 0, (size_t)n * nw * 8, st));
    for (int j = 0; j < n; ++j)
      for (int i = 0; i < m; ++i) {
        k_bm_or<<<nblk(nw), TB, 0, st>>>(U.p + (size_t)j * nw, bms.p + (size_t)(i * n + lay[i * n + j]) * nw, nw);
        HT_LAUNCH_CHECK(ctx);
      }
    HT_HIP(ctx, hipMemsetAsync(cnt.p, 0, (size_t)2 * n * 8, st));
    for (int j = 0; j < n; ++j) {   // slot j: |U_j|; slot n + j: |U_j ^ U_{j-1}|
      k_overlap<<<dim3(gx, 1), TB, 0, st>>>(U.p + (size_t)j * nw, nw, U.p + (size_t)j * nw, cnt.p + j);
      HT_LAUNCH_CHECK(ctx);
      if (j > 0) {
        k_overlap<<<dim3(gx, 1), TB, 0, st>>>(U.p + (size_t)j * nw, nw, U.p + (size_t)(j - 1) * nw, cnt.p + n + j);
        HT_LAUNCH_CHECK(ctx);
      }
    }
    HT_HIP(ctx, hipMemcpyAsync(hcnt.data(), cnt.p, (size_t)2 * n * 8, hipMemcpyDeviceToHost, st));
    HT_HIP(ctx, hipStreamSynchronize(st));
    out[0] = g->v_ori;
    out[1] = out[2] = 0;
    for (int j = 0; j < n; ++j) {
      out[1] += (int64_t)hcnt[j];
      out[2] += (int64_t)hcnt[j] - (j > 0 ? (int64_t)hcnt[n + j] : 0);
    }
    return HT_OK;
  };
  std::vector<int32_t> lay((size_t)mn);
  for (int c = 0; c < mn; ++c) lay[c] = c % n;
  if (before) HT_TRY(volumes(lay, before));
  // ---- phase 1: the batches start as partition 0's subgraphs; every other partition hands each batch, in
  // batch order, its unassigned subgraph with the most neighbours in common with the batch's union so far
  std::vector<int32_t> Gt((size_t)mn);
  for (int j = 0; j < n; ++j) Gt[j] = j;
  HT_HIP(ctx, hipMemcpyAsync(U.p, bms.p, (size_t)n * nw * 8, hipMemcpyDeviceToDevice, st));
  for (int i = 1; i < m; ++i) {
    std::vector<char> taken(n, 0);
    for (int j = 0; j < n; ++j) {
      HT_TRY(common(bms.p + (size_t)i * n * nw, n, U.p + (size_t)j * nw));
      int best = -1;
      for (int k = 0; k < n; ++k)
        if (!taken[k] && (best < 0 || hcnt[k] > hcnt[best])) best = k;
      Gt[(size_t)i * n + j] = best;
      taken[best] = 1;
      k_bm_or<<<nblk(nw), TB, 0, st>>>(U.p + (size_t)j * nw, bms.p + (size_t)(i * n + best) * nw, nw);
      HT_LAUNCH_CHECK(ctx);
    }
  }
  // ---- phase 2: batch 0 first, then always the unplaced batch whose union shares the most with the last one
  std::vector<int32_t> at(n, 0);
  std::vector<char> placed(n, 0);
  if (n > 0) placed[0] = 1;
  for (int j = 1; j < n; ++j) {
    HT_TRY(common(U.p, n, U.p + (size_t)at[j - 1] * nw));
    int best = -1;
    for (int k = 0; k < n; ++k)
      if (!placed[k] && (best < 0 || hcnt[k] > hcnt[best])) best = k;
    at[j] = best;
    placed[best] = 1;
  }
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < n; ++j) lay[(size_t)i * n + j] = Gt[(size_t)i * n + at[j]];
  if (after) HT_TRY(volumes(lay, after));
  for (int c = 0; c < mn; ++c) layout[c] = lay[c];
  HT_HIP(ctx, hipStreamSynchronize(st));
  return HT_OK;
}

int ht_graph_reorganize(ht_ctx* ctx, const ht_graph* g, int32_t m, int32_t* layout, int64_t* before, int64_t* after) {
  if (!ctx) return HT_EINVAL;
  return ht_with_room(ctx, [&] { return reorganize_impl(ctx, g, m, layout, before, after); });
}

}  // extern "C"
