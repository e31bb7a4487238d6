// Device-wide primitives for the integer (preprocessing) part: exclusive scan,
// stable LSD radix sort of 64-bit keys, bitmap rank.  Wave64 ballot,
// popcount and shuffle scans do the in-wave work.
#include <utility>

#include "ht_internal.h"

namespace {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

__device__ __forceinline__ int64_t wave_incl_scan_i64(int64_t x, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// Exclusive scan of one value per thread across a 256-thread block.
// Returns the exclusive prefix; *total gets the block sum (valid in all threads).
__device__ __forceinline__ int64_t block_excl_scan_i64(int64_t x, int64_t* total) {
  __shared__ int64_t wsum[SCAN_THREADS / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t inc = wave_incl_scan_i64(x, lane);
  __syncthreads();  // protect wsum against a previous use
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int64_t off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < SCAN_THREADS / 64; ++w) {
    if (w < wave) off += wsum[w];
    tot += wsum[w];
  }
  *total = tot;
  return off + inc - x;
}

template <typename Tin>
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_reduce(const Tin* __restrict__ in, int64_t n,
                                                             int64_t* __restrict__ block_sums) {
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  int64_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    int64_t idx = base + i;
    if (idx < n) s += (int64_t)in[idx];
  }
  int64_t tot;
  block_excl_scan_i64(s, &tot);
  if (threadIdx.x == 0) block_sums[blockIdx.x] = tot;
}

// block_offsets may be null (single block).  out may alias in when Tin is int64.
// RAW_SUMS: block_offsets holds the blocks' own sums, not their prefix; a block adds up the sums
// before it by itself (a few thousand values at most), which saves the launch that scans them.
template <typename Tin, bool RAW_SUMS>
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_apply(const Tin* in, int64_t n,
                                                            const int64_t* __restrict__ block_offsets,
                                                            int64_t* out, int want_total) {
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  int64_t before = 0;
  if (RAW_SUMS) {
    int64_t part = 0;
    for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += SCAN_THREADS) part += block_offsets[i];
    block_excl_scan_i64(part, &before);
  } else if (block_offsets) {
    before = block_offsets[blockIdx.x];
  }
  int64_t v[SCAN_ITEMS];
  int64_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    int64_t idx = base + i;
    v[i] = idx < n ? (int64_t)in[idx] : 0;
    s += v[i];
  }
  int64_t tot;
  int64_t off = block_excl_scan_i64(s, &tot) + before;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    int64_t idx = base + i;
    if (idx < n) out[idx] = off;
    off += v[i];
  }
  if (want_total && blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_THREADS - 1) out[n] = off;
}

// One block walks the whole input tile by tile with a running carry: one launch for short inputs
// (bitmap word counts, per-row item counts of a chunk).  out may alias in when Tin is int64.
template <typename Tin>
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_one_block(const Tin* in, int64_t n, int64_t* out,
                                                                int want_total) {
  int64_t carry = 0;
  for (int64_t t0 = 0; t0 < n; t0 += SCAN_TILE) {
    const int64_t base = t0 + (int64_t)threadIdx.x * SCAN_ITEMS;
    int64_t v[SCAN_ITEMS];
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
      int64_t idx = base + i;
      v[i] = idx < n ? (int64_t)in[idx] : 0;
      s += v[i];
    }
    int64_t tot;
    int64_t off = block_excl_scan_i64(s, &tot) + carry;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
      int64_t idx = base + i;
      if (idx < n) out[idx] = off;
      off += v[i];
    }
    carry += tot;
  }
  if (want_total && threadIdx.x == 0) out[n] = carry;
}

// Up to here one block is faster than two launches: 2.6 us per tile (10,000 words 13.5 us, 22,000 words 28.7), the two 8 us and a launch gap.
constexpr int64_t SCAN_ONE_BLOCK_MAX = 4 * SCAN_TILE;
constexpr int64_t SCAN_RAW_SUMS_MAX = 4096;              // blocks whose sums each block adds up by itself

// Block sums of every level live back to back in one scratch slot of the context (the level of n elements
// needs ceil(n / SCAN_TILE) sums, the next one a tile-th of that, ...): no allocation, hence no
// implicit device synchronisation, per call.  ws points at this level's sums.
template <typename Tin>
int scan_level(ht_ctx* ctx, const Tin* in, int64_t* out, int64_t n, bool want_total, int64_t* ws) {
  const int64_t nb = ceil_div64(n, SCAN_TILE);
  const int wt = want_total ? 1 : 0;
  if (n <= SCAN_ONE_BLOCK_MAX) {
    k_scan_one_block<Tin><<<1, SCAN_THREADS, 0, ctx->stream>>>(in, n, out, wt);
    HT_LAUNCH_CHECK(ctx);
    return HT_OK;
  }
  k_scan_reduce<Tin><<<(unsigned)nb, SCAN_THREADS, 0, ctx->stream>>>(in, n, ws);
  HT_LAUNCH_CHECK(ctx);
  if (nb <= SCAN_RAW_SUMS_MAX) {
    k_scan_apply<Tin, true><<<(unsigned)nb, SCAN_THREADS, 0, ctx->stream>>>(in, n, ws, out, wt);
    HT_LAUNCH_CHECK(ctx);
    return HT_OK;
  }
  HT_TRY(scan_level<int64_t>(ctx, ws, ws, nb, false, ws + nb));
  k_scan_apply<Tin, false><<<(unsigned)nb, SCAN_THREADS, 0, ctx->stream>>>(in, n, ws, out, wt);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}

template <typename Tin>
int scan_impl(ht_ctx* ctx, const Tin* in, int64_t* out, int64_t n, bool want_total) {
  if (n < 0) return ht_set_err(ctx, HT_EINVAL, "scan: negative length");
  if (n == 0) {
    if (want_total) HT_HIP(ctx, hipMemsetAsync(out, 0, sizeof(int64_t), ctx->stream));
    return HT_OK;
  }
  size_t sums = 0;
  for (int64_t m = ceil_div64(n, SCAN_TILE); m > 1; m = ceil_div64(m, SCAN_TILE)) sums += (size_t)m;
  int64_t* ws = nullptr;
  if (sums > 0) HT_TRY(ht_scratch(ctx, HT_S_SCAN, sums * sizeof(int64_t), (void**)&ws));
  return scan_level<Tin>(ctx, in, out, n, want_total, ws);
}

// ------------------------------------------------------------------ radix sort
// A pass counts digits per block, turns the counts into places, and scatters.  Long inputs take 512 threads of 16 keys and digits of up to 9 bits, with a scan
// launch between the two kernels.  Short ones (up to RS_SHORT_BLOCKS blocks) take 256 threads of 8 keys, for more blocks with shorter
// chains, and digits of 8 bits, and every block of the scatter adds up the counts by itself, a digit per thread: that is at most 128 rows of 1 KB out
// of the L2, where the scan is a launch of one block (110,000 keys: 23 -> 12 us per pass).
template <int THREADS>
struct RadixShape {
  static constexpr bool brief = THREADS == 256;
  static constexpr int waves = THREADS / 64, rounds = brief ? 8 : 16, tile = THREADS * rounds, bits = brief ? 8 : 9, bins = 1 << bits;
};
constexpr int RS_SHORT = 256, RS_LONG = 512;   // threads
constexpr int64_t RS_SHORT_BLOCKS = 128;

// The keys first, first + stride, ... below n of a thread: from the keys, or (the first pass over edges) from the edges they are made of.
template <int R, bool EDGES>
struct RadixKeys {
  uint64_t key[R];
  __device__ __forceinline__ bool load(const uint64_t* __restrict__ keys, const EdgeKeys& E, int64_t first, int stride, int64_t n) {
    if (!EDGES) {
#pragma unroll
      for (int r = 0; r < R; ++r) key[r] = first + r * stride < n ? keys[first + r * stride] : 0ull;
      return true;
    }
    uint32_t u[R], v[R];
    bool ok = true;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      u[r] = v[r] = 0;
      if (first + r * stride < n) E.load(first + r * stride, &u[r], &v[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ok = ok && E.valid(u[r], v[r]);
      key[r] = E.key(u[r], v[r]);
    }
    return ok;
  }
};

// table: [digit][block] for the scan, [block][digit] for short inputs
template <int THREADS, bool EDGES>
__global__ void __launch_bounds__(THREADS) k_rs_hist(const uint64_t* __restrict__ keys, EdgeKeys E, int64_t n, int shift, uint32_t mask,
                                                     int32_t* __restrict__ table, int64_t nblocks) {
  using S = RadixShape<THREADS>;
  __shared__ uint32_t h[S::bins];
  for (int i = threadIdx.x; i < S::bins; i += THREADS) h[i] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * S::tile + threadIdx.x;
  RadixKeys<S::rounds, EDGES> k;
  if (!k.load(keys, E, base, THREADS, n)) *E.flag = 1;
#pragma unroll
  for (int r = 0; r < S::rounds; ++r)
    if (base + r * THREADS < n) atomicAdd(&h[(uint32_t)(k.key[r] >> shift) & mask], 1u);
  __syncthreads();
  for (int d = threadIdx.x; d < S::bins; d += THREADS) {
    if (S::brief) table[(int64_t)blockIdx.x * S::bins + d] = (int32_t)h[d];
    else table[(int64_t)d * nblocks + blockIdx.x] = (int32_t)h[d];
  }
}

// Stable scatter.  Key order inside a block is (wave, round, lane) = index
// order.  A lane's rank among equal digits: earlier waves' counts, earlier
// rounds of its own wave, lower lanes of its own round (ballot match).
// The block first puts its keys into digit order in LDS and then writes them out in that order, so that
// consecutive lanes store consecutive keys of one digit's run (a lane storing its own key straight to its
// final place touches a 128-byte line of the output from up to 16 different store instructions).
// What bounds it is the runs' ragged ends: a line that two blocks share leaves the caches of two XCDs as two partial writes.  So each XCD takes a contiguous
// part of the tiles (the next tile's run of a digit then finds the line in the same L2), and a tile is as large as two blocks in a CU's LDS allow.  64 M
// keys, a pass's scatter: 4,096 keys a tile in launch order 375 us, 8,192 keys 295, each XCD its own part 265 (3.9 TB/s read and written); 16,384 keys, one
// block a CU 370.  With digits of 9 bits 275, and 44 bits take five passes instead of six (in launch order 9 bits lost by shorter runs what the pass saved).
// 2.45 M vertices, 62 M edges: partition and one layer 13.5 -> 11.7 ms.
template <int THREADS, bool EDGES>
__global__ void __launch_bounds__(THREADS) k_rs_scatter(const uint64_t* __restrict__ in, EdgeKeys E, uint64_t* __restrict__ out, int64_t n, int shift,
                                                        uint32_t mask, const int64_t* __restrict__ offs, const int32_t* __restrict__ table,
                                                        int64_t nblocks) {
  using S = RadixShape<THREADS>;
  static_assert(S::bins <= THREADS, "a digit per thread");
  __shared__ uint16_t cnt[S::waves][S::bins];
  __shared__ int64_t goff[S::bins];     // where the block's run of a digit starts in the output, minus lstart
  __shared__ uint16_t lstart[S::bins];  // where it starts in the block's tile
  __shared__ uint32_t wtot[S::bins / 64];
  __shared__ uint64_t tile[S::tile];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t block = S::brief ? (int64_t)blockIdx.x : (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (block >= nblocks) return;
  for (int i = threadIdx.x; i < S::waves * S::bins; i += THREADS) (&cnt[0][0])[i] = 0;
  __syncthreads();

  RadixKeys<S::rounds, EDGES> mine;
  const uint64_t (&key)[S::rounds] = mine.key;
  uint16_t rank[S::rounds];
  const int64_t base = block * S::tile + (int64_t)wave * (64 * S::rounds);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  mine.load(in, E, base + lane, 64, n);
#pragma unroll
  for (int r = 0; r < S::rounds; ++r) {
    const bool valid = base + r * 64 + lane < n;
    const uint32_t dg = (uint32_t)(key[r] >> shift) & mask;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < S::bits; ++b) {
      const bool bit = (dg >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const uint32_t before = valid ? cnt[wave][dg] : 0u;
    __builtin_amdgcn_wave_barrier();
    const uint32_t lower = (uint32_t)__popcll(peers & lt);
    if (valid && lower == 0) cnt[wave][dg] = (uint16_t)(before + (uint32_t)__popcll(peers));
    __builtin_amdgcn_wave_barrier();
    rank[r] = (uint16_t)(before + lower);
  }
  __syncthreads();
  {
    const int dgt = threadIdx.x;  // one digit per thread (threads behind them have none)
    const bool has = dgt < S::bins;
    uint32_t run = 0;
    if (has) {
#pragma unroll
      for (int w = 0; w < S::waves; ++w) {
        const uint32_t c = cnt[w][dgt];
        cnt[w][dgt] = (uint16_t)run;
        run += c;
      }
    }
    // exclusive prefix of the digit totals over the block's digits
    uint32_t inc = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(inc, o, 64);
      if (lane >= o) inc += y;
    }
    if (has && lane == 63) wtot[wave] = inc;
    __syncthreads();
    uint32_t off = 0;
#pragma unroll
    for (int w = 0; w < S::bins / 64; ++w)
      if (w < wave) off += wtot[w];
    const uint32_t ls = off + inc - run;
    if (has) lstart[dgt] = (uint16_t)ls;
    if (!S::brief) {
      if (has) goff[dgt] = offs[(int64_t)dgt * nblocks + block] - (int64_t)ls;
    } else {   // keys of smaller digits, and of this digit in the blocks before
      uint32_t earlier = 0, total = 0;
#pragma unroll 16
      for (int b = 0; b < (int)nblocks; ++b) {
        const uint32_t c = (uint32_t)table[b * S::bins + dgt];
        total += c;
        earlier += b < (int)block ? c : 0u;
      }
      uint32_t upto = total;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(upto, o, 64);
        if (lane >= o) upto += y;
      }
      __syncthreads();   // (wtot is read above)
      if (lane == 63) wtot[wave] = upto;
      __syncthreads();
      uint32_t lower = upto - total;
#pragma unroll
      for (int w = 0; w < S::bins / 64; ++w)
        if (w < wave) lower += wtot[w];
      goff[dgt] = (int64_t)(lower + earlier) - (int64_t)ls;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < S::rounds; ++r) {
    if (base + r * 64 + lane < n) {
      const uint32_t dg = (uint32_t)(key[r] >> shift) & mask;
      tile[(uint32_t)lstart[dg] + cnt[wave][dg] + rank[r]] = key[r];
    }
  }
  __syncthreads();
  const int64_t left = n - block * S::tile;
  const int here = left < S::tile ? (int)left : S::tile;
#pragma unroll 4
  for (int i = threadIdx.x; i < here; i += THREADS) {
    const uint64_t k = tile[i];
    const uint32_t dg = (uint32_t)(k >> shift) & mask;
    out[goff[dg] + i] = k;
  }
}

// ------------------------------------------------------------------ bitmaps
__global__ void k_popc(const uint64_t* __restrict__ bm, int64_t nw, int32_t* __restrict__ cnt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nw) cnt[i] = __popcll(bm[i]);
}

}  // namespace

int ht_scan_i32(ht_ctx* ctx, const int32_t* in, int64_t* out, int64_t n, bool want_total) {
  return scan_impl<int32_t>(ctx, in, out, n, want_total);
}
int ht_scan_i64(ht_ctx* ctx, const int64_t* in, int64_t* out, int64_t n, bool want_total) {
  return scan_impl<int64_t>(ctx, in, out, n, want_total);
}

namespace {

template <int THREADS, bool EDGES>
int radix_pass(ht_ctx* ctx, const uint64_t* in, const EdgeKeys& E, uint64_t* out, int64_t n, int shift, int bits, int64_t* offs, int32_t* table) {
  using S = RadixShape<THREADS>;
  const int64_t nblocks = ceil_div64(n, S::tile);
  const uint32_t mask = (1u << bits) - 1u;
  k_rs_hist<THREADS, EDGES><<<(unsigned)nblocks, THREADS, 0, ctx->stream>>>(in, E, n, shift, mask, table, nblocks);
  HT_LAUNCH_CHECK(ctx);
  if (!S::brief) HT_TRY(ht_scan_i32(ctx, table, offs, S::bins * nblocks, false));
  k_rs_scatter<THREADS, EDGES><<<(unsigned)(S::brief ? nblocks : (nblocks + 7) / 8 * 8), THREADS, 0, ctx->stream>>>(in, E, out, n, shift, mask, offs, table, nblocks);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}

template <int THREADS>
int radix_sort(ht_ctx* ctx, const EdgeKeys* edges, uint64_t* keys, uint64_t* tmp, int64_t n, int bit_lo, int bit_hi, uint64_t** sorted) {
  using S = RadixShape<THREADS>;
  // per-block digit counts and their offsets, in a scratch slot of the context (no allocation per call)
  const size_t cells = (size_t)(S::bins * ceil_div64(n, S::tile));
  char* rs = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_RSORT, cells * 12 + 16, (void**)&rs));
  int64_t* offs = (int64_t*)rs;
  int32_t* table = (int32_t*)(rs + cells * 8);
  const int passes = (bit_hi - bit_lo + S::bits - 1) / S::bits;
  uint64_t *a = keys, *b = tmp;
  for (int p = 0; p < passes; ++p) {
    const int lo = bit_lo + (bit_hi - bit_lo) * p / passes, hi = bit_lo + (bit_hi - bit_lo) * (p + 1) / passes;   // (digits of like width)
    if (p == 0 && edges) HT_TRY((radix_pass<THREADS, true>(ctx, nullptr, *edges, b, n, lo, hi - lo, offs, table)));
    else HT_TRY((radix_pass<THREADS, false>(ctx, a, EdgeKeys{}, b, n, lo, hi - lo, offs, table)));
    std::swap(a, b);
  }
  *sorted = a;
  return HT_OK;
}

__global__ void k_pack_keys(EdgeKeys E, int64_t n, uint64_t* __restrict__ keys) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t u, v;
  E.load(i, &u, &v);
  if (!E.valid(u, v)) *E.flag = 1;
  keys[i] = E.key(u, v);
}

int sort_any(ht_ctx* ctx, const EdgeKeys* edges, uint64_t* keys, uint64_t* tmp, int64_t n, int bit_lo, int bit_hi, uint64_t** sorted) {
  return n <= RS_SHORT_BLOCKS * RadixShape<RS_SHORT>::tile ? radix_sort<RS_SHORT>(ctx, edges, keys, tmp, n, bit_lo, bit_hi, sorted)
                                                          : radix_sort<RS_LONG>(ctx, edges, keys, tmp, n, bit_lo, bit_hi, sorted);
}

}  // namespace

int ht_radix_sort_u64(ht_ctx* ctx, uint64_t* keys, uint64_t* tmp, int64_t n, int bit_lo, int bit_hi,
                      uint64_t** sorted) {
  *sorted = keys;
  if (n <= 1 || bit_hi <= bit_lo) return HT_OK;
  return sort_any(ctx, nullptr, keys, tmp, n, bit_lo, bit_hi, sorted);
}

int ht_radix_sort_edges(ht_ctx* ctx, const EdgeKeys& edges, uint64_t* keys, uint64_t* tmp, int64_t n, uint64_t** sorted) {
  *sorted = keys;
  if (n <= 0) return HT_OK;
  if (edges.bits > 0) return sort_any(ctx, &edges, keys, tmp, n, 0, 2 * edges.bits, sorted);
  k_pack_keys<<<(unsigned)ceil_div64(n, 256), 256, 0, ctx->stream>>>(edges, n, keys);   // (one vertex: nothing to sort)
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}

int ht_bitmap_prefix(ht_ctx* ctx, const uint64_t* bm, int64_t nw, int32_t* cnt_tmp, int64_t* pref) {
  if (nw > 0) {
    k_popc<<<(unsigned)ceil_div64(nw, 256), 256, 0, ctx->stream>>>(bm, nw, cnt_tmp);
    HT_LAUNCH_CHECK(ctx);
  }
  return ht_scan_i32(ctx, cnt_tmp, pref, nw, true);
}
