// Aggregation over the dense core of a graph on the matrix cores (Eq. 2's AGGREGATE and its backward).
//
// On a power-law graph the rows with most entries and the columns named most often meet in blocks that are far from sparse (233 k vertices,
// 78 M distinct pairs: two thirds of them lie in tiles of 256 rows x 64 columns that are at least 4 % full, once both sides are
// sorted by degree).  A gather moves 4 d bytes per entry and is held up by the requests a CU can have in flight; a tile's product
// costs the same whatever it holds, so above a few per cent of fill it is cheaper on the matrix cores.
//
// The entries in such tiles are multiplicities, small whole numbers that bf16 holds exactly (those above 255 stay with the gather).  The rows
// they multiply, s_u h_u in fp32, are split into three bf16 values whose sum they are, so that every product is exact and what
// is rounded is the fp32 sums alone, one rounding per 16 products where the gather rounds each.  The large and the two small parts have sums of their own
// (one sum for all three would round the small ones away: see k_split_tn).
//
// What a tile does not hold, the work items of ht_spmm.hip do, over a list of the remaining entries; k_spmm_fix adds both in a
// fixed order, so results are bit-reproducible.
//
// Measured, ms an epoch, all entries by 256-entry items | with this: 233 k vertices, 115 M edges, 602-256-41 20.8 | 13.0; 116 k, 57 M, 301-129-47
// 4.18 | 2.86; 2.45 M, 62 M, 100-256-256-47 64.3 | 51.2 (there 14 % of the entries lie in tiles; the short items of the rest give as much).
// Relative error against fp64 (2-norm), all by items | with this: 40 k vertices, 4 M edges, 602 columns 3.4e-8 | 3.0e-8; 20 k, 2 M, 41 columns
// 3.2e-8 | 3.2e-8; 5 k, 0.4 M, 130 columns 4.3e-8 | 3.5e-8.  Where duplicates are not merged, s_u h_u is rounded here and was inside the FMA there:
// the same graphs 3.6e-8 | 3.0e-8, 3.2e-8 | 3.2e-8, 5.2e-8 | 3.5e-8; backward 3.6e-8 | 3.4e-8, 3.6e-8 | 3.6e-8, 4.8e-8 | 3.8e-8.
#include <algorithm>
#include <vector>

#include "ht_internal.h"

namespace {

constexpr int TB = 256;
constexpr int64_t PART_ENTRIES = 32768;         // entries that one block looks at
constexpr int MAX_RB = 512, MAX_CG = 2048;      // row blocks and column groups looked at: the 131,072 rows and columns with most entries
constexpr int ETILE = 2048;
// Entries from which a tile is taken, 4 % of its cells.  A tile takes 28 ns of the card for 256 columns at 0.95 PFLOP/s; what its entries
// would take in the gather is 0.05 ns each where rows come out of L2 and up to 0.17 where they do not.  Epochs with the line at 200, 300, 450, 650 entries:
// 233 k vertices, 115 M edges 18.4, 18.2, 17.1, 17.1 ms, 2.45 M, 62 M 65.9, 65.6, 64.5, 65.8; 60 k, 3 M edges, layer at 450, 650, 1000, 2000 537, 513, 480,
// 468 us (all with other kernels beside them).
constexpr int32_t DENSE_LEAST = 650;
constexpr int SEG_BLOCKS = 512;                 // segments that a graph's tiles are cut into at least
// Entries of a work item.  The shorter, the narrower the range of rows that the items in flight read, and the more of them the L2s keep; but a row that is cut has its partial
// sums written and read.  ms an epoch with items of the rest of 24 | 32 | 40 | 48 | 64 | 96 entries: 2.45 M vertices, 22 entries
// a row left, 49.6 | 49.2 | 50.7 | 51.2 | 52.0 | 52.7; 233 k, 111 a row, 13.4 | 13.0 | 12.8 | 12.7 | 13.0 | 13.2; 116 k, 82 a row, 2.83 | 2.72 | 2.67 | 2.67 | 2.67 | 2.82.
// So items of 32 where few entries a row are left, and few rows are ones that items of 48 leave whole.  32 | 48, R-MAT epochs at 29, 40, 41, 51, 57 and 74 a row: 9.50 | 10.0, 5.14 | 5.18,
// 5.70 | 5.81, 6.20 | 6.21, 5.03 | 5.10, 5.11 | 5.11 (up to 2 % of the rows have 33 to 48 entries, 8 to 11 from 51 a row on); layers of 200 k vertices, 256 columns, whose rows are alike, 20 a row (1 %) 1.84 | 1.83, 24
// (7 %) 2.08 | 2.04, 28 (20 %) 2.40 | 2.27, 36 (70 %) 3.03 | 2.73, every row 37 2.96 | 2.65.
// Over all entries 64, however sparse the graph: with 48, graphs whose rows are alike lose more than skewed ones gain.  Layers, forward and backward, ms with items of 48 | 64
// entries: every row 54 entries, 1 M vertices, 64 columns 7.24 | 5.89, 200 k 1.08 | 0.92, 160 columns 13.7 | 13.2; 46 on average 5.76 | 5.06; R-MAT, 100 k vertices, 50 a row, 160
// columns 0.628 | 0.608, 60 k, 50 a row, 129 columns 0.374 | 0.365; 1.5 M, 13 a row, 128 columns 4.33 | 4.37, 256 columns 8.36 | 8.56, an epoch of 1 M, 10 a row, three layers 6.77 | 6.88.
constexpr int REST_SEG = 48, REST_SEG_SPARSE = 32, FINE_SEG = 64;
constexpr int64_t REST_SPARSE = 48;   // entries left a row up to which they may be the shorter ones ...
constexpr int64_t REST_ALIKE = 32;    // ... unless one row of so many has more than those take and no more than the longer ones do
inline int64_t rest_items_bound(int64_t V, int64_t most) {   // whatever part of `most` entries is left
  return std::max(ht_row_items_bound(V, most, REST_SEG), ht_row_items_bound(V, std::min(most, REST_SPARSE * V), REST_SEG_SPARSE));
}
inline unsigned nblk(int64_t n, int tb = TB) { return (unsigned)((n + tb - 1) / tb); }

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// ---- choosing the tiles

// Numbers of entries of both sides' vertices: [0] destinations, [1] sources, by a list's first entries or counted.
struct Degrees {
  const int64_t* ptr[2];
  const int32_t* cnt;      // sources, where ptr[1] is null
  __device__ __forceinline__ int64_t of(int side, int64_t v) const { return ptr[side] ? ptr[side][v + 1] - ptr[side][v] : (int64_t)cnt[v]; }
};

// How many vertices of each side have how many entries: bins of an eighth of an octave, vertices and their entries in each.
constexpr int DEG_BINS = 256;
__global__ void __launch_bounds__(TB) k_degree_bins(Degrees D, int64_t V, unsigned long long* __restrict__ bins) {
  __shared__ unsigned long long n[DEG_BINS], sum[DEG_BINS];
  static_assert(DEG_BINS == TB, "a thread per bin");
  const int side = blockIdx.y;
  n[threadIdx.x] = sum[threadIdx.x] = 0;
  __syncthreads();
  for (int64_t v = (int64_t)blockIdx.x * TB + threadIdx.x; v < V; v += (int64_t)gridDim.x * TB) {
    const int64_t d = D.of(side, v);
    if (d <= 0) continue;
    const int e = 63 - __clzll((unsigned long long)d);
    const int b = e * 8 + (int)(e >= 3 ? (d >> (e - 3)) & 7 : (d << (3 - e)) & 7);   // (entries are below 2^31)
    atomicAdd(&n[b], 1ull);
    atomicAdd(&sum[b], (unsigned long long)d);
  }
  __syncthreads();
  if (n[threadIdx.x]) {
    atomicAdd(&bins[(side * 2 + 0) * DEG_BINS + threadIdx.x], n[threadIdx.x]);
    atomicAdd(&bins[(side * 2 + 1) * DEG_BINS + threadIdx.x], sum[threadIdx.x]);
  }
}

// key = (side, most entries first, vertex)
__global__ void k_rank_keys(Degrees D, int64_t V, uint64_t* __restrict__ keys) {
  const int64_t v = (int64_t)blockIdx.x * TB + threadIdx.x;
  const int side = blockIdx.y;
  if (v >= V) return;
  const int64_t deg = D.of(side, v);
  const uint64_t k = 0x7FFFFFu - (uint64_t)(deg < 0x7FFFFF ? deg : 0x7FFFFF);
  keys[side * V + v] = ((uint64_t)side << 55) | (k << 32) | (uint64_t)v;
}
// order[side][i] = the i-th vertex (-1 behind the last), rank[side][v] = its place
__global__ void k_rank(const uint64_t* __restrict__ keys, int64_t V, int64_t n_order, int32_t* __restrict__ order0, int32_t* __restrict__ order1,
                       int32_t* __restrict__ rank0, int32_t* __restrict__ rank1) {
  const int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x;
  const int side = blockIdx.y;
  const int32_t v = i < V ? (int32_t)(keys[side * V + i] & 0xFFFFFFFFu) : -1;
  if (v >= 0) (side ? rank1 : rank0)[v] = (int32_t)i;
  if (i < n_order) (side ? order1 : order0)[i] = v;
}

// The entries of row blocks, in parts of about PART_ENTRIES: part p of block b takes an equal share of them, counted through its rows one
// after the other, so that neither a hub's row nor many short ones hold a part up.  Duplicates of an unmerged list come one after the other.
struct RowEntries {
  const int64_t* ptr;
  const int32_t* idx;
  const int32_t* order;    // rows by rank
  const int32_t* crank;    // ranks of the columns
  const int64_t* part0;    // [n_rb + 1] first part of each row block
  int n_rb;
};
// parts of every row block
__global__ void __launch_bounds__(TB) k_dense_parts(const int64_t* __restrict__ ptr, const int32_t* __restrict__ order, int32_t* __restrict__ parts) {
  __shared__ unsigned long long sum;
  if (threadIdx.x == 0) sum = 0;
  __syncthreads();
  const int32_t row = order[(int64_t)blockIdx.x * DENSE_ROWS + threadIdx.x];
  if (row >= 0) atomicAdd(&sum, (unsigned long long)(ptr[row + 1] - ptr[row]));
  __syncthreads();
  if (threadIdx.x == 0) parts[blockIdx.x] = (int32_t)((sum + PART_ENTRIES - 1) / PART_ENTRIES);
}
// The block's part: its rows' first entries and where they lie in the count.
struct Part {
  int rb;
  int64_t f0, f1;          // the share
  const int64_t* at;       // [DENSE_ROWS + 1] entries before each row
  const int64_t* first;    // [DENSE_ROWS] first entry of each row
  __device__ __forceinline__ bool open(const RowEntries& R) {
    __shared__ int64_t s_at[DENSE_ROWS + 1], s_first[DENSE_ROWS], s_wave[TB / 64];
    if ((int64_t)blockIdx.x >= R.part0[R.n_rb]) return false;
    int lo = 0, hi = R.n_rb;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (R.part0[mid] <= (int64_t)blockIdx.x) lo = mid; else hi = mid;
    }
    rb = lo;
    const int64_t p = blockIdx.x - R.part0[rb], P = R.part0[rb + 1] - R.part0[rb];
    const int tid = threadIdx.x, lane = tid & 63;      // (threads beyond the rows have none)
    const int32_t row = tid < DENSE_ROWS ? R.order[(int64_t)rb * DENSE_ROWS + tid] : -1;
    const int64_t e0 = row >= 0 ? R.ptr[row] : 0, len = row >= 0 ? R.ptr[row + 1] - e0 : 0;
    int64_t inc = len;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t y = __shfl_up(inc, o, 64);
      if (lane >= o) inc += y;
    }
    if (lane == 63 && tid < DENSE_ROWS) s_wave[tid >> 6] = inc;
    __syncthreads();
    int64_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < TB / 64; ++w) {
      if (w < (tid >> 6)) before += s_wave[w];
      tot += s_wave[w];
    }
    if (tid < DENSE_ROWS) {
      s_at[tid] = before + inc - len;
      s_first[tid] = e0;
    }
    if (tid == 0) s_at[DENSE_ROWS] = tot;
    at = s_at;
    first = s_first;
    f0 = tot * p / P;
    f1 = tot * (p + 1) / P;
    __syncthreads();
    return true;
  }
  // row (in the block) of entry f of the count
  __device__ __forceinline__ int row_of(int64_t f) const {
    int lo = 0;
#pragma unroll
    for (int b = DENSE_ROWS / 2; b > 0; b >>= 1)
      if (at[lo + b] <= f) lo += b;
    return lo;
  }
};
static_assert(DENSE_ROWS == TB, "a thread per row");

// cnt[part][column group] = distinct entries
__global__ void __launch_bounds__(TB) k_dense_count(RowEntries R, int n_cg, bool merged, int32_t* __restrict__ cnt) {
  __shared__ int32_t hist[MAX_CG];
  for (int c = threadIdx.x; c < n_cg; c += TB) hist[c] = 0;
  Part P;
  if (!P.open(R)) return;
  const int32_t limit = n_cg * DENSE_COLS;
  for (int64_t f = P.f0 + threadIdx.x; f < P.f1; f += 4 * TB) {
    int32_t u[4];
    bool ok[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t x = f + q * TB;
      ok[q] = x < P.f1;
      if (!ok[q]) continue;
      const int r = P.row_of(x);
      const int64_t e = P.first[r] + (x - P.at[r]);
      u[q] = R.idx[e];
      if (!merged && x > P.at[r] && R.idx[e - 1] == u[q]) ok[q] = false;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t c = ok[q] ? R.crank[u[q]] : limit;
      if (c < limit) atomicAdd(&hist[c / DENSE_COLS], 1);
    }
  }
  __syncthreads();
  int32_t* out = cnt + (int64_t)blockIdx.x * n_cg;
  for (int c = threadIdx.x; c < n_cg; c += TB) out[c] = hist[c];
}

// flag[block][group] = 1 where the tile is full enough; entries: what those hold together, and the column groups up to the last of them
__global__ void __launch_bounds__(TB) k_dense_select(const int32_t* __restrict__ cnt, const int64_t* __restrict__ part0, int n_cg, int64_t n, int32_t least, int32_t* __restrict__ flag,
                                                     unsigned long long* __restrict__ entries) {
  const int64_t t = (int64_t)blockIdx.x * TB + threadIdx.x;
  __shared__ int32_t used;
  if (threadIdx.x == 0) used = 0;
  __syncthreads();
  int32_t sum = 0;
  if (t < n) {
    const int64_t rb = t / n_cg, cg = t % n_cg, p1 = part0[rb + 1];
    for (int64_t p = part0[rb]; p < p1; ++p) sum += cnt[p * n_cg + cg];
    const bool take = sum >= least;
    flag[t] = take;
    if (!take) sum = 0;
    if (take) atomicMax(&used, (int32_t)cg + 1);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0 && sum > 0) atomicAdd(entries, (unsigned long long)sum);
  __syncthreads();
  if (threadIdx.x == 0 && used > 0) atomicMax(entries + 1, (unsigned long long)used);
}

// tile numbers in place of the flags (-1: not taken), the tiles' column groups, and to the host: first[block] = tiles before it, then the entries
__global__ void __launch_bounds__(TB) k_dense_tiles(const int64_t* __restrict__ id, int n_cg, int64_t n, int64_t n_rb, int32_t* __restrict__ flag,
                                                    int32_t* __restrict__ tile_cg, const unsigned long long* __restrict__ entries,
                                                    int64_t* __restrict__ host) {
  const int64_t t = (int64_t)blockIdx.x * TB + threadIdx.x;
  if (t <= n_rb) host[t] = id[t * n_cg];
  if (t == 0) {
    host[n_rb + 1] = (int64_t)entries[0];
    host[n_rb + 2] = (int64_t)entries[1];
  }
  if (t >= n) return;
  const bool take = flag[t] != 0;
  flag[t] = take ? (int32_t)id[t] : -1;
  if (take) tile_cg[id[t]] = (int32_t)(t % n_cg);
}

// ---- filling them

__global__ void k_row_lengths(const int64_t* __restrict__ ptr, int64_t V, int32_t* __restrict__ len) {
  const int64_t v = (int64_t)blockIdx.x * TB + threadIdx.x;
  if (v < V) len[v] = (int32_t)(ptr[v + 1] - ptr[v]);
}

// adds up how many lengths are above lo and not above hi
__global__ void __launch_bounds__(TB) k_count_lengths(const int32_t* __restrict__ len, int64_t V, int lo, int hi, unsigned long long* __restrict__ total) {
  const int64_t v = (int64_t)blockIdx.x * TB + threadIdx.x;
  const int32_t l = v < V ? len[v] : lo;
  const uint64_t in = __ballot(l > lo && l <= hi);
  if ((threadIdx.x & 63) == 0 && in) atomicAdd(total, (unsigned long long)__popcll(in));
}

// byte of (row, column) of a tile: 32-column stages, 32-row parts, and 16 bytes for each lane of the wave that multiplies them: its
// eight columns of the first 16, then of the second
__device__ __forceinline__ int64_t cell_at(int64_t tile, int row, int col) {
  const int k = col & 31;
  return tile * DENSE_ROWS * DENSE_COLS + (col >> 5) * (DENSE_ROWS * 32) + (row >> 5) * 1024 + ((k >> 3) & 1) * 512 + (row & 31) * 16 +
         (k >> 4) * 8 + (k & 7);
}

// The entries of the taken tiles go into their cells; keep[e] = 0 for them, and rest[row] loses them.
//
// A row's entries are in order of their columns' numbers, not ranks, so one after the other they go to tiles all over the row block, a byte each: a
// line of cells was written, and left the caches, once for each of the four or five entries that a part has for it (116 k vertices, 57 M edges, 25 M
// entries in tiles: 664 us forward, 746 backward).  The part's entries are therefore put in order of their tiles in LDS first, at the places that the
// counts give, and a tile's go out together.
constexpr int FILL_TB = 1024, FILL_LANES = 16;
__global__ void __launch_bounds__(FILL_TB) k_dense_fill(RowEntries R, const float* __restrict__ w, const float* __restrict__ mult,
                                                   const float* __restrict__ s, int n_cg, const int32_t* __restrict__ cnt,
                                                   const int32_t* __restrict__ tile_of, uint8_t* __restrict__ cells, uint8_t* __restrict__ keep,
                                                   int32_t* __restrict__ rest, int32_t* __restrict__ pos) {
  __shared__ uint32_t item[PART_ENTRIES];      // row in the block, column in the tile << 8, multiplicity << 14
  __shared__ int32_t tab[MAX_CG], next[MAX_CG], gone[DENSE_ROWS], waves[FILL_TB / 64];
  __shared__ uint16_t from[MAX_CG];
  Part P;
  if (!P.open(R)) return;
  const int tid = threadIdx.x;
  const int32_t* mine = tile_of + (int64_t)P.rb * n_cg;
  const int32_t* held = cnt + (int64_t)blockIdx.x * n_cg;
  // places: the part's entries of the taken tiles before each tile's
  constexpr int PER = MAX_CG / FILL_TB;
  int32_t n[PER], sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int c = tid * PER + q;
    const int32_t t = c < n_cg ? mine[c] : -1;
    tab[c] = t;
    n[q] = t >= 0 ? held[c] : 0;
    sum += n[q];
  }
  if (tid < DENSE_ROWS) gone[tid] = 0;
  if (!__syncthreads_or(sum)) return;
  int32_t inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(inc, o, 64);
    if ((tid & 63) >= o) inc += y;
  }
  if ((tid & 63) == 63) waves[tid >> 6] = inc;
  __syncthreads();
  int32_t place = inc - sum;
  for (int k = 0; k < (tid >> 6); ++k) place += waves[k];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    next[tid * PER + q] = place;
    from[tid * PER + q] = (uint16_t)place;
    place += n[q];
  }
  __syncthreads();
  const int32_t limit = n_cg * DENSE_COLS;
  // (four entries a thread at a time: each is a chain of loads)
  for (int64_t f = P.f0 + tid; f < P.f1; f += 4 * FILL_TB) {
    int r[4];
    int64_t e[4];
    int32_t u[4], c[4];
    float m[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t x = f + q * FILL_TB;
      r[q] = x < P.f1 ? P.row_of(x) : 0;
      e[q] = x < P.f1 ? P.first[r[q]] + (x - P.at[r[q]]) : -1;
      u[q] = e[q] >= 0 ? R.idx[e[q]] : 0;
      m[q] = w && e[q] >= 0 ? (mult ? mult : w)[e[q]] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      c[q] = e[q] >= 0 ? R.crank[u[q]] : limit;
      // (the multiplicity out of w = multiplicity * s: both roundings together are off by less than 2^-23 of it)
      if (w && !mult) m[q] = rintf(m[q] / s[u[q]]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t t = c[q] < limit ? tab[c[q] / DENSE_COLS] : -1;
      bool first = true;
      if (!w && t >= 0) {   // a run of equal entries; one of more than 255 stays as it is
        const int64_t e0 = P.first[r[q]], e1 = e0 + (P.at[r[q] + 1] - P.at[r[q]]);
        int64_t a = e[q], z = e[q] + 1;
        while (a > e0 && e[q] - a < 256 && R.idx[a - 1] == u[q]) --a;
        while (z < e1 && z - e[q] < 256 && R.idx[z] == u[q]) ++z;
        m[q] = (float)(z - a);
        first = a == e[q];
      }
      const bool take = t >= 0 && m[q] >= 1.f && m[q] <= 255.f;
      if (take) {
        if (first) item[atomicAdd(&next[c[q] / DENSE_COLS], 1)] = (uint32_t)r[q] | (uint32_t)(c[q] % DENSE_COLS) << 8 | (uint32_t)m[q] << 14;
        keep[e[q]] = 0;
      }
      // (a wave's entries are mostly one row's)
      const int r0 = __builtin_amdgcn_readfirstlane(r[q]);
      const uint64_t same = __ballot(take && r[q] == r0);
      if ((tid & 63) == __builtin_ctzll(same | (1ull << 63)) && same) atomicAdd(&gone[r0], __popcll(same));
      if (take && r[q] != r0) atomicAdd(&gone[r[q]], 1);
    }
  }
  __syncthreads();
  for (int c = tid / FILL_LANES; c < n_cg; c += FILL_TB / FILL_LANES) {
    const int32_t t = tab[c];
    if (t < 0) continue;
    for (int k = from[c] + tid % FILL_LANES; k < next[c]; k += FILL_LANES) {
      const uint32_t x = item[k];
      cells[cell_at(t, x & 255, (x >> 8) & 63)] = (uint8_t)(x >> 14);
    }
  }
  const int32_t row = tid < DENSE_ROWS ? R.order[(int64_t)P.rb * DENSE_ROWS + tid] : -1;
  if (row < 0) return;
  if (gone[tid] > 0) atomicSub(&rest[row], gone[tid]);
  pos[row] = (int32_t)(P.rb * DENSE_ROWS + tid);
}
static_assert(DENSE_ROWS == 256 && DENSE_COLS == 64 && PART_ENTRIES <= 65535, "row, column and place in an item");

// entries kept of every ETILE of them
__global__ void __launch_bounds__(TB) k_keep_count(const uint8_t* __restrict__ keep, int64_t n, int32_t* __restrict__ cnt) {
  __shared__ int32_t part[TB / 64];
  int32_t sum = 0;
  const int64_t e = (int64_t)blockIdx.x * ETILE + threadIdx.x * 8;
  if (e + 8 <= n) {
    const uint64_t q = *reinterpret_cast<const uint64_t*>(keep + e);
    sum = __popcll(q);
  } else {
    for (int j = 0; j < 8; ++j) sum += e + j < n ? keep[e + j] : 0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) cnt[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}
__global__ void __launch_bounds__(TB) k_keep_copy(const uint8_t* __restrict__ keep, int64_t n, const int64_t* __restrict__ base,
                                                  const int32_t* __restrict__ idx, const float* __restrict__ w, const float* __restrict__ s,
                                                  int32_t* __restrict__ idx_out, float* __restrict__ w_out) {
  __shared__ int32_t part[TB / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * ETILE + wave * (ETILE / 4);
  uint64_t m[ETILE / TB];
  int32_t tot = 0;
#pragma unroll
  for (int r = 0; r < ETILE / TB; ++r) {
    const int64_t e = first + r * 64 + lane;
    m[r] = __ballot(e < n && keep[e] != 0);
    tot += __popcll(m[r]);
  }
  if (lane == 0) part[wave] = tot;
  __syncthreads();
  int64_t at = base[blockIdx.x];
  for (int k = 0; k < wave; ++k) at += part[k];
#pragma unroll
  for (int r = 0; r < ETILE / TB; ++r) {
    const int64_t e = first + r * 64 + lane;
    if ((m[r] >> lane) & 1) {
      const int64_t to = at + __popcll(m[r] & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
      const int32_t u = idx[e];
      idx_out[to] = u;
      w_out[to] = w ? w[e] : s[u];
    }
    at += __popcll(m[r]);
  }
}

// ---- the products

constexpr float DSCALE = 0x1p24f, DUNSCALE = 0x1p-24f;
// Larger values (or any that are not finite) are zeros to the products and are added entry by entry behind them: 0 x inf would reach
// rows that do not name them, and scaled sums could overflow.  Below it 2^20 products of 255 and the scale stay finite.
constexpr float DLARGEST = 0x1p64f;

struct DenseArgs {
  const uint8_t* cells;
  const int32_t* tile_cg;
  const DenseSeg* segs;
  const int32_t* cols;
  const float* src;
  const float* s;
  int64_t ld, out_ld;
  int d, f0;
  float* partial;         // [segment][256] rows
};

// eight whole numbers below 256 as bf16
__device__ __forceinline__ v8bf cells8(uint32_t lo, uint32_t hi) {
  auto two = [](float a, float b) { return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u); };
  v4u r;
  r.x = two((float)(lo & 255u), (float)((lo >> 8) & 255u));
  r.y = two((float)((lo >> 16) & 255u), (float)(lo >> 24));
  r.z = two((float)(hi & 255u), (float)((hi >> 8) & 255u));
  r.w = two((float)((hi >> 16) & 255u), (float)(hi >> 24));
  return __builtin_bit_cast(v8bf, r);
}

// One segment (tiles of one row block) x BN features: 8 waves of 64 rows x BN / 2 features; one block per CU with 128 features (128 accumulators a lane), two
// with 64.  256 rows, because every column's values are read once per row block and 128 rows would ask L2 for 32 bytes a clock and CU, all
// it gives; 32 columns a stage.  The stage's columns' rows come as they are, three stages ahead (a wave takes eight of them, 256 bytes each, at
// addresses that are the same in all its lanes), and are scaled and split into three bf16 on their way into LDS.  Split by a pass of their own they were half as
// many bytes again to read: 22.6 k tiles x 602, 256 and 256 columns 2.51 ms and 0.42 for the pass, 2.79 now; 4.9 k tiles x 256 395 us, 348 now, in blocks of 64 features 320.  What bounds it: a barrier
// a stage, behind which all waves split, convert their cells and read LDS before the matrix cores have work again (39 to 42 % busy), and 3.7 TB/s of
// columns and cells that miss L2.  Tried: a range check of each value apart, with the lookup of its column, 3.9 ms; matrix and vector instructions interleaved by hand, no
// difference; LDS without its two-way conflicts (as it is here), no difference alone; segments of 24 or 88 tiles, no difference.
template <int BN>
__global__ void __launch_bounds__(512) k_dense(DenseArgs a) {
  constexpr int TJ = BN / 64, STAGE = 96 * BN, CPT = 32 * BN / 512;   // bf16 of a stage [part][8 columns][feature][8]; columns of a thread
  __shared__ __attribute__((aligned(16))) __bf16 Bs[2][STAGE];
  __shared__ int32_t col_of[DENSE_SEG * DENSE_COLS];     // the segment's columns: vertex (-1: none) ...
  __shared__ float scale_of[DENSE_SEG * DENSE_COLS];     // ... and factor
  __shared__ uint32_t odd[DENSE_SEG * 2];                // a bit for each that has a value out of range among these features
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, half = lane >> 5;
  const DenseSeg seg = a.segs[blockIdx.x];
  const int f0 = a.f0 + (int)blockIdx.y * BN, S = seg.n * 2;
  float* out = a.partial + (int64_t)blockIdx.x * DENSE_ROWS * a.out_ld;
  for (int c = tid; c < seg.n * DENSE_COLS; c += 512) {
    const int32_t u = a.cols[(int64_t)a.tile_cg[seg.tile0 + c / DENSE_COLS] * DENSE_COLS + c % DENSE_COLS];
    col_of[c] = u < 0 ? 0 : u;
    scale_of[c] = u >= 0 ? a.s[u] * DSCALE : 0.f;
  }
  if (tid < S) odd[tid] = 0;
  __syncthreads();

  v16f hi[2][TJ], lo[2][TJ];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) hi[i][j][e] = lo[i][j][e] = 0.f;

  // a thread's columns of a stage, and its feature (the columns are the same in all lanes of a wave)
  const int c0 = __builtin_amdgcn_readfirstlane(tid / BN) * CPT, fl = tid % BN, f = f0 + fl;
  const bool has = f < a.d;
  const int fc = has ? f : a.d - 1;
  float rb[2][CPT];
  v4u ra[2][2];
  int32_t cn[CPT];   // the columns of the next stage to be fetched
  auto next_cols = [&](int st) {
#pragma unroll
    for (int j = 0; j < CPT; ++j) cn[j] = col_of[(st < S ? st : S - 1) * 32 + c0 + j];
  };
  auto fetch_b = [&](int st, float* r) {
    st = st < S ? st : S - 1;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      r[j] = (a.src + (int64_t)__builtin_amdgcn_readfirstlane(cn[j]) * a.ld)[fc];
    }
  };
  auto store_b = [&](int st, int b, const float* r) {
    typedef __bf16 vbf __attribute__((ext_vector_type(CPT)));
    vbf p[3];
    float x[CPT];
    uint32_t most = 0;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      x[j] = scale_of[st * 32 + c0 + j] * r[j];
      const uint32_t mag = __float_as_uint(x[j]) & 0x7FFFFFFFu;
      most = mag > most ? mag : most;
    }
    if (__ballot(most > __float_as_uint(DLARGEST * DSCALE))) {
      uint32_t out_of_range = 0;
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const bool large = !(fabsf(x[j]) <= DLARGEST * DSCALE);
        if (__ballot(large)) out_of_range |= 1u << j;
        if (large) x[j] = 0.f;
      }
      if (lane == 0) atomicOr(&odd[st], out_of_range << c0);
    }
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      p[0][j] = (__bf16)x[j];
      const float q = x[j] - (float)p[0][j];
      p[1][j] = (__bf16)q;
      p[2][j] = (__bf16)(q - (float)p[1][j]);
    }
    __bf16* to = Bs[b] + ((c0 >> 3) * BN + fl) * 8 + (c0 & 7);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<vbf*>(to + q * 32 * BN) = p[q];
  };
  auto fetch_a = [&](int st, v4u* r) {
    st = st < S ? st : S - 1;
    const v4u* p = reinterpret_cast<const v4u*>(a.cells + ((int64_t)seg.tile0 * 2 + st) * (DENSE_ROWS * 32) + wm * 2048);
    r[0] = p[lane];
    r[1] = p[lane + 64];
  };
  next_cols(0);
  fetch_b(0, rb[0]);
  fetch_a(0, ra[0]);
  next_cols(1);
  fetch_b(1, rb[1]);
  fetch_a(1, ra[1]);
  next_cols(2);
  store_b(0, 0, rb[0]);
  fetch_b(2, rb[0]);
  next_cols(3);
  for (int st0 = 0; st0 < S; st0 += 2)   // (S is even)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int st = st0 + x;
      __syncthreads();
      v8bf m[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        m[0][i] = cells8(ra[x][i].x, ra[x][i].y);
        m[1][i] = cells8(ra[x][i].z, ra[x][i].w);
      }
      store_b(st + 1 < S ? st + 1 : S - 1, x ^ 1, rb[x ^ 1]);   // (behind the last: the last again, into the stage that nobody reads)
      fetch_a(st + 2, ra[x]);
      fetch_b(st + 3, rb[x ^ 1]);
      next_cols(st + 4);
      const __bf16* B = Bs[x] + (half * BN + wn * (BN / 2) + l32) * 8;
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          v8bf b[TJ];
#pragma unroll
          for (int j = 0; j < TJ; ++j) b[j] = *reinterpret_cast<const v8bf*>(B + ((p * 4 + k * 2) * BN + j * 32) * 8);
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
              v16f& c = p == 0 ? hi[i][j] : lo[i][j];
              c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(m[k][i], b[j], c, 0, 0, 0);
            }
        }
    }
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const int fo = f0 + wn * (BN / 2) + j * 32 + l32;
    if (fo >= ((a.d + 3) & ~3)) continue;   // (up to whole float4: lanes behind the last feature have worked on that one again, so the pads hold its sums)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = wm * 64 + i * 32 + (e >> 2) * 8 + half * 4 + (e & 3);
        out[(int64_t)r * a.out_ld + fo] = (hi[i][j][e] + lo[i][j][e]) * DUNSCALE;
      }
  }
  if (!__syncthreads_or(tid < S && odd[tid] != 0)) return;
  // What the products took for zeros: a feature and a quarter (an eighth) of the rows per thread, column by column.  233 k vertices, 115 M edges,
  // one value of 1e25 in a column that most segments hold: 61 ms an epoch when such a segment left the matrix cores altogether, 12.8 now (12.8
  // without the value); in one vertex of fifty 66 | 13.1, in one of fifty and in every block of 64 features 189 | 14.8.  Where every value is out of
  // range (a training run that has diverged) it is 61 ms, and 20.5 over work items alone.
  constexpr int PER = DENSE_ROWS / (512 / BN);
  const int r0 = __builtin_amdgcn_readfirstlane(tid / BN) * PER;
  if (!has) return;
  float acc[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) acc[i] = out[(int64_t)(r0 + i) * a.out_ld + f];
  for (int g = 0; g < S; ++g) {
    uint32_t left = __builtin_amdgcn_readfirstlane(odd[g]);
    while (left) {
      const int c = g * 32 + __builtin_ctz(left), k = c & 63;
      left &= left - 1;
      float x = scale_of[c] * a.src[(int64_t)col_of[c] * a.ld + f];
      x = fabsf(x) <= DLARGEST * DSCALE ? 0.f : a.s[col_of[c]] * a.src[(int64_t)col_of[c] * a.ld + f];   // (0: that one was in the products)
      const uint8_t* cell = a.cells + cell_at(seg.tile0 + (g >> 1), r0, k);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const uint32_t m = cell[(i >> 5) * 1024 + (i & 31) * 16];
        if (m) acc[i] = fmaf((float)m, x, acc[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) out[(int64_t)(r0 + i) * a.out_ld + f] = acc[i];
}

// Scratch memory of the making (slot HT_S_DENSE).
struct DenseTmp {
  DevBlock blk;
  DevArr<int32_t> rparts, parts, flag, tile_cg, rest, kcnt;
  DevArr<int64_t> part0, id, kbase, total;
  DevArr<uint8_t> keep;
  int64_t V, n_ent, n_rb, n_cg, n_parts;
  template <class F>
  void each(F&& f) {
    const int64_t T = n_rb * n_cg, et = ceil_div64(n_ent, ETILE);
    f(rparts, n_rb);
    f(part0, n_rb + 1);
    f(parts, n_parts * n_cg);
    f(flag, T);
    f(tile_cg, T);
    f(rest, V);
    f(kcnt, et);
    f(id, T + 1);
    f(kbase, et + 1);
    f(total, 2);
    f(keep, n_ent);
  }
  DenseTmp(int64_t v, int64_t e) : V(v), n_ent(e) {
    n_rb = std::min<int64_t>(ceil_div64(v, DENSE_ROWS), MAX_RB);
    n_cg = std::min<int64_t>(ceil_div64(v, DENSE_COLS), MAX_CG);
    n_parts = e / PART_ENTRIES + n_rb;      // at most
    each([&](auto& a, int64_t n) { blk.add<std::remove_reference_t<decltype(*a.p)>>((size_t)n); });
  }
  void take() {
    each([&](auto& a, int64_t n) { blk.take(a, (size_t)n); });
  }
};

// Both sides' numbers of entries, into a piece of `tmp` where the sources' have to be counted; `more` words behind it.
int take_degrees(ht_ctx* ctx, const ht_graph* g, DevBlock* tmp, size_t more, Degrees* out, DevArr<uint64_t>* words) {
  const bool listed = g->by_src.ok;
  DevArr<int32_t> cnt;
  DevArr<int64_t> lists;
  tmp->add<uint64_t>(more);
  if (!listed) {
    tmp->add<int32_t>((size_t)g->V);
    tmp->add<int64_t>(2 * ((size_t)g->n + 1));
  }
  HT_TRY(tmp->alloc_in(ctx, HT_S_DENSE));
  tmp->take(*words, more);
  if (!listed) {
    tmp->take(cnt, (size_t)g->V);
    tmp->take(lists, 2 * ((size_t)g->n + 1));
    HT_TRY(ht_graph_source_counts(ctx, g, lists.p, cnt.p));
  }
  *out = Degrees{{ht_row_ptr(g, true), listed ? g->by_src.ptr.p : nullptr}, cnt.p};
  return HT_OK;
}

// What the graph's dense tiles should hold if entries were spread by their row's and column's numbers of entries alone (r c / E where they have r and
// c), for either direction.  Against what they do hold: R-MAT graphs of 3 k to 2.45 M vertices 0.89 to 1.01 of it, with communities 1.15, bipartite
// 0.88.  It takes 60 us where counting the tiles of 1 M vertices, 20 M edges takes 580 for each direction, to find a fifth of what a pass over 64
// columns needs.
int estimate_tiles(ht_ctx* ctx, const ht_graph* g) {
  hipStream_t st = ctx->stream;
  DevBlock tmp;
  DevArr<uint64_t> bins;
  Degrees D;
  HT_TRY(take_degrees(ctx, g, &tmp, 4 * DEG_BINS, &D, &bins));
  HT_TRY(ht_fill_zero(ctx, st, bins.p, 4 * DEG_BINS * 8));
  k_degree_bins<<<dim3((unsigned)std::min<int64_t>(nblk(g->V), 512), 2), TB, 0, st>>>(D, g->V, (unsigned long long*)bins.p);
  HT_LAUNCH_CHECK(ctx);
  void* p = nullptr;
  HT_TRY(ht_host_scratch(ctx, HT_HS_READBACK, 4 * DEG_BINS * 8, &p));
  HT_HIP(ctx, hipMemcpyAsync(p, bins.p, 4 * DEG_BINS * 8, hipMemcpyDeviceToHost, st));
  HT_HIP(ctx, hipStreamSynchronize(st));
  // each side's heaviest vertices, as many as tiles are made of, most entries first
  struct Bin { double each, all; };
  std::vector<Bin> side[2];
  for (int k = 0; k < 2; ++k) {
    const uint64_t* h = (const uint64_t*)p + k * 2 * DEG_BINS;
    double left = (double)MAX_RB * DENSE_ROWS;
    static_assert(MAX_RB * DENSE_ROWS == MAX_CG * DENSE_COLS, "as many rows as columns");
    for (int b = DEG_BINS - 1; b >= 0 && left > 0; --b) {
      if (!h[b]) continue;
      const double n = std::min(left, (double)h[b]), each = (double)h[DEG_BINS + b] / (double)h[b];
      side[k].push_back(Bin{each, n * each});
      left -= n;
    }
  }
  const double E = (double)std::max<int64_t>(ht_entries(g), 1), least = (double)DENSE_LEAST * E / (DENSE_ROWS * DENSE_COLS);
  double sum = 0, cols = 0;
  size_t c = 0;
  for (size_t r = side[0].size(); r-- > 0;) {   // (the lightest rows first: they ask for the heaviest columns)
    for (; c < side[1].size() && side[0][r].each * side[1][c].each >= least; ++c) cols += side[1][c].all;
    sum += side[0][r].all * cols / E;
  }
  g->tile_estimate = (int64_t)sum;
  return HT_OK;
}

// g->ranks
int make_ranks(ht_ctx* ctx, const ht_graph* g) {
  hipStream_t st = ctx->stream;
  const int64_t V = g->V, n_order = std::min<int64_t>(ceil_div64(V, DENSE_ROWS), MAX_RB) * DENSE_ROWS;
  DegreeRanks& K = g->ranks;
  K = DegreeRanks();
  for (int k = 0; k < 2; ++k) {
    K.mem.add<int32_t>((size_t)n_order);
    K.mem.add<int32_t>((size_t)V);
  }
  HT_TRY(K.mem.alloc(ctx));
  for (int k = 0; k < 2; ++k) {
    K.mem.take(K.order[k], (size_t)n_order);
    K.mem.take(K.rank[k], (size_t)V);
  }
  DevBlock tmp;
  DevArr<uint64_t> keys;
  Degrees D;
  HT_TRY(take_degrees(ctx, g, &tmp, 4 * (size_t)V, &D, &keys));
  k_rank_keys<<<dim3(nblk(V), 2), TB, 0, st>>>(D, V, keys.p);
  HT_LAUNCH_CHECK(ctx);
  uint64_t* sorted = nullptr;
  HT_TRY(ht_radix_sort_u64(ctx, keys.p, keys.p + 2 * V, 2 * V, 32, 56, &sorted));
  k_rank<<<dim3(nblk(std::max(V, n_order)), 2), TB, 0, st>>>(sorted, V, n_order, K.order[0].p, K.order[1].p, K.rank[0].p, K.rank[1].p);
  HT_LAUNCH_CHECK(ctx);
  K.ok = true;
  return HT_OK;
}

// Counts the graph's dense tiles (D.taken), and makes the dense part where they hold enough for a pass over d columns.
int build_dense(ht_ctx* ctx, const ht_graph* g, bool fwd, int32_t d, DenseSide& D) {
  hipStream_t st = ctx->stream;
  const int64_t V = g->V, n_ent = ht_entries(g);
  const int64_t* ptr = ht_row_ptr(g, fwd);
  const int32_t* idx = fwd ? (g->merged ? g->ucol.p : g->col.p) : g->by_src.idx.p;
  const float* w = !g->merged ? nullptr : fwd ? g->uw_fwd.p : g->by_src.w.p;
  DenseTmp t(V, n_ent);
  // (no more than a quarter of what is there: other passes want memory too)
  const int64_t room = ht_room(ctx);
  // The slot at once as large as any step asks for it: sorting, the counts, the items of what is left.
  const size_t most = std::max(std::max(t.blk.planned, 36 * (size_t)V + 16 * ((size_t)g->n + 1) + 2048),
                               (size_t)(rest_items_bound(V, n_ent) * 32 + ceil_div64(V, 16) + 65536));
  if ((int64_t)most > room / 4 && most > ctx->scratch_bytes[HT_S_DENSE]) return HT_ENOMEM;
  void* slot = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_DENSE, most, &slot));
  if (!g->ranks.ok) HT_TRY(make_ranks(ctx, g));
  const int32_t *order_r = g->ranks.order[fwd ? 0 : 1].p, *order_c = g->ranks.order[fwd ? 1 : 0].p, *crank = g->ranks.rank[fwd ? 1 : 0].p;
  HT_TRY(t.blk.alloc_in(ctx, HT_S_DENSE));
  t.take();
  const int64_t n_rb = t.n_rb, T = n_rb * t.n_cg;
  const int n_cg = (int)t.n_cg;
  const RowEntries R{ptr, idx, order_r, crank, t.part0.p, (int)n_rb};
  k_dense_parts<<<(unsigned)n_rb, TB, 0, st>>>(ptr, order_r, t.rparts.p);
  HT_LAUNCH_CHECK(ctx);
  HT_TRY(ht_scan_i32(ctx, t.rparts.p, t.part0.p, n_rb, true));
  void *p = nullptr, *host_dev = nullptr;
  HT_TRY(ht_host_scratch(ctx, HT_HS_READBACK, (size_t)(n_rb + 8) * 8, &p));
  int64_t* host = (int64_t*)p;
  HT_HIP(ctx, hipHostGetDevicePointer(&host_dev, host, 0));
  k_dense_count<<<(unsigned)t.n_parts, TB, 0, st>>>(R, n_cg, g->merged, t.parts.p);
  HT_LAUNCH_CHECK(ctx);
  HT_TRY(ht_fill_zero(ctx, st, t.total.p, 16));
  k_dense_select<<<nblk(T), TB, 0, st>>>(t.parts.p, t.part0.p, n_cg, T, DENSE_LEAST, t.flag.p, (unsigned long long*)t.total.p);
  HT_LAUNCH_CHECK(ctx);
  HT_TRY(ht_scan_i32(ctx, t.flag.p, t.id.p, T, true));
  k_dense_tiles<<<nblk(std::max(T, n_rb + 1)), TB, 0, st>>>(t.id.p, n_cg, T, n_rb, t.flag.p, t.tile_cg.p, (const unsigned long long*)t.total.p,
                                                          (int64_t*)host_dev);
  HT_LAUNCH_CHECK(ctx);
  HT_HIP(ctx, hipStreamSynchronize(st));
  const std::vector<int64_t> first(host, host + n_rb + 1);
  const int64_t n_tiles = first[n_rb], taken = host[n_rb + 1];
  D.taken = taken;
  if (taken * d < ctx->dense_work) return HT_OK;
  // segments: the tiles of a row block, cut where there are more than a block should work through
  const int64_t seg_tiles = std::min<int64_t>(DENSE_SEG, std::max<int64_t>(2, n_tiles / SEG_BLOCKS));
  std::vector<DenseSeg> segs;
  std::vector<int32_t> seg0(n_rb + 1);
  for (int64_t b = 0; b < n_rb; ++b) {
    seg0[b] = (int32_t)segs.size();
    const int64_t n = first[b + 1] - first[b], k = ceil_div64(n, seg_tiles);
    for (int64_t j = 0; j < k; ++j) {
      const int64_t a = n * j / k, z = n * (j + 1) / k;
      segs.push_back(DenseSeg{(int32_t)(first[b] + a), (int32_t)(z - a)});
    }
  }
  seg0[n_rb] = (int32_t)segs.size();
  D.n_tiles = n_tiles;
  D.n_segs = (int64_t)segs.size();
  D.n_cols = host[n_rb + 2] * DENSE_COLS;
  const size_t cell_bytes = (size_t)n_tiles * DENSE_ROWS * DENSE_COLS;
  const int64_t left = n_ent - taken;
  auto fits = [&](int seg) { return (int64_t)cell_bytes + 8 * left + 16 * ht_row_items_bound(V, left, seg) <= room / 4; };
  if (!fits(REST_SEG)) return HT_ENOMEM;
  D.tiles.add<uint8_t>(cell_bytes);
  D.tiles.add<int32_t>((size_t)n_tiles);
  D.tiles.add<DenseSeg>(segs.size());
  D.tiles.add<int32_t>(seg0.size());
  D.tiles.add<int32_t>((size_t)V);
  D.tiles.add<int32_t>((size_t)D.n_cols);
  HT_TRY(D.tiles.alloc(ctx));
  D.tiles.take(D.cells, cell_bytes);
  D.tiles.take(D.tile_cg, (size_t)n_tiles);
  D.tiles.take(D.segs, segs.size());
  D.tiles.take(D.seg0, seg0.size());
  D.tiles.take(D.pos, (size_t)V);
  D.tiles.take(D.cols, (size_t)D.n_cols);
  HT_HIP(ctx, hipMemcpyAsync(D.segs.p, segs.data(), segs.size() * sizeof(DenseSeg), hipMemcpyHostToDevice, st));
  HT_HIP(ctx, hipMemcpyAsync(D.seg0.p, seg0.data(), seg0.size() * 4, hipMemcpyHostToDevice, st));
  HT_HIP(ctx, hipMemcpyAsync(D.cols.p, order_c, (size_t)D.n_cols * 4, hipMemcpyDeviceToDevice, st));
  HT_HIP(ctx, hipMemcpyAsync(D.tile_cg.p, t.tile_cg.p, (size_t)n_tiles * 4, hipMemcpyDeviceToDevice, st));
  HT_TRY(ht_fill_zero(ctx, st, D.cells.p, cell_bytes));
  HT_TRY(ht_fill_words(ctx, st, D.pos.p, (size_t)V * 4, 0xFFFFFFFFu));
  HT_TRY(ht_fill_words(ctx, st, t.keep.p, ((size_t)n_ent + 3) & ~(size_t)3, 0x01010101u));
  k_row_lengths<<<nblk(V), TB, 0, st>>>(ptr, V, t.rest.p);
  HT_LAUNCH_CHECK(ctx);
  k_dense_fill<<<(unsigned)t.n_parts, FILL_TB, 0, st>>>(R, w, fwd && g->merged ? g->umult.p : nullptr, g->s.p, n_cg, t.parts.p, t.flag.p, D.cells.p, t.keep.p, t.rest.p, D.pos.p);
  HT_LAUNCH_CHECK(ctx);
  // what is left, in the same order
  const int64_t et = ceil_div64(n_ent, ETILE);
  k_keep_count<<<(unsigned)et, TB, 0, st>>>(t.keep.p, n_ent, t.kcnt.p);
  HT_LAUNCH_CHECK(ctx);
  HT_TRY(ht_scan_i32(ctx, t.kcnt.p, t.kbase.p, et, true));
  HT_TRY(ht_fill_zero(ctx, st, t.total.p, 16));
  k_count_lengths<<<nblk(V), TB, 0, st>>>(t.rest.p, V, REST_SEG_SPARSE, REST_SEG, (unsigned long long*)t.total.p);
  HT_LAUNCH_CHECK(ctx);
  HT_HIP(ctx, hipMemcpyAsync(host, t.kbase.p + et, 8, hipMemcpyDeviceToHost, st));
  HT_HIP(ctx, hipMemcpyAsync(host + 1, t.total.p, 8, hipMemcpyDeviceToHost, st));
  HT_HIP(ctx, hipStreamSynchronize(st));
  D.n_rest = host[0];
  const int seg = left <= REST_SPARSE * V && host[1] * REST_ALIKE <= V && fits(REST_SEG_SPARSE) ? REST_SEG_SPARSE : REST_SEG;
  const size_t n_rest = (size_t)std::max<int64_t>(D.n_rest, 1);
  const size_t items = (size_t)ht_row_items_bound(V, D.n_rest, seg), cuts = (size_t)ht_row_cuts_bound(D.n_rest, seg, n_rb * DENSE_ROWS);
  D.rest.add<int32_t>(n_rest);
  D.rest.add<float>(n_rest);
  D.rest.add<int64_t>((size_t)V + 1);
  D.rest.add<WorkItem>(items);
  D.rest.add<CutRow>(cuts);
  HT_TRY(D.rest.alloc(ctx));
  D.rest.take(D.idx, n_rest);
  D.rest.take(D.w, n_rest);
  DevArr<int64_t> rptr;
  D.rest.take(rptr, (size_t)V + 1);
  D.rest.take(D.items.items, items);
  D.rest.take(D.items.cuts, cuts);
  k_keep_copy<<<(unsigned)et, TB, 0, st>>>(t.keep.p, n_ent, t.kbase.p, idx, w, g->s.p, D.idx.p, D.w.p);
  HT_LAUNCH_CHECK(ctx);
  HT_TRY(ht_scan_i32(ctx, t.rest.p, rptr.p, V, true));
  HT_TRY(ht_graph_row_items(ctx, V, rptr.p, D.n_rest, D.idx.p, D.pos.p, seg, HT_S_DENSE, nullptr, &D.items));
  D.ok = true;
  return HT_OK;
}

}  // namespace

namespace {

// Whether a pass over short items of the graph's own entries is the faster one, by direction, width, rows and entries.  Measured over 18 R-MAT graphs of 10 k to
// 2 M vertices, 10 to 400 entries a row, and 19 widths of 16 to 602 columns; time over the graph's own items / over short ones:
//   column units   forward   1.02 .. 1.74; 8 lanes (32 columns and less) over long rows that are hardly more than the caches hold 0.94
//                  backward  up to 64 columns 1.01 .. 1.39 below 64 entries a row, 0.93 .. 0.98 above; wider ones in (nearly) whole units 0.99 .. 1.16 (three
//                            units and fewer than 16 entries a row 0.98); with half a unit at the end (96, 160 columns) 0.89 .. 1.06
//   slab kernel    forward   from 64 columns on 1.01 .. 1.38, 0.95 .. 1.04 below 16 entries a row; narrower 0.83 .. 1.00
//                  backward  0.84 .. 1.03; 129 to 256 columns below 48 entries a row 1.00 .. 1.04, wider ones 0.96 .. 0.99, below 24 entries 1.00 .. 1.08
// (Items of the graph itself have 256 entries forward and 128 backward, so that there is less to gain backward.)
bool short_items_pay(const ht_graph* g, bool fwd, int32_t d, int64_t src_ld) {
  const int64_t V = g->V, n_ent = ht_entries(g);
  const int nvec = (std::min(d, 1024) + 3) / 4, n_units = (nvec + UNIT_LANES - 1) / UNIT_LANES;
  if (ht_unit_shape(V, src_ld, nvec, true)) {
    if (fwd) return nvec > 8 || n_ent <= 64 * V || V * src_ld * 4 >= ((int64_t)128 << 20);
    if (n_units == 1) return n_ent <= 64 * V;
    return nvec * 10 >= n_units * UNIT_LANES * 9 && (n_units != 3 || n_ent >= 16 * V);
  }
  if (fwd) return d >= 64 && n_ent >= 16 * V;
  return d > 128 && n_ent <= (d <= 256 ? 48 : 24) * V;
}

}  // namespace

int ht_pass_plan(ht_ctx* ctx, const ht_graph* g, bool fwd, int32_t d, int64_t src_ld, PassPlan* out) {
  *out = PassPlan();
  GraphPlan& P = fwd ? g->plan_fwd : g->plan_bwd;
  const int64_t n_ent = ht_entries(g);
  if (n_ent >= ((int64_t)1 << 31)) return HT_OK;
  const bool may = !ctx->static_mode && !ctx->no_grow && ht_may_spend(ctx);
  // makes `what` (its part of the plan) unless there was no memory for it with as much room as there is now
  auto make = [&](auto& what, auto&& build) -> int {
    if (!may || (what.refused >= 0 && ht_room(ctx) <= what.refused)) return HT_OK;
    if (ht_caller_captures(ctx)) return HT_OK;   // (building allocates and waits)
    const int rc = build();
    if (rc != HT_ENOMEM) return rc;
    (void)hipStreamSynchronize(ctx->stream);
    what = std::remove_reference_t<decltype(what)>();
    g->ranks = DegreeRanks();
    (void)ht_scratch_release(ctx, HT_S_DENSE);
    what.refused = ht_room(ctx);
    return HT_OK;
  };
  if (ctx->dense && n_ent * d >= ctx->dense_work) {
    DenseSide& D = P.dense;
    // (half as much again as the estimate: see there)
    auto enough = [&] { return D.taken >= 0 ? D.taken * d >= ctx->dense_work : g->tile_estimate < 0 || g->tile_estimate * 3 / 2 * d >= ctx->dense_work; };
    if (!D.ok && enough())
      HT_TRY(make(D, [&]() -> int {
        if (g->tile_estimate < 0) HT_TRY(estimate_tiles(ctx, g));
        if (!enough()) return HT_OK;
        HT_TRY(build_dense(ctx, g, fwd, d, D));
        if (g->plan_fwd.dense.taken >= 0 && g->plan_bwd.dense.taken >= 0) g->ranks = DegreeRanks();
        return HT_OK;
      }));
    if (D.ok && D.taken * d >= ctx->dense_work) {
      out->items = &D.items;
      out->dense = &D;
      return HT_OK;
    }
  }
  if (ctx->fine && n_ent * d >= ctx->fine_work && g->V * d * 4 >= ctx->fine_rows && (ctx->fine_rows == 0 || short_items_pay(g, fwd, d, src_ld))) {
    ShortItems& F = P.fine;
    if (!F.ok)
      HT_TRY(make(F, [&]() -> int {
        const int32_t* idx = fwd ? (g->merged ? g->ucol.p : g->col.p) : g->by_src.idx.p;
        HT_TRY(ht_graph_row_items(ctx, g->V, ht_row_ptr(g, fwd), n_ent, idx, nullptr, FINE_SEG, HT_S_DENSE, &F.mem, &F.items));
        F.ok = true;
        return HT_OK;
      }));
    if (F.ok) out->items = &F.items;
  }
  return HT_OK;
}

// The segments' sums into partial ([segment][256] rows of pitch out_ld).
int ht_dense_launch(ht_ctx* ctx, hipStream_t st, const DenseSide& D, const float* src, int64_t ld, const float* s, int32_t d, float* partial,
                    int64_t out_ld) {
  // Blocks of 128 features decode a cell half as often, blocks of 64 leave shorter last rounds and take what is left behind the last 128 along.  us, 128 (and 64) | 64 alone: 22.6 k
  // tiles x 602 1546 | 1634, x 256 610 | 659; 4.9 k x 256 346 | 320, x 100 199 | 197; 7 k x 129 312 | 283.
  // Between them either does; ms a layer forward and backward, 12.3 k x 256 2.38 | 2.37, x 384 3.37 | 3.35, x 602 5.28 | 5.27; 16.9 k x 256 3.21 | 3.22, x 512 6.56 | 6.60; 20.3 k x 256 4.21 | 4.18.
  int n128 = d / 128 + (d % 128 > 64);
  if (D.n_tiles * n128 < ctx->dense_wide) n128 = 0;
  DenseArgs a{D.cells.p, D.tile_cg.p, D.segs.p, D.cols.p, src, s, ld, out_ld, d, 0, partial};
  if (n128 > 0) {
    k_dense<128><<<dim3((unsigned)D.n_segs, n128), 512, 0, st>>>(a);
    HT_LAUNCH_CHECK(ctx);
  }
  if (d > n128 * 128) {
    a.f0 = n128 * 128;
    k_dense<64><<<dim3((unsigned)D.n_segs, (unsigned)((d - a.f0 + 63) / 64)), 512, 0, st>>>(a);
    HT_LAUNCH_CHECK(ctx);
  }
  return HT_OK;
}
