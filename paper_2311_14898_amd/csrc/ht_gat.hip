// GAT layer (Eq. 3), one attention head, forward and backward over the chunks
// of a partitioned graph.  The layer's tensors H_in, H_out, dH_out, dH_in may live
// in HBM or in pinned host memory; the parameterised rows t = H W of all vertices
// always stay in HBM for the duration of a call, so neighbour rows never cross the
// host link: a host-resident tensor is only ever read or written in contiguous row
// ranges (V rows per pass instead of the sum of |N_j|), through staging pairs on
// side streams.
//
//   t = H W ;  p_v = a_dst . t_v ;  q_u = a_src . t_u
//   edge (u -> v):  y = p_v + q_u ;  x = LeakyReLU(y) ;  alpha = softmax over in(v)
//   z_v = sum alpha_e t_u ;  h'_v = act(z_v)
//
// A chunk holds every in-edge of its destinations (Sec. 4.1), so the neighbour
// softmax is complete inside a chunk.  With everything in HBM the chunks run
// together, as many as the scratch memory of their scores allows.  Nothing of size
// O(E) survives a call: the backward pass of a layer call recomputes t, p, q and the
// scores (Sec. 4.2: for models with edge computation recomputation is cheaper than
// caching O(|E|) data); an epoch with room for it keeps rows of size O(V) from each
// layer's forward pass (GatKeep), which spare its backward pass the recomputation.
//
// Backward.  With dz = dh' * act'(z) and S_v = dz_v . z_v  (= sum_e alpha_e dalpha_e):
//   dalpha_e = dz_v . t_u ;  dy_e = alpha_e (dalpha_e - S_v) f_e ,  f_e = LeakyReLU'(y_e)
//   dp_v = sum_{e in in(v)} dy_e  = dz_v . (sum_e alpha_e f_e t_u) - S_v sum_e alpha_e f_e
//                                     (pass over destinations, an aggregation of rows of t)
//   dq_u = sum_{e in out(u)} dy_e = t_u . (sum_e alpha_e f_e dz_v) - sum_e alpha_e f_e S_v
//   dt_u = sum_{e in out(u)} alpha_e dz_v
//                                     (pass over sources, two aggregations of the same rows of dz)
//   dt_v += dp_v a_dst + dq_v a_src ;  da_dst = sum_v dp_v t_v ;  da_src = sum_v dq_v t_v
//   dW = H^T dt ;  dH = dt W^T
// Both passes are pulls over the work items built at partition time; rows cut
// into several items are finished in a fixed order, so results are bit-reproducible.
// Merged duplicate edges: an entry of multiplicity k stands for k equal edges,
// its coefficient is k times the single edge's.
#include <algorithm>
#include <chrono>
#include <vector>

#include "ht_internal.h"

namespace {

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void st4(float* p, float4 v) { *reinterpret_cast<float4*>(p) = v; }
__device__ __forceinline__ float4 fma4(float w, float4 v, float4 a) {
  return make_float4(fmaf(w, v.x, a.x), fmaf(w, v.y, a.y), fmaf(w, v.z, a.z), fmaf(w, v.w, a.w));
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ __forceinline__ float lrelu(float y, float slope) { return y > 0.f ? y : slope * y; }
// coefficient of one entry; the same expression in every kernel, so the forward, the
// destination pass and the source pass of a chunk see identical values
__device__ __forceinline__ float coef(float y, float slope, float m, float zinv, float mult) {
  const float x = lrelu(y, slope);
  return mult * expf(x - m) * zinv;
}

// sum over a group of `lpr` lanes (a power of two)
__device__ __forceinline__ float group_sum(float x, int lpr) {
  for (int o = lpr >> 1; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
// the attention vectors (at most 1024 long) in LDS, zero behind their end
struct AttVec {
  float4 dst[256], src[256];
};
__device__ __forceinline__ void load_att(AttVec& s, const float* a_dst, const float* a_src, int d) {
  for (int c = threadIdx.x; c < ((d + 3) & ~3); c += 256) {
    reinterpret_cast<float*>(s.dst)[c] = c < d ? a_dst[c] : 0.f;
    reinterpret_cast<float*>(s.src)[c] = c < d ? a_src[c] : 0.f;
  }
  __syncthreads();
}
__device__ __forceinline__ float dot4(float4 a, float4 b, float s) { return fmaf(a.x, b.x, fmaf(a.y, b.y, fmaf(a.z, b.z, fmaf(a.w, b.w, s)))); }
// Lanes per row of the kernels below, which go over the rows of a matrix once: a float4 each, 8 to 64 (a wave per row left most
// lanes of narrow rows idle: 20 k rows of 33 and 7 columns, 6.7 + 5.4 us for dz and dp, 5.0 us for both now).
unsigned row_grid(int64_t rows, int lpr) { return (unsigned)std::min<int64_t>((rows * lpr + 255) / 256, 8192); }
int row_lanes(int64_t ld) { return ld <= 32 ? 8 : ld <= 64 ? 16 : ld <= 128 ? 32 : 64; }

// p[v] = a_dst . T[v], q[v] = a_src . T[v]; lpr lanes per vertex.  The pads of T up to the next multiple of 4 columns, which later passes read as data, become
// zeros on the way (clearing all of T before the product was a launch of its own).
__global__ void __launch_bounds__(256) k_gat_pq(float* __restrict__ T, int64_t ld, int d, const float* __restrict__ a_dst,
                                                const float* __restrict__ a_src, int64_t V, float* __restrict__ p,
                                                float* __restrict__ q, int lpr) {
  __shared__ AttVec sa;
  load_att(sa, a_dst, a_src, d);
  const int rpb = 256 / lpr, ll = threadIdx.x % lpr;
  for (int64_t v = (int64_t)blockIdx.x * rpb + threadIdx.x / lpr; v < V; v += (int64_t)gridDim.x * rpb) {
    float sp = 0.f, sq = 0.f;
    for (int c = ll * 4; c < d; c += lpr * 4) {
      float4 t = ld4(T + v * ld + c);
      if (c + 4 > d) {
        if (c + 1 >= d) t.y = 0.f;
        if (c + 2 >= d) t.z = 0.f;
        t.w = 0.f;
        st4(T + v * ld + c, t);
      }
      sp = dot4(sa.dst[c >> 2], t, sp);
      sq = dot4(sa.src[c >> 2], t, sq);
    }
    sp = group_sum(sp, lpr);
    sq = group_sum(sq, lpr);
    if (ll == 0) {
      p[v] = sp;
      q[v] = sq;
    }
  }
}

// Neighbour softmax of a range of rows in three steps over the work items (a wave per
// item, so a hub row is shared by many waves):
//   1. per item: the scores x_e (kept in w[]), their maximum m_i and s_i = sum mult_e exp(x_e - m_i);
//   2. per row cut into several items: m_v = max m_i, Z_v = sum s_i exp(m_i - m_v), in a fixed order;
//   3. where they are used: w_e = mult_e exp(x_e - m_v) / Z_v.
// Rows are vertices; w holds the entries from ent0 on, part_* the partial results from part0 on.
// What bounds step 1 is the chain of loads of an entry (its source, the source's q) in items of up to 256 entries: one after the other they took 485 us for 78 M
// entries, 360 with four a lane on the way together and kept.
constexpr int SCORE_REGS = 4;
__global__ void __launch_bounds__(256) k_gat_scores(const WorkItem* __restrict__ items, int64_t n_items, int64_t ent0, int64_t part0,
                                                    const int32_t* __restrict__ col, const float* __restrict__ mult,
                                                    const float* __restrict__ p, const float* __restrict__ q, float slope,
                                                    float* __restrict__ w, float* __restrict__ m_row, float* __restrict__ zinv,
                                                    float* __restrict__ part_m, float* __restrict__ part_s) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t t = (int64_t)blockIdx.x * 4 + wave;
  if (t >= n_items) return;
  const WorkItem it = items[t];
  const uint32_t r = it.row;
  const int32_t len = it.len, part = it.part;
  const int64_t e0 = it.e0;
  w -= ent0;
  const float pv = p[r];
  float m = -3.0e38f, s = 0.f;
  if (len <= 64 * SCORE_REGS) {   // the entries' scores stay in registers between the two sums, and their loads are on the way together
    int32_t c[SCORE_REGS];
    float x[SCORE_REGS], w_e[SCORE_REGS];
#pragma unroll
    for (int j = 0; j < SCORE_REGS; ++j) {
      const int32_t k = j * 64 + lane;
      c[j] = k < len ? col[e0 + k] : -1;
      w_e[j] = k < len && mult ? mult[e0 + k] : 1.f;
    }
#pragma unroll
    for (int j = 0; j < SCORE_REGS; ++j) x[j] = c[j] >= 0 ? q[c[j]] : 0.f;
#pragma unroll
    for (int j = 0; j < SCORE_REGS; ++j) {
      if (c[j] < 0) continue;
      x[j] = lrelu(pv + x[j], slope);
      w[e0 + j * 64 + lane] = x[j];
      m = fmaxf(m, x[j]);
    }
    m = wave_max(m);
#pragma unroll
    for (int j = 0; j < SCORE_REGS; ++j)
      if (c[j] >= 0) s += w_e[j] * expf(x[j] - m);
  } else {
    for (int32_t k = lane; k < len; k += 64) {
      const float x = lrelu(pv + q[col[e0 + k]], slope);
      w[e0 + k] = x;
      m = fmaxf(m, x);
    }
    m = wave_max(m);
    for (int32_t k = lane; k < len; k += 64) s += (mult ? mult[e0 + k] : 1.f) * expf(w[e0 + k] - m);
  }
  s = wave_sum(s);
  if (lane == 0) {
    if (part >= 0) {
      part_m[part - part0] = m;
      part_s[part - part0] = s;
    } else {
      m_row[r] = m;
      zinv[r] = s > 0.f ? 1.f / s : 0.f;
    }
  }
}

__global__ void __launch_bounds__(256) k_gat_rowstats(const CutRow* __restrict__ cuts, int64_t n_cut, int64_t part0,
                                                      const float* __restrict__ part_m, const float* __restrict__ part_s,
                                                      float* __restrict__ m_row, float* __restrict__ zinv) {
  // a wave per cut row; lanes take the row's items 64 apart, lane sums are added in lane order
  const int lane = threadIdx.x & 63;
  const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (f >= n_cut) return;
  const CutRow cut = cuts[f];
  const int64_t p0 = cut.part0 - part0;
  const int32_t ns = cut.nseg;
  float m = -3.0e38f;
  for (int32_t k = lane; k < ns; k += 64) m = fmaxf(m, part_m[p0 + k]);
  m = wave_max(m);
  float s = 0.f;
  for (int32_t k = lane; k < ns; k += 64) s += part_s[p0 + k] * expf(part_m[p0 + k] - m);
  s = wave_sum(s);
  if (lane == 0) {
    m_row[cut.row] = m;
    zinv[cut.row] = s > 0.f ? 1.f / s : 0.f;
  }
}

// The weighted sums over the in-edges of a row, the coefficients made on the way from the scores x_e that k_gat_scores left:
//   AGG_Z: z_v = sum w_e t_u;   AGG_ZQ: also Q_v = sum w_e f_e t_u and r_v = sum w_e f_e (f_e = LeakyReLU'(y_e));   AGG_Q: Q, r
// What bounds it is the gather of the rows of t (the slab split is that of the GCN aggregation, for its reasons); the second sum
// of the same rows costs four fused multiply-adds per loaded float4, where a pass of its own costs the gather again, and the
// exponential of an entry costs less than the kernel that wrote the coefficients and the read of them did (233 k vertices, 115 M
// edges, widths 256 and 41: forward, coefficients and destination pass 12.3 ms per epoch as passes of their own, 6.0 ms here).
struct GatAgg {
  const WorkItem* items; int64_t n_items; int64_t ent0, part0, row0;
  const int32_t* col; const float* mult;      // per entry of the graph
  const float* x;                             // scores, the first one for entry ent0
  const float* m; const float* zinv;          // per vertex
  float slope;
  const float* T; int64_t ld; int d;
  float* z; int64_t z_ld; float* z_part; int relu;    // row r - row0
  float* Q; int64_t q_ld; float* q_part;
  float* r; float* r_part;                    // per vertex; per partial sum
};
enum { AGG_Z = 0, AGG_ZQ = 1, AGG_Q = 2 };

template <bool UNI, int MODE>
__global__ void __launch_bounds__(256) k_gat_agg(GatAgg a, int S, int nvs, int eps, int64_t grp_per_part, int slab0) {
  constexpr int U = 4;
  constexpr bool Z = MODE != AGG_Q, Q = MODE != AGG_Z;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int xcd = blockIdx.x & 7;
  const int slab = slab0 + xcd % S;
  const int64_t i = blockIdx.x >> 3;
  if (grp_per_part > 0 && i >= grp_per_part) return;
  const int64_t grp = grp_per_part > 0 ? (int64_t)(xcd / S) * grp_per_part + i : i * (8 / S) + xcd / S;
  const int64_t t = grp * 4 + wave;
  if (t >= a.n_items) return;
  const int nvec = (a.d + 3) >> 2;
  const int v0 = slab * nvs;
  const int nv_here = (nvec - v0) < nvs ? (nvec - v0) : nvs;
  if (nv_here <= 0) return;
  const WorkItem it = a.items[t];
  const uint32_t row = it.row;
  const int32_t len = it.len;
  const int64_t e0 = it.e0;
  const int es = lane / nvs, vec = lane - es * nvs;
  const bool active = es < eps && vec < nv_here;
  const int coff = (v0 + vec) * 4;
  const float* srcc = a.T + coff;
  const float m = a.m[row], zinv = a.zinv[row];
  const float* xs = a.x - a.ent0;
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 acc = zero, G = zero;
  float rs = 0.f;
  for (int32_t base = 0; base < len; base += 64) {
    const int32_t nh = (len - base) < 64 ? (len - base) : 64;
    int32_t my_u = 0;
    float my_c = 0.f, my_cf = 0.f;
    if (lane < nh) {
      const int64_t e = e0 + base + lane;
      my_u = a.col[e];
      const float x = xs[e];           // the score LeakyReLU(y_e): same sign as y_e
      my_c = (a.mult ? a.mult[e] : 1.f) * expf(x - m) * zinv;
      my_cf = my_c * (x > 0.f ? 1.f : a.slope);
      if (Q) rs += my_cf;
    }
    const int step = UNI ? U : U * eps;
    for (int32_t k = 0; k < nh; k += step) {
      int32_t c[U];
      float w[U], wf[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int kk = UNI ? k + u : k + u * eps + es;
        const int kc = kk < nh ? kk : (nh - 1);     // past the end: the last entry again with weight 0
        if (UNI) {
          c[u] = __builtin_amdgcn_readlane(my_u, kc);
          if (Z) w[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_c), kc));
          if (Q) wf[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_cf), kc));
        } else {
          c[u] = __shfl(my_u, kc, 64);
          if (Z) w[u] = __shfl(my_c, kc, 64);
          if (Q) wf[u] = __shfl(my_cf, kc, 64);
        }
        if (kk >= nh) w[u] = wf[u] = 0.f;
      }
      if (active) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ld4(srcc + (int64_t)c[u] * a.ld);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (Z) acc = fma4(w[u], v[u], acc);
          if (Q) G = fma4(wf[u], v[u], G);
        }
      }
    }
  }
  // the sum of a row's edge slots, the upper half added to the lower one until slot 0 holds the result (one after the other, 31
  // additions at 7 columns: 20 k vertices, 300 k edges, 33 and 7 columns, 43 -> 20 us per launch)
  auto slots = [&](float4 tot) {
    for (int n = eps; n > 1;) {
      const int h = (n + 1) >> 1, from = (lane + h * nvs) & 63;
      const float4 o = make_float4(__shfl(tot.x, from, 64), __shfl(tot.y, from, 64), __shfl(tot.z, from, 64), __shfl(tot.w, from, 64));
      if (es + h < n) tot = make_float4(tot.x + o.x, tot.y + o.y, tot.z + o.z, tot.w + o.w);
      n = h;
    }
    return tot;
  };
  if (Z) acc = slots(acc);
  if (Q) {
    G = slots(G);
    if (slab == 0) {
      rs = wave_sum(rs);
      if (lane == 0) {
        if (it.part >= 0) a.r_part[it.part - a.part0] = rs;
        else a.r[row] = rs;
      }
    }
  }
  if (es != 0 || vec >= nv_here) return;
  if (it.part >= 0) {
    if (Z) st4(a.z_part + (it.part - a.part0) * a.z_ld + coff, acc);
    if (Q) st4(a.q_part + (it.part - a.part0) * a.q_ld + coff, G);
  } else {
    if (Z) {
      if (a.relu) acc = make_float4(acc.x > 0.f ? acc.x : 0.f, acc.y > 0.f ? acc.y : 0.f, acc.z > 0.f ? acc.z : 0.f, acc.w > 0.f ? acc.w : 0.f);
      st4(a.z + (row - a.row0) * a.z_ld + coff, acc);
    }
    if (Q) st4(a.Q + (row - a.row0) * a.q_ld + coff, G);
  }
}

// Over the rows of a range, lpr lanes per row: dz = dh * [h > 0] (or dh), pad columns zero; S_v = dz_v . h_v;
// dp_v = dz_v . Q_v - S_v r_v; d4[row] = (p_v, m_v, 1/Z_v, S_v).  (p, m, zinv, r, dp point at the range's first row.)
__global__ void __launch_bounds__(256) k_gat_dz(const float* __restrict__ dh, int64_t ld_dh, const float* __restrict__ h,
                                                int64_t ld_h, int relu, int64_t rows, int d, float* __restrict__ dz,
                                                const float* __restrict__ Q, int64_t ld, const float* __restrict__ p,
                                                const float* __restrict__ m, const float* __restrict__ zinv,
                                                const float* __restrict__ r, float* __restrict__ dp, float* __restrict__ d4, int lpr) {
  const int rpb = 256 / lpr, ll = threadIdx.x % lpr;
  for (int64_t v = (int64_t)blockIdx.x * rpb + threadIdx.x / lpr; v < rows; v += (int64_t)gridDim.x * rpb) {
    float S = 0.f, dq = 0.f;
    for (int c = ll * 4; c < (int)ld; c += lpr * 4) {
      float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
      if (c < d) {   // (rows are pitched to a multiple of 4: pads are read and dropped)
        float4 hv = ld4(h + v * ld_h + c), qv = ld4(Q + v * ld + c);
        g = ld4(dh + v * ld_dh + c);
        if (c + 1 >= d) hv.y = qv.y = g.y = 0.f;
        if (c + 2 >= d) hv.z = qv.z = g.z = 0.f;
        if (c + 3 >= d) hv.w = qv.w = g.w = 0.f;
        if (relu) {
          if (!(hv.x > 0.f)) g.x = 0.f;
          if (!(hv.y > 0.f)) g.y = 0.f;
          if (!(hv.z > 0.f)) g.z = 0.f;
          if (!(hv.w > 0.f)) g.w = 0.f;
        }
        S = dot4(g, hv, S);
        dq = dot4(g, qv, dq);
      }
      st4(dz + v * ld + c, g);
    }
    S = group_sum(S, lpr);
    dq = group_sum(dq, lpr);
    if (ll == 0) {
      dp[v] = dq - S * r[v];
      // what the source pass needs of a destination, in one 16-byte read per entry instead of four 4-byte ones
      st4(d4 + v * 4, make_float4(p[v], m[v], zinv[v], S));
    }
  }
}

struct GatPass {
  // items of the source pass (rows = local sources of a chunk, or vertices)
  const WorkItem* items; int64_t n_items; int64_t part0;
  const int32_t* idx;        // per entry: row of `mat` to read (destination of the chunk, or vertex)
  const float* mult;         // multiplicity per entry (nullable: 1)
  const float* mat;          // rows gathered per entry: dz
  int64_t mat_ld;
  const float* own;          // the item's own row: t
  int64_t own_ld;
  const int32_t* own_idx;    // row r -> row of `own` and of `out` (nullable: r)
  int d;
  const float* q;            // per vertex
  const float* d4;           // per row of `mat`: (p_v, m_v, 1/Z_v, S_v), from which the coefficients are recomputed
  float slope;
  // outputs
  float* out; int64_t out_ld;  // dt rows, scalar in column sc_col
  bool add;                    // out is added to
  float* partial;            // [n_part x out_ld] partial rows of cut items
  int sc_col;
};

// Cut rows of k_gat_agg: the partial sums of z, Q and r added in item order, a block per row (each wave a contiguous quarter)
__global__ void __launch_bounds__(256) k_gat_fix(GatAgg a, const CutRow* __restrict__ cuts, int mode) {
  __shared__ float4 sh[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const CutRow cut = cuts[blockIdx.x];
  const int64_t p0 = cut.part0 - a.part0;
  const int32_t ns = cut.nseg, per = (ns + 3) >> 2;
  const int32_t k0 = wave * per, k1 = (k0 + per) < ns ? (k0 + per) : ns;
  const int d4 = (a.d + 3) & ~3;
  auto rows = [&](const float* part, int64_t ld, float* out, bool relu) {
    for (int cb = 0; cb < d4; cb += 256) {
      const int c4 = cb + lane * 4;
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
      if (c4 < d4) {
        const float* p = part + p0 * ld + c4;
#pragma unroll 4
        for (int32_t k = k0; k < k1; ++k) {
          const float4 v = ld4(p + (int64_t)k * ld);
          s = make_float4(s.x + v.x, s.y + v.y, s.z + v.z, s.w + v.w);
        }
      }
      sh[wave][lane] = s;
      __syncthreads();
      if (wave == 0 && c4 < d4) {
        for (int q = 1; q < 4; ++q) {
          const float4 v = sh[q][lane];
          s = make_float4(s.x + v.x, s.y + v.y, s.z + v.z, s.w + v.w);
        }
        if (relu) s = make_float4(s.x > 0.f ? s.x : 0.f, s.y > 0.f ? s.y : 0.f, s.z > 0.f ? s.z : 0.f, s.w > 0.f ? s.w : 0.f);
        st4(out + (cut.row - a.row0) * ld + c4, s);
      }
      __syncthreads();
    }
  };
  if (mode != AGG_Q) rows(a.z_part, a.z_ld, a.z, a.relu != 0);
  if (mode == AGG_Z) return;
  rows(a.q_part, a.q_ld, a.Q, false);
  if (wave == 0) {
    float s = 0.f;
    for (int32_t k = lane; k < ns; k += 64) s += a.r_part[p0 + k];
    s = wave_sum(s);
    if (lane == 0) a.r[cut.row] = s;
  }
}

// Source pass: for local source i (vertex u) over its entries (u -> v) of the chunk, w_e recomputed:
//   dt_u += sum_e w_e dz_v
//   dq_u += sum_e w_e f_e (dz_v . t_u - S_v) = t_u . (sum_e w_e f_e dz_v) - sum_e w_e f_e S_v
// i.e. two aggregations of the same gathered rows of dz and one dot product per item.
template <int VPL>
__global__ void __launch_bounds__(256) k_gat_src(GatPass a) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t t = (int64_t)blockIdx.x * 4 + wave;
  if (t >= a.n_items) return;
  const WorkItem it = a.items[t];
  const uint32_t r = it.row;
  const int64_t e0 = it.e0;
  const int32_t len = it.len, part = it.part;
  const int32_t u_id = a.own_idx ? a.own_idx[r] : (int32_t)r;
  float4 acc[VPL], G[VPL];
#pragma unroll
  for (int j = 0; j < VPL; ++j) acc[j] = G[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  const float qu = a.q[u_id];
  float csum = 0.f;
  for (int32_t base = 0; base < len; base += 64) {
    const int32_t nh = (len - base) < 64 ? (len - base) : 64;
    int32_t my_v = 0;
    float my_c = 0.f, my_cf = 0.f, my_cs = 0.f;   // w_e, w_e f_e, w_e f_e S_v of the lane's entry
    if (lane < nh) {
      my_v = a.idx[e0 + base + lane];
      const float4 dv = ld4(a.d4 + (int64_t)my_v * 4);
      const float y = dv.x + qu;
      my_c = coef(y, a.slope, dv.y, dv.z, a.mult ? a.mult[e0 + base + lane] : 1.f);
      my_cf = my_c * (y > 0.f ? 1.f : a.slope);
      my_cs = my_cf * dv.w;
    }
    csum += wave_sum(my_cs);
    for (int32_t k = 0; k < nh; k += 4) {
      int32_t c[4];
      float w[4], wf[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int kc = (k + u) < nh ? (k + u) : (nh - 1);
        c[u] = __builtin_amdgcn_readlane(my_v, kc);
        w[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_c), kc));
        wf[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_cf), kc));
        if (k + u >= nh) w[u] = wf[u] = 0.f;
      }
      float4 x[4][VPL];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
          const int cc = (j * 64 + lane) * 4;
          x[u][j] = cc < a.d ? ld4(a.mat + (int64_t)c[u] * a.mat_ld + cc) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
          acc[j].x = fmaf(w[u], x[u][j].x, acc[j].x);
          acc[j].y = fmaf(w[u], x[u][j].y, acc[j].y);
          acc[j].z = fmaf(w[u], x[u][j].z, acc[j].z);
          acc[j].w = fmaf(w[u], x[u][j].w, acc[j].w);
          G[j].x = fmaf(wf[u], x[u][j].x, G[j].x);
          G[j].y = fmaf(wf[u], x[u][j].y, G[j].y);
          G[j].z = fmaf(wf[u], x[u][j].z, G[j].z);
          G[j].w = fmaf(wf[u], x[u][j].w, G[j].w);
        }
    }
  }
  float s = 0.f;
  float* row = part >= 0 ? a.partial + (part - a.part0) * a.out_ld : a.out + (int64_t)u_id * a.out_ld;
#pragma unroll
  for (int j = 0; j < VPL; ++j) {
    const int c = (j * 64 + lane) * 4;
    if (c >= a.d) continue;
    const float4 mine = ld4(a.own + (int64_t)u_id * a.own_ld + c);   // pads of t are zero
    s = fmaf(mine.x, G[j].x, fmaf(mine.y, G[j].y, fmaf(mine.z, G[j].z, fmaf(mine.w, G[j].w, s))));
    float4 v = acc[j];
    if (part < 0 && a.add) {
      const float4 o = ld4(row + c);
      v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
    }
    st4(row + c, v);
  }
  s = wave_sum(s);
  if (lane == 0) {
    // the scalar travels in its own float4 column block behind the data columns
    float4 sc = make_float4(s - csum, 0.f, 0.f, 0.f);
    if (part < 0 && a.add) sc.x += row[a.sc_col];
    st4(row + a.sc_col, sc);
  }
}

template <int G_>
__global__ void __launch_bounds__(256) k_gat_src_g(GatPass a) {
  constexpr int NG = 64 / G_;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t t = (int64_t)blockIdx.x * 4 + wave;
  if (t >= a.n_items) return;
  const WorkItem it = a.items[t];
  const uint32_t r = it.row;
  const int64_t e0 = it.e0;
  const int32_t len = it.len, part = it.part;
  const int32_t u_id = a.own_idx ? a.own_idx[r] : (int32_t)r;
  const int grp = lane / G_, c4 = (lane % G_) * 4;
  const bool has = c4 < a.d;
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 acc = zero, G = zero;
  const float qu = a.q[u_id];
  float csum = 0.f;
  for (int32_t base = 0; base < len; base += 64) {
    const int32_t nh = (len - base) < 64 ? (len - base) : 64;
    int32_t my_v = 0;
    float my_c = 0.f, my_cf = 0.f, my_cs = 0.f;
    if (lane < nh) {
      my_v = a.idx[e0 + base + lane];
      const float4 dv = ld4(a.d4 + (int64_t)my_v * 4);
      const float y = dv.x + qu;
      my_c = coef(y, a.slope, dv.y, dv.z, a.mult ? a.mult[e0 + base + lane] : 1.f);
      my_cf = my_c * (y > 0.f ? 1.f : a.slope);
      my_cs = my_cf * dv.w;
    }
    csum += wave_sum(my_cs);
    for (int32_t k = 0; k < nh; k += 4 * NG) {
      float4 x[4];
      float w[4], wf[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int ent = k + u * NG + grp;
        const int kc = ent < nh ? ent : (nh - 1);
        const int32_t c = __shfl(my_v, kc, 64);
        w[u] = __shfl(my_c, kc, 64);
        wf[u] = __shfl(my_cf, kc, 64);
        if (ent >= nh) w[u] = wf[u] = 0.f;
        x[u] = has ? ld4(a.mat + (int64_t)c * a.mat_ld + c4) : zero;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        acc.x = fmaf(w[u], x[u].x, acc.x);
        acc.y = fmaf(w[u], x[u].y, acc.y);
        acc.z = fmaf(w[u], x[u].z, acc.z);
        acc.w = fmaf(w[u], x[u].w, acc.w);
        G.x = fmaf(wf[u], x[u].x, G.x);
        G.y = fmaf(wf[u], x[u].y, G.y);
        G.z = fmaf(wf[u], x[u].z, G.z);
        G.w = fmaf(wf[u], x[u].w, G.w);
      }
    }
  }
#pragma unroll
  for (int o = G_; o < 64; o <<= 1) {
    acc.x += __shfl_xor(acc.x, o, 64);
    acc.y += __shfl_xor(acc.y, o, 64);
    acc.z += __shfl_xor(acc.z, o, 64);
    acc.w += __shfl_xor(acc.w, o, 64);
  }
  float s = 0.f;
  float* row = part >= 0 ? a.partial + (part - a.part0) * a.out_ld : a.out + (int64_t)u_id * a.out_ld;
  if (has) {
    const float4 mine = ld4(a.own + (int64_t)u_id * a.own_ld + c4);
    s = fmaf(mine.x, G.x, fmaf(mine.y, G.y, fmaf(mine.z, G.z, mine.w * G.w)));
    if (grp == 0) {
      float4 v = acc;
      if (part < 0 && a.add) {
        const float4 o = ld4(row + c4);
        v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
      }
      st4(row + c4, v);
    }
  }
  s = wave_sum(s);
  if (lane == 0) {
    float4 sc = make_float4(s - csum, 0.f, 0.f, 0.f);
    if (part < 0 && a.add) sc.x += row[a.sc_col];
    st4(row + a.sc_col, sc);
  }
}

// dt_v += dp_v a_dst + dq_v a_src; the pair (dp_v, dq_v) also goes to a [V x 4] matrix for da = T^T [dp dq]
__global__ void __launch_bounds__(256) k_gat_finish(float* __restrict__ dT, int64_t ld, int d, int sc_col,
                                                    const float* __restrict__ dp, const float* __restrict__ a_dst,
                                                    const float* __restrict__ a_src, int64_t V, float* __restrict__ pq4, int lpr) {
  __shared__ AttVec sa;
  load_att(sa, a_dst, a_src, d);
  const int rpb = 256 / lpr, ll = threadIdx.x % lpr;
  for (int64_t v = (int64_t)blockIdx.x * rpb + threadIdx.x / lpr; v < V; v += (int64_t)gridDim.x * rpb) {
    const float dpv = dp[v], dqv = dT[v * ld + sc_col];
    for (int c = ll * 4; c < d; c += lpr * 4) {
      float4 t = ld4(dT + v * ld + c);
      const float4 ad = sa.dst[c >> 2], as = sa.src[c >> 2];
      t.x += dpv * ad.x + dqv * as.x;
      t.y += dpv * ad.y + dqv * as.y;
      t.z += dpv * ad.z + dqv * as.z;
      t.w += dpv * ad.w + dqv * as.w;
      st4(dT + v * ld + c, t);
    }
    if (ll == 0) st4(pq4 + v * 4, make_float4(dpv, dqv, 0.f, 0.f));
  }
}

__global__ void k_gat_split(const float* __restrict__ da4, int d, float* __restrict__ da_dst, float* __restrict__ da_src) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < d) {
    da_dst[c] = da4[c * 4 + 0];
    da_src[c] = da4[c * 4 + 1];
  }
}

// What a layer's forward pass leaves for its backward pass inside one epoch: t, the scores' halves, the softmax's row values, and
// the sums that dp needs (Q, r).  Without it the backward pass makes all of this again.
struct GatKeep {
  float *T = nullptr, *Q = nullptr, *p = nullptr, *q = nullptr, *m = nullptr, *zinv = nullptr, *r = nullptr;
};

struct GatWs {
  float *T, *p, *q, *m, *zinv, *dp, *r, *pq4, *d4;
  int64_t ld_t;
};

// A contiguous range of chunks in vertex order that runs as one set of launches.
struct GatRange {
  ItemRange it;
  int64_t ent0, n_ent, row0, rows;
};
GatRange range_of(const ht_graph* g, const ChunkMeta& c) {
  return GatRange{c.fwd, c.ue0, g->merged ? c.nu : c.nnz, c.dst0, c.dst1 - c.dst0};
}
// Scratch memory of one range (scores, partial sums), and of a backward pass that holds dz and Q of all vertices; what an epoch
// keeps between its passes.  Beyond these the passes go chunk by chunk, and the backward pass recomputes.
constexpr int64_t GAT_RANGE_BYTES = (int64_t)4 << 30, GAT_DIRECT_BYTES = (int64_t)8 << 30, GAT_KEEP_BYTES = (int64_t)16 << 30;
// Chunks that follow each other in vertex order share a range while its scores (4 bytes per entry) and partial sums
// (part_bytes each) stay below the cap: what a launch per chunk costs is in the launches and in the last waves of each
// (20,011 vertices in 3 chunks: 861 -> 458 us per epoch; 233 k vertices, 115 M edges in 8: 26.0 -> 16.2 ms, the sums kept for
// the backward pass included).
std::vector<GatRange> ranges_of(const ht_graph* g, int64_t part_bytes, bool merge) {
  std::vector<GatRange> out;
  for (int k = 0; k < g->n; ++k) {
    const GatRange c = range_of(g, g->chunks[g->pos[k]]);
    if (c.rows == 0) continue;
    if (merge && !out.empty()) {
      GatRange& r = out.back();
      if ((r.n_ent + c.n_ent) * 4 + (r.it.n_part + c.it.n_part) * part_bytes <= GAT_RANGE_BYTES) {
        r.it.n_items += c.it.n_items;
        r.it.n_part += c.it.n_part;
        r.it.n_cut += c.it.n_cut;
        r.n_ent += c.n_ent;
        r.rows += c.rows;
        continue;
      }
    }
    out.push_back(c);
  }
  return out;
}
// Scratch memory for any of these ranges: scores, partial sums of the softmax and of z and Q (pitches z_ld, q_ld; 0: no such sum).
struct RangeWs {
  float *x = nullptr, *part = nullptr, *z_part = nullptr, *q_part = nullptr;
  int64_t n_part = 0;
};
// what range_ws will ask for
void range_wants(const std::vector<GatRange>& ranges, int64_t ld, std::vector<ScratchWant>* want) {
  int64_t ent = 1, parts = 0;
  for (const GatRange& r : ranges) {
    ent = std::max(ent, r.n_ent);
    parts = std::max(parts, r.it.n_part);
  }
  want->push_back({HT_S_GATE, (size_t)ent * 4});
  want->push_back({HT_S_GATP, (size_t)parts * 3 * 4});
  want->push_back({HT_S_SPART, (size_t)(parts * ld) * 4});
}
int range_ws(ht_ctx* ctx, const std::vector<GatRange>& ranges, int64_t z_ld, int64_t q_ld, RangeWs* ws) {
  int64_t ent = 1;
  ws->n_part = 0;
  for (const GatRange& r : ranges) {
    ent = std::max(ent, r.n_ent);
    ws->n_part = std::max(ws->n_part, r.it.n_part);
  }
  HT_TRY(ht_scratch(ctx, HT_S_GATE, (size_t)ent * 4, (void**)&ws->x));
  if (ws->n_part == 0) return HT_OK;
  HT_TRY(ht_scratch(ctx, HT_S_GATP, (size_t)ws->n_part * 3 * 4, (void**)&ws->part));
  HT_TRY(ht_scratch(ctx, HT_S_SPART, (size_t)(ws->n_part * (z_ld + q_ld)) * 4, (void**)&ws->z_part));
  ws->q_part = ws->z_part + ws->n_part * z_ld;
  return HT_OK;
}

// Contiguous row ranges between pinned host memory and staging pairs in HBM: copies run on the
// side streams, the compute stream waits for the block it needs and frees the block it has read.
struct Link {
  ht_ctx* ctx;
  ht_stats* st;
  Timer* tm;
  hipStream_t s_c, s_in, s_out;
  hipEvent_t last_out = nullptr;
  bool used = false;
  Link(ht_ctx* c, ht_stats* s, Timer* t) : ctx(c), st(s), tm(t), s_c(c->stream), s_in(c->side[0]), s_out(c->side[1]) {}
  // A failed call must not leave side-stream work that refers to the caller's buffers.
  ~Link() {
    if (used) {
      (void)hipStreamSynchronize(s_in);
      (void)hipStreamSynchronize(s_out);
    }
  }
  int rec(hipStream_t s, hipEvent_t* out) {
    hipEvent_t e = ht_event(ctx);
    if (!e) return ht_set_err(ctx, HT_EHIP, "hipEventCreate failed");
    HT_HIP(ctx, hipEventRecord(e, s));
    *out = e;
    return HT_OK;
  }
  int wait(hipStream_t s, hipEvent_t e) {
    if (e) HT_HIP(ctx, hipStreamWaitEvent(s, e, 0));
    return HT_OK;
  }
  // the side streams start behind everything the compute stream has been given so far
  int fork() {
    hipEvent_t e = nullptr;
    HT_TRY(rec(s_c, &e));
    HT_TRY(wait(s_in, e));
    HT_TRY(wait(s_out, e));
    used = true;
    return HT_OK;
  }
  // the compute stream continues behind every store to the host
  int join() {
    HT_TRY(wait(s_c, last_out));
    hipEvent_t e = nullptr;
    HT_TRY(rec(s_in, &e));
    return wait(s_c, e);
  }
  int copy(hipStream_t s, void* dst, const void* src, size_t bytes, bool to_host) {
    if (bytes == 0) return HT_OK;
    const int id = tm->begin_on(&st->t_copy_ms, s);
    if (ctx->link_memcpy) {
      HT_HIP(ctx, hipMemcpyAsync(dst, src, bytes, to_host ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice, s));
    } else {
      void* mapped = nullptr;
      HT_HIP(ctx, hipHostGetDevicePointer(&mapped, to_host ? dst : const_cast<void*>(src), 0));
      HT_TRY(ht_copy_link(ctx, s, to_host ? mapped : dst, to_host ? src : mapped, bytes, ctx->link_blocks));
    }
    tm->end_id(id);
    (to_host ? st->bytes_d2h : st->bytes_h2d) += (int64_t)bytes;
    return HT_OK;
  }
};

inline bool on_host(const ht_tensor* t) { return t && t->loc == HT_LOC_HOST_PINNED; }

int check(ht_ctx* ctx, const ht_graph* g, const ht_gat_desc* desc, const ht_tensor* t, int32_t cols, const char* name) {
  if (!t || !t->ptr) return ht_set_err(ctx, HT_EINVAL, "%s: null tensor", name);
  if (t->rows != g->V || t->cols != cols) return ht_set_err(ctx, HT_ESHAPE, "%s: expected [%lld x %d]", name, (long long)g->V, cols);
  if (t->ld < cols || (t->ld & 3) || ((uintptr_t)t->ptr & 15)) return ht_set_err(ctx, HT_ESHAPE, "%s: bad pitch or alignment", name);
  if (t->loc != HT_LOC_DEVICE && t->loc != HT_LOC_HOST_PINNED) return ht_set_err(ctx, HT_ESHAPE, "%s: unknown location", name);
  (void)desc;
  return HT_OK;
}

int check_desc(ht_ctx* ctx, const ht_gat_desc* d) {
  if (d->d_in <= 0 || d->d_out <= 0) return ht_set_err(ctx, HT_ESHAPE, "layer widths must be positive");
  if (d->d_out > 1024) return ht_set_err(ctx, HT_ESHAPE, "GAT layer: d_out %d > 1024", d->d_out);
  if (d->act != HT_ACT_NONE && d->act != HT_ACT_RELU) return ht_set_err(ctx, HT_EINVAL, "unknown activation %d", d->act);
  if (!(d->slope >= 0.f && d->slope <= 1.f)) return ht_set_err(ctx, HT_EINVAL, "LeakyReLU slope must lie in [0, 1]");
  return HT_OK;
}

int bind_ws(ht_ctx* ctx, const ht_graph* g, int d_out, const GatKeep* keep, GatWs* ws) {
  const int64_t V = std::max<int64_t>(g->V, 1);
  ws->ld_t = ht_row_pitch(d_out, true);
  if (keep) ws->T = keep->T;
  else HT_TRY(ht_scratch(ctx, HT_S_TFULL, (size_t)V * ws->ld_t * 4, (void**)&ws->T));
  float* vec = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_GATV, (size_t)V * 16 * 4, (void**)&vec));
  ws->p = vec; ws->q = vec + V; ws->m = vec + 2 * V; ws->zinv = vec + 3 * V; ws->dp = vec + 4 * V;
  ws->r = vec + 5 * V;
  ws->pq4 = vec + 8 * V;      // 16-byte aligned whatever V is
  ws->d4 = vec + 12 * V;
  if (keep) { ws->p = keep->p; ws->q = keep->q; ws->m = keep->m; ws->zinv = keep->zinv; ws->r = keep->r; }
  return HT_OK;
}

// t = H W (pad columns that are read zero), p, q
constexpr int64_t BLOCK_HBM = (int64_t)1 << 22;    // rows per GEMM call

int prepare(ht_ctx* ctx, const ht_graph* g, const ht_gat_desc* desc, const ht_tensor* H, const float* W, const float* a_dst,
            const float* a_src, const GatWs* ws, ht_stats* st, Timer* tm, Link* lk) {
  hipStream_t s = ctx->stream;
  const int64_t V = std::max<int64_t>(g->V, 1);
  const bool host = on_host(H);
  const int64_t step = host ? ctx->link_block_rows : BLOCK_HBM;   // rows per staged block / per GEMM call
  float* stage[2] = {nullptr, nullptr};
  hipEvent_t ev_free[2] = {nullptr, nullptr};
  if (host) {
    const int64_t rows = std::min<int64_t>(step, V);
    HT_TRY(ht_scratch(ctx, HT_S_LINK0, (size_t)rows * H->ld * 4 * 2, (void**)&stage[0]));
    stage[1] = stage[0] + rows * H->ld;
  }
  int k = 0;
  for (int64_t r0 = 0; r0 < g->V; r0 += step, ++k) {
    const int64_t nr = std::min(step, g->V - r0);
    const float* rows = H->ptr + r0 * H->ld;
    const int b = k & 1;
    if (host) {
      hipEvent_t ev_in = nullptr;
      HT_TRY(lk->wait(lk->s_in, ev_free[b]));
      HT_TRY(lk->copy(lk->s_in, stage[b], rows, (size_t)nr * H->ld * 4, false));
      HT_TRY(lk->rec(lk->s_in, &ev_in));
      HT_TRY(lk->wait(s, ev_in));
      rows = stage[b];
    }
    tm->begin(&st->t_gemm_ms);
    HT_TRY(ht_gemm_nn(ctx, s, rows, H->ld, W, ws->T + r0 * ws->ld_t, ws->ld_t, nr, desc->d_in, desc->d_out, 0));
    tm->end();
    if (host) HT_TRY(lk->rec(s, &ev_free[b]));
    st->n_gemm += 1;
    st->gemm_flops += 2.0 * nr * desc->d_in * desc->d_out;
  }
  if (g->V > 0) {
    const int lpr = row_lanes(ws->ld_t);
    k_gat_pq<<<row_grid(g->V, lpr), 256, 0, s>>>(ws->T, ws->ld_t, desc->d_out, a_dst, a_src, g->V, ws->p, ws->q, lpr);
    HT_LAUNCH_CHECK(ctx);
  }
  return HT_OK;
}

// Scores, row maxima and 1 / Z of a range (a row without an in-edge has an item of no entries: 1 / Z = 0).
int softmax_range(ht_ctx* ctx, const ht_graph* g, const GatRange& r, const ht_gat_desc* desc, const GatWs& ws, const RangeWs& rw,
                  ht_stats* st, Timer* tm) {
  const ItemRange& it = r.it;
  if (it.n_items == 0) return HT_OK;
  float* part_s = rw.part ? rw.part + rw.n_part : nullptr;
  tm->begin(&st->t_gat_softmax_ms);
  HT_TRY(ht_in_launches(it.n_items, HT_LAUNCH_WAVES, [&](int64_t i, int64_t n) {
    k_gat_scores<<<(unsigned)((n + 3) / 4), 256, 0, ctx->stream>>>(
        g->fwd_items.items.p + it.it0 + i, n, r.ent0, it.part0, g->merged ? g->ucol.p : g->col.p, g->merged ? g->umult.p : nullptr,
        ws.p, ws.q, desc->slope, rw.x, ws.m, ws.zinv, rw.part, part_s);
    HT_LAUNCH_CHECK(ctx);
    return (int)HT_OK;
  }));
  HT_TRY(ht_in_launches(it.n_cut, HT_LAUNCH_WAVES, [&](int64_t i, int64_t n) {
    k_gat_rowstats<<<(unsigned)((n + 3) / 4), 256, 0, ctx->stream>>>(g->fwd_items.cuts.p + it.cut0 + i, n, it.part0, rw.part, part_s,
                                                                     ws.m, ws.zinv);
    HT_LAUNCH_CHECK(ctx);
    return (int)HT_OK;
  }));
  tm->end();
  return HT_OK;
}

template <bool UNI>
void launch_agg(hipStream_t st, int mode, const GatAgg& a, const SlabShape& sh, int slab0) {
  int64_t gpp;
  const unsigned blocks = sh.grid(a.n_items, &gpp);
  if (mode == AGG_Z) k_gat_agg<UNI, AGG_Z><<<blocks, 256, 0, st>>>(a, sh.S, sh.nvs, sh.eps, gpp, slab0);
  else if (mode == AGG_ZQ) k_gat_agg<UNI, AGG_ZQ><<<blocks, 256, 0, st>>>(a, sh.S, sh.nvs, sh.eps, gpp, slab0);
  else k_gat_agg<UNI, AGG_Q><<<blocks, 256, 0, st>>>(a, sh.S, sh.nvs, sh.eps, gpp, slab0);
}

// The sums of a range out of its scores: z (row 0 = the range's first row; relu) and / or Q (row 0 likewise) and r.
int agg_range(ht_ctx* ctx, const ht_graph* g, const GatRange& rg, const ht_gat_desc* desc, const GatWs& ws, const RangeWs& rw, int mode,
              float* z, int64_t z_ld, float* Q, double* t_items, double* t_fix, Timer* tm) {
  const ItemRange& it = rg.it;
  if (it.n_items == 0) return HT_OK;
  hipStream_t st = ctx->stream;
  SpmmArgs s{};
  s.n_items = it.n_items; s.n_edges = rg.n_ent; s.src = ws.T; s.src_ld = ws.ld_t; s.d = desc->d_out;
  SlabShape sh;
  HT_TRY(ht_slab_shape(ctx, s, &sh));
  GatAgg a{};
  a.items = g->fwd_items.items.p + it.it0; a.n_items = it.n_items; a.ent0 = rg.ent0; a.part0 = it.part0; a.row0 = rg.row0;
  a.col = g->merged ? g->ucol.p : g->col.p; a.mult = g->merged ? g->umult.p : nullptr;
  a.x = rw.x; a.m = ws.m; a.zinv = ws.zinv; a.slope = desc->slope;
  a.T = ws.T; a.ld = ws.ld_t; a.d = desc->d_out;
  a.z = z; a.z_ld = z_ld; a.z_part = rw.z_part; a.relu = desc->act == HT_ACT_RELU;
  a.Q = Q; a.q_ld = ws.ld_t; a.q_part = rw.q_part;
  a.r = ws.r; a.r_part = rw.part ? rw.part + 2 * rw.n_part : nullptr;
  if (t_items) tm->begin(t_items);
  for (int p = 0; p < sh.P; ++p)
    HT_TRY(ht_in_launches(it.n_items, sh.launch_items(), [&](int64_t i, int64_t n) {
      GatAgg b = a;
      b.items += i;
      b.n_items = n;
      if (sh.eps == 1) launch_agg<true>(st, mode, b, sh, p * sh.S);
      else launch_agg<false>(st, mode, b, sh, p * sh.S);
      HT_LAUNCH_CHECK(ctx);
      return (int)HT_OK;
    }));
  if (t_items) tm->end();
  if (it.n_cut == 0) return HT_OK;
  if (t_fix) tm->begin(t_fix);
  HT_TRY(ht_in_launches(it.n_cut, HT_LAUNCH_WAVES / 4, [&](int64_t i, int64_t n) {
    k_gat_fix<<<(unsigned)n, 256, 0, st>>>(a, g->fwd_items.cuts.p + it.cut0 + i, mode);
    HT_LAUNCH_CHECK(ctx);
    return (int)HT_OK;
  }));
  if (t_fix) tm->end();
  return HT_OK;
}

int launch_src(ht_ctx* ctx, const GatPass& all, int nvec) {
  return ht_in_launches(all.n_items, HT_LAUNCH_WAVES, [&](int64_t i, int64_t n) {
    GatPass a = all;
    a.items += i;
    a.n_items = n;
    const unsigned nb = (unsigned)((n + 3) / 4);
    if (nvec <= 8) k_gat_src_g<8><<<nb, 256, 0, ctx->stream>>>(a);
    else if (nvec <= 16) k_gat_src_g<16><<<nb, 256, 0, ctx->stream>>>(a);
    else if (nvec <= 32) k_gat_src_g<32><<<nb, 256, 0, ctx->stream>>>(a);
    else if (nvec <= 64) k_gat_src<1><<<nb, 256, 0, ctx->stream>>>(a);
    else if (nvec <= 128) k_gat_src<2><<<nb, 256, 0, ctx->stream>>>(a);
    else k_gat_src<4><<<nb, 256, 0, ctx->stream>>>(a);
    HT_LAUNCH_CHECK(ctx);
    return (int)HT_OK;
  });
}

// The scratch memory of the dense steps of a backward pass, over V rows in blocks of `step`.
void dense_wants(int64_t V, int64_t step, int d_in, int d, std::vector<ScratchWant>* want) {
  for (int64_t rows : {std::min(step, V), V % step}) {
    want->push_back({HT_S_TNPART, ht_gemm_tn_bytes(rows, d, 4)});
    want->push_back({HT_S_TNPART, ht_gemm_tn_bytes(rows, d_in, d)});
  }
  want->push_back({HT_S_PACKW, (size_t)ht_packed_w_bytes(d, d_in)});
}

// keep (nullable, everything in HBM): where t, the row values, Q and r go for this epoch's backward pass
int gat_fwd_impl(ht_ctx* ctx, const ht_graph* g, const ht_gat_desc* desc, const ht_tensor* H_in, const float* W,
                 const float* a_dst, const float* a_src, ht_tensor* H_out, const GatKeep* keep, ht_stats* local, Timer* tm, int layer) {
  HT_TRY(check_desc(ctx, desc));
  HT_TRY(check(ctx, g, desc, H_in, desc->d_in, "H_in"));
  HT_TRY(check(ctx, g, desc, H_out, desc->d_out, "H_out"));
  hipStream_t st = ctx->stream;
  GatWs ws{};
  Link lk(ctx, local, tm);
  const bool out_host = on_host(H_out);
  if (on_host(H_in) || out_host) HT_TRY(lk.fork());
  HT_TRY(bind_ws(ctx, g, desc->d_out, keep, &ws));
  const int64_t q_ld = keep ? ws.ld_t : 0;
  auto ranges = ranges_of(g, (H_out->ld + q_ld + 3) * 4, !out_host && ht_may_spend(ctx));
  std::vector<ScratchWant> want = {{HT_S_PACKW, (size_t)ht_packed_w_bytes(desc->d_in, desc->d_out)}};
  range_wants(ranges, H_out->ld + q_ld, &want);
  const int rc = ht_scratch_all(ctx, want);
  if (rc == HT_ENOMEM) ranges = ranges_of(g, 0, false);   // less memory at a time: chunk by chunk
  else HT_TRY(rc);
  RangeWs rw;
  HT_TRY(range_ws(ctx, ranges, H_out->ld, q_ld, &rw));
  HT_TRY(prepare(ctx, g, desc, H_in, W, a_dst, a_src, &ws, local, tm, &lk));
  float* obuf[2] = {nullptr, nullptr};
  hipEvent_t ev_ofree[2] = {nullptr, nullptr};
  if (out_host) {
    const int64_t rows = std::max<int64_t>(g->max_ndst, 1);
    HT_TRY(ht_scratch(ctx, HT_S_LINK1, (size_t)rows * H_out->ld * 4 * 2, (void**)&obuf[0]));
    obuf[1] = obuf[0] + rows * H_out->ld;
  }
  const int li = layer < HT_MAX_LAYERS ? layer : HT_MAX_LAYERS - 1;
  int q = 0;
  for (const GatRange& r : ranges) {
    const int b = q++ & 1;
    HT_TRY(softmax_range(ctx, g, r, desc, ws, rw, local, tm));
    if (out_host) {
      HT_TRY(lk.wait(st, ev_ofree[b]));
      HT_TRY(ht_fill_zero(ctx, st, obuf[b], (size_t)r.rows * H_out->ld * 4));     // (pads reach the host)
    }
    HT_TRY(agg_range(ctx, g, r, desc, ws, rw, keep ? AGG_ZQ : AGG_Z, out_host ? obuf[b] : H_out->ptr + r.row0 * H_out->ld, H_out->ld,
                     keep ? keep->Q + r.row0 * ws.ld_t : nullptr, &local->t_agg_fwd_layer_ms[li], &local->t_agg_fix_ms, tm));
    if (out_host) {
      hipEvent_t ev_done = nullptr;
      HT_TRY(lk.rec(st, &ev_done));
      HT_TRY(lk.wait(lk.s_out, ev_done));
      HT_TRY(lk.copy(lk.s_out, H_out->ptr + r.row0 * H_out->ld, obuf[b], (size_t)r.rows * H_out->ld * 4, true));
      HT_TRY(lk.rec(lk.s_out, &ev_ofree[b]));
      lk.last_out = ev_ofree[b];
    }
  }
  for (const ChunkMeta& c : g->chunks) {   // chunk aggregations, whatever number of launches they take
    if (c.dst1 == c.dst0) continue;
    local->n_spmm_fwd += 1;
    local->n_agg_fwd_layer[li] += 1;
    local->edges += c.nnz;
  }
  if (lk.used) HT_TRY(lk.join());
  return HT_OK;
}

// The source pass of a layer of width d can take all vertices at once (with the list by source, once that is there).
bool src_fits(const ht_graph* g, int d, bool kept) {
  const int64_t ld = ht_row_pitch(d, true);
  return g->V * ld * 4 * (kept ? 1 : 2) <= GAT_DIRECT_BYTES && g->by_src.items.n_part * (ld + 4) * 4 <= GAT_RANGE_BYTES;
}

// Backward over the rows with everything in HBM, all vertices at once: dz of all rows, the destination pass over ranges of chunks
// (or what the forward pass kept), and the source pass over the whole graph's entries by source, which writes every row of dt
// once; chunk by chunk a row is read and written again for every chunk that names its vertex.  *done = false: it would take more
// memory than it may have, nothing was enqueued.
int gat_bwd_rows_direct(ht_ctx* ctx, const ht_graph* g, const ht_gat_desc* desc, const GatWs& ws, const GatKeep* keep,
                        const ht_tensor* H_in, const float* W, const float* a_dst, const float* a_src, const ht_tensor* H_out,
                        const ht_tensor* dH_out, float* dT, int64_t ld_dt, ht_stats* local, Timer* tm, Link* lk, bool* done) {
  *done = false;
  hipStream_t st = ctx->stream;
  const int64_t V = g->V;
  const int d = desc->d_out, nvec = (d + 3) / 4, sc_col = (int)ws.ld_t;
  const size_t mat = (size_t)V * ws.ld_t * 4;
  if (V <= 0) return HT_OK;
  if (!ht_may_spend(ctx) || !src_fits(g, d, keep != nullptr)) return HT_OK;
  const SourceRows& S = g->by_src;
  float *dz = nullptr, *Q = keep ? keep->Q : nullptr;
  float* s_part = nullptr;
  std::vector<GatRange> ranges;
  RangeWs rw;
  ScratchMark mark(ctx);
  auto take = [&]() -> int {
    std::vector<ScratchWant> want = {{HT_S_DZCHUNK, mat}};
    if (!keep) {
      ranges = ranges_of(g, (ws.ld_t + 3) * 4, true);
      want.push_back({HT_S_ACHUNK, mat});
      want.push_back({HT_S_PACKW, (size_t)ht_packed_w_bytes(desc->d_in, d)});
      range_wants(ranges, ws.ld_t, &want);
    }
    // the dense steps behind this pass add to the caller's tensors: nothing may fail there for want of memory that is held here
    dense_wants(V, BLOCK_HBM, desc->d_in, d, &want);
    int64_t list;
    size_t making;
    ht_graph_by_source_bytes(g, &list, &making);
    want.push_back({HT_S_DZCHUNK, making});
    HT_TRY(ht_scratch_all(ctx, want, list + (g->merged && !S.mult.p ? g->n_unique * 4 : 0)));
    HT_TRY(ht_graph_by_source(ctx, g, HT_S_DZCHUNK));
    if (!src_fits(g, d, keep != nullptr)) return HT_ENOMEM;
    HT_TRY(ht_graph_by_source_mult(ctx, g));
    // (the partial sums of both passes share a slot, one after the other)
    want.push_back({HT_S_SPART, (size_t)(S.items.n_part * ld_dt) * 4});
    return ht_scratch_all(ctx, want);
  };
  const int rc = take();
  if (rc == HT_ENOMEM) {
    mark.undo();
    return HT_OK;
  }
  HT_TRY(rc);
  HT_TRY(ht_scratch(ctx, HT_S_DZCHUNK, mat, (void**)&dz));
  if (!keep) {
    HT_TRY(ht_scratch(ctx, HT_S_ACHUNK, mat, (void**)&Q));
    HT_TRY(range_ws(ctx, ranges, 0, ws.ld_t, &rw));
  }
  HT_TRY(ht_scratch(ctx, HT_S_SPART, (size_t)(S.items.n_part * ld_dt) * 4, (void**)&s_part));
  *done = true;
  if (!keep) HT_TRY(prepare(ctx, g, desc, H_in, W, a_dst, a_src, &ws, local, tm, lk));
  for (const GatRange& r : ranges) {
    HT_TRY(softmax_range(ctx, g, r, desc, ws, rw, local, tm));
    HT_TRY(agg_range(ctx, g, r, desc, ws, rw, AGG_Q, nullptr, 0, Q + r.row0 * ws.ld_t, &local->t_gat_dst_ms, &local->t_gat_dst_ms, tm));
  }
  tm->begin(&local->t_gat_dst_ms);
  const int lpr = row_lanes(ws.ld_t);
  k_gat_dz<<<row_grid(V, lpr), 256, 0, st>>>(dH_out->ptr, dH_out->ld, H_out->ptr, H_out->ld, desc->act == HT_ACT_RELU, V, d, dz, Q, ws.ld_t,
                                             ws.p, ws.m, ws.zinv, ws.r, ws.dp, ws.d4, lpr);
  HT_LAUNCH_CHECK(ctx);
  tm->end();
  GatPass a{};
  a.items = S.items.items.p; a.n_items = S.items.n_items;
  a.idx = S.idx.p; a.mult = g->merged ? S.mult.p : nullptr;
  a.mat = dz; a.mat_ld = ws.ld_t; a.own = ws.T; a.own_ld = ws.ld_t; a.d = d;
  a.q = ws.q; a.d4 = ws.d4; a.slope = desc->slope;
  a.out = dT; a.out_ld = ld_dt; a.partial = s_part; a.sc_col = sc_col;
  tm->begin(&local->t_gat_src_ms);
  HT_TRY(launch_src(ctx, a, nvec));
  if (S.items.n_cut > 0) {
    SpmmArgs f{};
    f.cuts = S.items.cuts.p; f.n_fix = S.items.n_cut;
    f.d = sc_col + 4; f.out = dT; f.out_ld = ld_dt; f.partial = s_part;
    HT_TRY(ht_spmm_fix_launch(ctx, st, f));
  }
  tm->end();
  return HT_OK;
}

int gat_bwd_impl(ht_ctx* ctx, const ht_graph* g, const ht_gat_desc* desc, const ht_tensor* H_in, const float* W,
                 const float* a_dst, const float* a_src, const ht_tensor* H_out, const ht_tensor* dH_out,
                 ht_tensor* dH_in, float* dW, float* da_dst, float* da_src, const GatKeep* keep, ht_stats* local, Timer* tm,
                 bool dhin_is_zero, bool* changed) {
  HT_TRY(check_desc(ctx, desc));
  HT_TRY(check(ctx, g, desc, H_in, desc->d_in, "H_in"));
  HT_TRY(check(ctx, g, desc, H_out, desc->d_out, "H_out"));
  HT_TRY(check(ctx, g, desc, dH_out, desc->d_out, "dH_out"));
  if (dH_in) HT_TRY(check(ctx, g, desc, dH_in, desc->d_in, "dH_in"));
  hipStream_t st = ctx->stream;
  GatWs ws{};
  Link lk(ctx, local, tm);
  const bool hin_host = on_host(H_in), hout_host = on_host(H_out), dho_host = on_host(dH_out), dhi_host = on_host(dH_in);
  const bool on_link = hin_host || hout_host || dho_host || dhi_host;
  if (on_link) HT_TRY(lk.fork());
  HT_TRY(bind_ws(ctx, g, desc->d_out, keep, &ws));
  const int d = desc->d_out;
  const int nvec = (d + 3) / 4;
  const int lpr = row_lanes(ws.ld_t);
  const int sc_col = (int)ws.ld_t;              // the scalar column block sits behind the padded data columns
  const int64_t ld_dt = ws.ld_t + 4;
  const int64_t mx = std::max<int64_t>(g->max_ndst, 1);
  float *dT = nullptr, *dz = nullptr, *Q = nullptr, *da4 = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_TFULL2, (size_t)std::max<int64_t>(g->V, 1) * ld_dt * 4, (void**)&dT));
  HT_TRY(ht_scratch(ctx, HT_S_MISC, (size_t)d * 16, (void**)&da4));
  bool at_once = false;
  if (!on_link)
    HT_TRY(gat_bwd_rows_direct(ctx, g, desc, ws, keep, H_in, W, a_dst, a_src, H_out, dH_out, dT, ld_dt, local, tm, &lk, &at_once));
  if (!at_once && keep) return ht_set_err(ctx, HT_ENOMEM, "GAT backward: no memory for all vertices at once beside what the forward pass kept");
  RangeWs rw;
  float* src_part = nullptr;
  if (!at_once) {
    // Both passes of a chunk keep their partial sums in one slot, one after the other.  It is taken at the larger size before
    // either pointer into it is kept: a slot that grew between two chunks would leave the first pass writing into freed memory.
    if (g->max_bpart > 0) HT_TRY(ht_scratch(ctx, HT_S_SPART, (size_t)g->max_bpart * ld_dt * 4, (void**)&src_part));
    HT_TRY(range_ws(ctx, ranges_of(g, 0, false), 0, ws.ld_t, &rw));
    if (g->max_bpart > 0) HT_TRY(ht_scratch(ctx, HT_S_SPART, (size_t)g->max_bpart * ld_dt * 4, (void**)&src_part));
    HT_TRY(prepare(ctx, g, desc, H_in, W, a_dst, a_src, &ws, local, tm, &lk));
    HT_TRY(ht_scratch(ctx, HT_S_DZCHUNK, (size_t)mx * ws.ld_t * 4, (void**)&dz));
    HT_TRY(ht_scratch(ctx, HT_S_ACHUNK, (size_t)mx * ws.ld_t * 4, (void**)&Q));
    HT_TRY(ht_fill_zero(ctx, st, dT, (size_t)g->V * ld_dt * 4));
  }
  // host-resident H_out / dH_out: the rows of the next chunk are staged while this one computes
  float* hbuf[2] = {nullptr, nullptr};
  float* gbuf[2] = {nullptr, nullptr};
  hipEvent_t ev_in[2] = {nullptr, nullptr}, ev_free[2] = {nullptr, nullptr};
  if (hout_host) {
    HT_TRY(ht_scratch(ctx, HT_S_LINK1, (size_t)mx * H_out->ld * 4 * 2, (void**)&hbuf[0]));
    hbuf[1] = hbuf[0] + mx * H_out->ld;
  }
  if (dho_host) {
    HT_TRY(ht_scratch(ctx, HT_S_LINK2, (size_t)mx * dH_out->ld * 4 * 2, (void**)&gbuf[0]));
    gbuf[1] = gbuf[0] + mx * dH_out->ld;
  }
  std::vector<int> live;
  for (int j = 0; j < g->n; ++j)
    if (g->chunks[j].dst1 > g->chunks[j].dst0) {
      live.push_back(j);
      local->n_spmm_bwd += 2;
      local->edges += 2 * g->chunks[j].nnz;
    }
  if (at_once) live.clear();
  auto stage_chunk = [&](size_t i) -> int {
    if (!(hout_host || dho_host) || i >= live.size()) return HT_OK;
    const ChunkMeta& c = g->chunks[live[i]];
    const int b = (int)(i & 1);
    const int64_t nd = c.dst1 - c.dst0;
    HT_TRY(lk.wait(lk.s_in, ev_free[b]));
    if (hout_host) HT_TRY(lk.copy(lk.s_in, hbuf[b], H_out->ptr + c.dst0 * H_out->ld, (size_t)nd * H_out->ld * 4, false));
    if (dho_host) HT_TRY(lk.copy(lk.s_in, gbuf[b], dH_out->ptr + c.dst0 * dH_out->ld, (size_t)nd * dH_out->ld * 4, false));
    return lk.rec(lk.s_in, &ev_in[b]);
  };
  HT_TRY(stage_chunk(0));
  for (size_t i = 0; i < live.size(); ++i) {
    const ChunkMeta& c = g->chunks[live[i]];
    const int64_t ndst = c.dst1 - c.dst0;
    const int b = (int)(i & 1);
    HT_TRY(stage_chunk(i + 1));
    const GatRange range = range_of(g, c);
    HT_TRY(softmax_range(ctx, g, range, desc, ws, rw, local, tm));
    // destination pass: Q_v = sum_e w_e f_e t_u, then dz, S and dp
    tm->begin(&local->t_gat_dst_ms);
    HT_TRY(agg_range(ctx, g, range, desc, ws, rw, AGG_Q, nullptr, 0, Q, nullptr, nullptr, tm));
    if (hout_host || dho_host) HT_TRY(lk.wait(st, ev_in[b]));
    k_gat_dz<<<row_grid(ndst, lpr), 256, 0, st>>>(dho_host ? gbuf[b] : dH_out->ptr + c.dst0 * dH_out->ld, dH_out->ld,
                                                  hout_host ? hbuf[b] : H_out->ptr + c.dst0 * H_out->ld, H_out->ld,
                                                  desc->act == HT_ACT_RELU, ndst, d, dz, Q, ws.ld_t, ws.p + c.dst0, ws.m + c.dst0,
                                                  ws.zinv + c.dst0, ws.r + c.dst0, ws.dp + c.dst0, ws.d4, lpr);
    HT_LAUNCH_CHECK(ctx);
    if (hout_host || dho_host) HT_TRY(lk.rec(st, &ev_free[b]));   // the staged rows have been consumed
    tm->end();
    GatPass a{};
    a.d = d; a.q = ws.q; a.d4 = ws.d4; a.slope = desc->slope;
    // source pass
    a.items = g->bwd_items.items.p + c.bwd.it0; a.n_items = c.bwd.n_items; a.part0 = c.bwd.part0;
    a.idx = g->merged ? g->usdst.p : g->sdst.p;
    a.mult = g->merged ? g->umult_bwd.p : nullptr;
    a.mat = dz; a.mat_ld = ws.ld_t;
    a.own = ws.T; a.own_ld = ws.ld_t; a.own_idx = g->nbr.p;
    a.out = dT; a.out_ld = ld_dt; a.add = true;
    a.partial = src_part; a.sc_col = sc_col;
    tm->begin(&local->t_gat_src_ms);
    if (a.n_items > 0) HT_TRY(launch_src(ctx, a, nvec));
    if (c.bwd.n_cut > 0) {
      SpmmArgs f{};
      f.cuts = g->bwd_items.cuts.p + c.bwd.cut0; f.n_fix = c.bwd.n_cut; f.part0 = c.bwd.part0;
      f.d = sc_col + 4;
      f.out = dT; f.out_ld = ld_dt; f.out_idx = g->nbr.p;
      f.accumulate = 1;
      f.partial = src_part;
      HT_TRY(ht_spmm_fix_launch(ctx, st, f));
    }
    tm->end();
  }
  if (g->V > 0) {
    k_gat_finish<<<row_grid(g->V, lpr), 256, 0, st>>>(dT, ld_dt, d, sc_col, ws.dp, a_dst, a_src, g->V, ws.pq4, lpr);
    HT_LAUNCH_CHECK(ctx);
  }
  // da = T^T [dp dq 0 0]; dW = H^T dt; dH += dt W^T, in row blocks; host-resident H_in / dH_in blocks go
  // through staging pairs (dH_in: in, add, out; straight out when it is known to hold zeros)
  const int64_t step = (hin_host || dhi_host) ? ctx->link_block_rows : BLOCK_HBM;
  const int64_t brows = std::min<int64_t>(step, std::max<int64_t>(g->V, 1));
  float* sH[2] = {nullptr, nullptr};
  float* sD[2] = {nullptr, nullptr};
  hipEvent_t ev_bfree[2] = {nullptr, nullptr}, ev_dout[2] = {nullptr, nullptr};
  if (hin_host) {
    HT_TRY(ht_scratch(ctx, HT_S_LINK0, (size_t)brows * H_in->ld * 4 * 2, (void**)&sH[0]));
    sH[1] = sH[0] + brows * H_in->ld;
  }
  if (dhi_host) {
    // (the chunk loop is over: its staging pair is free)
    HT_TRY(ht_scratch(ctx, HT_S_LINK1, (size_t)brows * dH_in->ld * 4 * 2, (void**)&sD[0]));
    sD[1] = sD[0] + brows * dH_in->ld;
  }
  {
    std::vector<ScratchWant> want;
    dense_wants(g->V, step, desc->d_in, d, &want);
    HT_TRY(ht_scratch_each(ctx, want));
  }
  *changed = true;    // dH_in is added to from here on
  // the staging memory was used by the earlier phases: copies into it start behind their last reader
  if (lk.used) HT_TRY(lk.fork());
  bool first = true;
  TnLater da_later;
  da_later.column[0] = da_dst;
  da_later.column[1] = da_src;
  int k = 0;
  for (int64_t r0 = 0; r0 < g->V; r0 += step, ++k) {
    const int64_t nr = std::min(step, g->V - r0);
    const int b = k & 1;
    const float* h_rows = H_in->ptr + r0 * H_in->ld;
    float* dh_rows = dH_in ? dH_in->ptr + r0 * dH_in->ld : nullptr;
    const bool dh_add = !dhin_is_zero;
    if (hin_host || dhi_host) {
      hipEvent_t ev_bin = nullptr;
      HT_TRY(lk.wait(lk.s_in, ev_bfree[b]));
      HT_TRY(lk.wait(lk.s_in, ev_dout[b]));
      if (hin_host) {
        HT_TRY(lk.copy(lk.s_in, sH[b], h_rows, (size_t)nr * H_in->ld * 4, false));
        h_rows = sH[b];
      }
      if (dhi_host) {
        if (dh_add) HT_TRY(lk.copy(lk.s_in, sD[b], dh_rows, (size_t)nr * dH_in->ld * 4, false));
        else HT_TRY(lk.wait(st, ev_dout[b]));      // the compute stream overwrites the block
        dh_rows = sD[b];
      }
      HT_TRY(lk.rec(lk.s_in, &ev_bin));
      HT_TRY(lk.wait(st, ev_bin));
    }
    tm->begin(&local->t_gemm_ms);
    const bool all = nr == g->V;
    TnLater later;
    HT_TRY(ht_gemm_tn(ctx, st, ws.T + r0 * ws.ld_t, ws.ld_t, ws.pq4 + r0 * 4, 4, da4, nr, d, 4, first ? 0 : 1, all ? &da_later : nullptr));
    HT_TRY(ht_gemm_tn(ctx, st, h_rows, H_in->ld, dT + r0 * ld_dt, ld_dt, dW, nr, desc->d_in, d, first ? 0 : 1, all ? &later : nullptr));
    if (dH_in)
      HT_TRY(ht_gemm_nt(ctx, st, dT + r0 * ld_dt, ld_dt, W, dh_rows, dH_in->ld, nr, d, desc->d_in, dh_add ? 1 : 0));
    tm->end();
    if (hin_host || dhi_host) HT_TRY(lk.rec(st, &ev_bfree[b]));
    if (dhi_host) {
      HT_TRY(lk.wait(lk.s_out, ev_bfree[b]));
      HT_TRY(lk.copy(lk.s_out, dH_in->ptr + r0 * dH_in->ld, sD[b], (size_t)nr * dH_in->ld * 4, true));
      HT_TRY(lk.rec(lk.s_out, &ev_dout[b]));
      lk.last_out = ev_dout[b];
    }
    local->n_gemm += 3;
    local->gemm_flops += 4.0 * nr * desc->d_in * d;
    first = false;
  }
  if (first) {
    HT_TRY(ht_fill_zero(ctx, st, dW, (size_t)desc->d_in * d * 4));
    HT_TRY(ht_fill_zero(ctx, st, da4, (size_t)d * 16));
  }
  if (!da_later.left) {
    k_gat_split<<<(unsigned)((d + 255) / 256), 256, 0, st>>>(da4, d, da_dst, da_src);
    HT_LAUNCH_CHECK(ctx);
  }
  if (lk.used) HT_TRY(lk.join());
  return HT_OK;
}

// The end of a layer call.
int gat_done(ht_ctx* ctx, int rc, ht_stats* local, Timer* tm, std::chrono::steady_clock::time_point t0, ht_stats* stats) {
  hipError_t e = hipStreamSynchronize(ctx->stream);
  if (rc == HT_OK && e == hipSuccess) rc = tm->resolve();
  ctx->ev_next = 0;
  if (rc != HT_OK) return rc;
  HT_HIP(ctx, e);
  if (stats) {
    local->t_total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    *stats = *local;
  }
  return HT_OK;
}

}  // namespace

extern "C" {

int ht_gat_layer_fwd(ht_ctx* ctx, const ht_graph* g, const ht_gat_desc* desc, const ht_tensor* H_in, const float* W,
                     const float* a_dst, const float* a_src, ht_tensor* H_out, ht_stats* stats) {
  if (!ctx) return HT_EINVAL;
  if (!g || !desc || !H_in || !H_out || !W || !a_dst || !a_src) return ht_set_err(ctx, HT_EINVAL, "ht_gat_layer_fwd: null argument");
  if (g->ctx != ctx) return ht_set_err(ctx, HT_ESTATE, "graph belongs to another context");
  HT_HIP(ctx, hipSetDevice(ctx->device));
  return ht_with_room(ctx, [&]() -> int {
    auto t0 = std::chrono::steady_clock::now();
    ht_stats local{};
    Timer tm(ctx, ctx->stream, stats != nullptr);
    int rc = gat_fwd_impl(ctx, g, desc, H_in, W, a_dst, a_src, H_out, nullptr, &local, &tm, 0);
    return gat_done(ctx, rc, &local, &tm, t0, stats);
  });
}

int ht_gat_layer_bwd(ht_ctx* ctx, const ht_graph* g, const ht_gat_desc* desc, const ht_tensor* H_in, const float* W,
                     const float* a_dst, const float* a_src, const ht_tensor* H_out, const ht_tensor* dH_out,
                     ht_tensor* dH_in, float* dW, float* da_dst, float* da_src, ht_stats* stats) {
  if (!ctx) return HT_EINVAL;
  if (!g || !desc || !H_in || !H_out || !dH_out || !W || !a_dst || !a_src || !dW || !da_dst || !da_src)
    return ht_set_err(ctx, HT_EINVAL, "ht_gat_layer_bwd: null argument");
  if (g->ctx != ctx) return ht_set_err(ctx, HT_ESTATE, "graph belongs to another context");
  HT_HIP(ctx, hipSetDevice(ctx->device));
  bool changed = false;
  return ht_with_room(ctx, [&]() -> int {
    auto t0 = std::chrono::steady_clock::now();
    ht_stats local{};
    Timer tm(ctx, ctx->stream, stats != nullptr);
    int rc = gat_bwd_impl(ctx, g, desc, H_in, W, a_dst, a_src, H_out, dH_out, dH_in, dW, da_dst, da_src, nullptr, &local, &tm, false, &changed);
    return gat_done(ctx, rc, &local, &tm, t0, stats);
  }, &changed);
}

// Alg. 1 with GAT layers: forward over the layers, softmax cross-entropy on the labelled
// vertices, backward layer by layer, SGD step on W^l and a^l.  Beside the layer outputs a
// forward pass keeps rows of size O(V) for its backward pass where there is room for them
// (GatKeep); elsewhere every layer's intermediates are recomputed from its input.  With res_h = HT_RES_HOST
// the layer outputs h^1..h^{L-1} and their gradients live in pinned host memory (Alg. 1 keeps
// h^l and grad h^l on the CPU); the logits h^L and their gradient stay in HBM for the loss.
static int gat_epoch_impl(ht_ctx* ctx, const ht_graph* g, const ht_gat_model* model, const ht_tensor* X, const int32_t* labels,
                          float* loss_out, ht_stats* stats) {
  if (!g || !model || !X || !labels || !loss_out) return ht_set_err(ctx, HT_EINVAL, "ht_gat_epoch: null argument");
  if (g->ctx != ctx) return ht_set_err(ctx, HT_ESTATE, "graph belongs to another context");
  const int L = model->n_layers;
  if (L < 1 || L > HT_MAX_LAYERS || !model->dims || !model->W || !model->a_dst || !model->a_src)
    return ht_set_err(ctx, HT_EINVAL, "ht_gat_epoch: bad model");
  for (int l = 0; l <= L; ++l)
    if (model->dims[l] <= 0) return ht_set_err(ctx, HT_ESHAPE, "ht_gat_epoch: layer widths must be positive");
  for (int l = 0; l < L; ++l)
    if (!model->W[l] || !model->a_dst[l] || !model->a_src[l]) return ht_set_err(ctx, HT_EINVAL, "ht_gat_epoch: null parameter of layer %d", l);
  HT_HIP(ctx, hipSetDevice(ctx->device));
  auto t0 = std::chrono::steady_clock::now();
  hipStream_t st = ctx->stream;
  const int64_t V = g->V;
  if (model->res_h != HT_RES_AUTO && model->res_h != HT_RES_HBM && model->res_h != HT_RES_HOST)
    return ht_set_err(ctx, HT_EINVAL, "ht_gat_epoch: unknown residency %d", model->res_h);
  const bool h_host = model->res_h == HT_RES_HOST;
  auto in_hbm = [&](int l) { return !h_host || l == L; };
  // workspace: h^1..h^L, grad h^1..grad h^L (HBM or pinned host), then dW^l, da_dst^l, da_src^l, loss
  size_t floats = 64 + 64 * (size_t)L, hfloats = 64 * (size_t)L;
  for (int l = 1; l <= L; ++l)
    (in_hbm(l) ? floats : hfloats) += 2 * ((size_t)std::max<int64_t>(V, 1) * ht_row_pitch(model->dims[l], in_hbm(l)) + 32);
  for (int l = 0; l < L; ++l) floats += (size_t)model->dims[l] * model->dims[l + 1] + 2 * (size_t)model->dims[l + 1] + 96;
  float* base = nullptr;
  float* hbase = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_GATWS, floats * 4, (void**)&base));
  if (h_host && L > 1) HT_TRY(ht_host_scratch(ctx, 2, hfloats * 4, (void**)&hbase));
  std::vector<ht_tensor> h(L + 1), gh(L + 1);
  std::vector<float*> dW(L), dad(L), das(L);
  float* cur = base;
  float* hcur = hbase;
  auto take = [&](size_t n) { float* p = cur; cur += (n + 31) & ~(size_t)31; return p; };
  auto take_host = [&](size_t n) { float* p = hcur; hcur += (n + 31) & ~(size_t)31; return p; };
  for (int l = 1; l <= L; ++l) {
    const bool dev = in_hbm(l);
    const int64_t ld = ht_row_pitch(model->dims[l], dev);
    const size_t n = (size_t)std::max<int64_t>(V, 1) * ld;
    const int loc = dev ? HT_LOC_DEVICE : HT_LOC_HOST_PINNED;
    h[l] = ht_tensor{dev ? take(n) : take_host(n), V, model->dims[l], ld, loc};
    gh[l] = ht_tensor{dev ? take(n) : take_host(n), V, model->dims[l], ld, loc};
  }
  for (int l = 0; l < L; ++l) {
    dW[l] = take((size_t)model->dims[l] * model->dims[l + 1]);
    dad[l] = take(model->dims[l + 1]);
    das[l] = take(model->dims[l + 1]);
  }
  float *loss_host = nullptr, *loss_gpu = nullptr;
  HT_TRY(ht_host_scratch(ctx, HT_HS_LOSS, 64, (void**)&loss_host));
  HT_HIP(ctx, hipHostGetDevicePointer((void**)&loss_gpu, loss_host, 0));
  LossParts loss_parts{};
  ht_stats local{};
  Timer tm(ctx, st, stats != nullptr);
  auto fail = [&](int rc) {
    (void)hipStreamSynchronize(st);
    (void)hipStreamSynchronize(ctx->side[0]);
    (void)hipStreamSynchronize(ctx->side[1]);
    (void)ht_flush_products(ctx, st, true);
    ctx->ev_next = 0;
    return rc;
  };
  // What the layers' forward passes leave for their backward passes, with everything in HBM and room for it: the backward pass
  // then neither transforms, scores nor gathers over the destinations again (each layer's second gather of t rides on the first).
  std::vector<GatKeep> keep;
  if (!h_host && X->loc == HT_LOC_DEVICE && V > 0) {
    size_t kf = 0;
    for (int l = 1; l <= L; ++l) kf += (size_t)V * (2 * ht_row_pitch(model->dims[l], true) + 5) + 7 * 32;
    float* kp = nullptr;
    bool room = kf * 4 <= (size_t)GAT_KEEP_BYTES && ht_may_spend(ctx) &&
                (ctx->gat_keep_limit == 0 || kf * 4 < ctx->gat_keep_limit || ht_room(ctx) > ctx->gat_keep_room);
    if (room) {
      ScratchMark mark(ctx);
      int64_t list;
      size_t making;
      ht_graph_by_source_bytes(g, &list, &making);
      int rc = ht_scratch_all(ctx, {{HT_S_GATKEEP, kf * 4}, {HT_S_DZCHUNK, making}}, list);
      if (rc == HT_OK) rc = ht_graph_by_source(ctx, g, HT_S_DZCHUNK);
      if (rc != HT_OK && rc != HT_ENOMEM) return rc;
      room = rc == HT_OK;
      for (int l = 1; l <= L; ++l) room = room && src_fits(g, model->dims[l], true);
      if (room) HT_TRY(ht_scratch(ctx, HT_S_GATKEEP, kf * 4, (void**)&kp));
      else mark.undo();
    }
    auto cut = [&](size_t n) { float* p = kp; kp += (n + 31) & ~(size_t)31; return p; };
    for (int l = 1; l <= L && kp; ++l) {
      const size_t n = (size_t)V * ht_row_pitch(model->dims[l], true);
      GatKeep k;
      k.T = cut(n); k.Q = cut(n);
      k.p = cut(V); k.q = cut(V); k.m = cut(V); k.zinv = cut(V); k.r = cut(V);
      keep.push_back(k);
    }
  }
  bool changed = false;   // (only this call's own buffers)
  auto passes = [&]() -> int {
    std::vector<size_t> products;
    for (int l = 0; l < L; ++l)
      for (int32_t d : {model->dims[l], 0})
        products.push_back(ht_gemm_tn_bytes(V, d ? d : model->dims[l + 1], d ? model->dims[l + 1] : 4));
    HT_TRY(ht_defer_products(ctx, products));
    for (int l = 0; l < L; ++l) {
      ht_gat_desc d{model->dims[l], model->dims[l + 1], l < L - 1 ? HT_ACT_RELU : HT_ACT_NONE, model->slope};
      HT_TRY(gat_fwd_impl(ctx, g, &d, l == 0 ? X : &h[l], model->W[l], model->a_dst[l], model->a_src[l], &h[l + 1],
                          keep.empty() ? nullptr : &keep[l], &local, &tm, l));
    }
    tm.begin(&local.t_loss_ms);
    HT_TRY(ht_softmax_ce(ctx, st, h[L].ptr, h[L].ld, labels, V, model->dims[L], gh[L].ptr, gh[L].ld, &loss_parts));
    tm.end();
    for (int l = L - 1; l >= 0; --l) {
      ht_gat_desc d{model->dims[l], model->dims[l + 1], l < L - 1 ? HT_ACT_RELU : HT_ACT_NONE, model->slope};
      HT_TRY(gat_bwd_impl(ctx, g, &d, l == 0 ? X : &h[l], model->W[l], model->a_dst[l], model->a_src[l], &h[l + 1], &gh[l + 1],
                          l > 0 ? &gh[l] : nullptr, dW[l], dad[l], das[l], keep.empty() ? nullptr : &keep[l], &local, &tm, true, &changed));
    }
    return HT_OK;
  };
  int rc = passes();
  if (rc == HT_ENOMEM && !keep.empty()) {   // again without keeping anything (nothing of the caller's was changed yet)
    (void)fail(rc);
    ctx->gat_keep_limit = ctx->scratch_bytes[HT_S_GATKEEP] * 8 / 9;      // (a slot is an eighth larger than asked for)
    (void)ht_scratch_release(ctx, HT_S_GATKEEP);
    ctx->gat_keep_room = ht_room(ctx);
    keep.clear();
    local = ht_stats{};
    tm.ev.clear();
    rc = passes();
  }
  if (rc != HT_OK) return fail(rc);
  std::vector<ht_sgd_item> params;
  for (int l = 0; l < L; ++l) {
    params.push_back({model->W[l], dW[l], (int64_t)model->dims[l] * model->dims[l + 1]});
    params.push_back({model->a_dst[l], dad[l], model->dims[l + 1]});
    params.push_back({model->a_src[l], das[l], model->dims[l + 1]});
  }
  rc = ht_step(ctx, st, params, model->lr, loss_parts, loss_gpu);
  if (rc != HT_OK) return fail(rc);
  {
    hipError_t e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(ht_set_err(ctx, HT_EHIP, "synchronize: %s", hipGetErrorString(e)));
    int rc = tm.resolve();
    ctx->ev_next = 0;
    if (rc != HT_OK) return rc;
    *loss_out = *(volatile float*)loss_host;
  }
  if (stats) {
    for (int l = 0; l < HT_MAX_LAYERS; ++l) local.t_spmm_fwd_ms += local.t_agg_fwd_layer_ms[l];
    local.t_spmm_fwd_ms += local.t_agg_fix_ms;
    local.t_total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    *stats = local;
  }
  return HT_OK;
}

int ht_gat_epoch(ht_ctx* ctx, const ht_graph* g, const ht_gat_model* model, const ht_tensor* X, const int32_t* labels,
                 float* loss_out, ht_stats* stats) {
  if (!ctx) return HT_EINVAL;
  // (the caller's parameters change in the last launch, behind everything that takes memory)
  return ht_with_room(ctx, [&] { return gat_epoch_impl(ctx, g, model, X, labels, loss_out, stats); });
}

}  // extern "C"
