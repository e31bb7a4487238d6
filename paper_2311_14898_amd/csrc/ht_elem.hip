// Small HBM-bound kernels: ReLU derivative mask (Sec. 2.3), softmax
// cross-entropy and its gradient (the downstream task of Alg. 1),
// SGD step (Alg. 1), zero fill.
#include <algorithm>

#include "ht_internal.h"

namespace {

// (dz may be ref: a thread writes only where it alone has read)
__global__ void k_relu_mask(const float* __restrict__ dh, int64_t ld_dh, const float* ref,
                            int64_t ld_ref, float* dz, int64_t ld_dz, int64_t rows, int cols4) {
  // one thread per float4 of the padded row
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int vec_per_row = cols4 >> 2;
  if (i >= rows * vec_per_row) return;
  const int64_t r = i / vec_per_row;
  const int c = (int)(i % vec_per_row) * 4;
  const float4 g = *reinterpret_cast<const float4*>(dh + r * ld_dh + c);
  const float4 z = *reinterpret_cast<const float4*>(ref + r * ld_ref + c);
  float4 o;
  o.x = z.x > 0.f ? g.x : 0.f;
  o.y = z.y > 0.f ? g.y : 0.f;
  o.z = z.z > 0.f ? g.z : 0.f;
  o.w = z.w > 0.f ? g.w : 0.f;
  *reinterpret_cast<float4*>(dz + r * ld_dz + c) = o;
}

// The loss in two launches whatever V is: labelled vertices per block; gradient rows and per-block loss sums.  k_step adds those up.
// (With an atomic per wave for the count, a wave per vertex and the vertices' losses through memory it was six, 1.5 ms at 2.45 M
// vertices and 47 classes, where the rows' bytes take 0.2; now 0.4 ms.)
constexpr int COUNT_BLOCKS = 256;
constexpr int64_t LOSS_BLOCKS = 4096;

template <typename T>
__device__ __forceinline__ T block_sum(T x, T* sh) {   // 256 threads, in a fixed order; all get the result
  sh[threadIdx.x] = x;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  return sh[0];
}

__global__ void __launch_bounds__(256) k_count_labelled(const int32_t* __restrict__ labels, int64_t V, unsigned long long* __restrict__ cnt) {
  __shared__ unsigned long long sh[256];
  unsigned long long c = 0;
  for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < V; v += (int64_t)gridDim.x * 256) c += labels[v] >= 0;
  c = block_sum(c, sh);
  if (threadIdx.x == 0) cnt[blockIdx.x] = c;
}

__device__ __forceinline__ float4 logits4(const float* x, int c, int C) {   // columns past the end (pads) count as -inf
  float4 v = *reinterpret_cast<const float4*>(x + c);
  if (c + 1 >= C) v.y = -INFINITY;
  if (c + 2 >= C) v.z = -INFINITY;
  if (c + 3 >= C) v.w = -INFINITY;
  return v;
}

// lpr lanes per vertex, four classes per lane and step.  loss[block] = sum of lse - x[y] over the block's labelled vertices.
__global__ void __launch_bounds__(256) k_softmax_ce(const float* __restrict__ logits, int64_t ld,
                                                    const int32_t* __restrict__ labels, int64_t V, int C,
                                                    const unsigned long long* __restrict__ cnt, int n_cnt,
                                                    float* __restrict__ grad, int64_t ld_g, double* __restrict__ loss, int lpr) {
  __shared__ double sh[256];
  __shared__ unsigned long long shc[256];
  const unsigned long long T = block_sum((int)threadIdx.x < n_cnt ? cnt[threadIdx.x] : 0ull, shc);
  const float invT = 1.f / (float)T;
  const int rpb = 256 / lpr, ll = threadIdx.x % lpr;
  double mine = 0.0;
  for (int64_t v = (int64_t)blockIdx.x * rpb + threadIdx.x / lpr; v < V; v += (int64_t)gridDim.x * rpb) {
    const int32_t y = labels[v];
    const float* x = logits + v * ld;
    float* g = grad + v * ld_g;
    if (y < 0) {
      for (int c = ll * 4; c < C; c += lpr * 4) *reinterpret_cast<float4*>(g + c) = make_float4(0.f, 0.f, 0.f, 0.f);
      continue;
    }
    float m = -INFINITY;
    for (int c = ll * 4; c < C; c += lpr * 4) {
      const float4 t = logits4(x, c, C);
      m = fmaxf(m, fmaxf(fmaxf(t.x, t.y), fmaxf(t.z, t.w)));
    }
    for (int o = lpr >> 1; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    float z = 0.f;
    for (int c = ll * 4; c < C; c += lpr * 4) {
      const float4 t = logits4(x, c, C);
      z += (expf(t.x - m) + expf(t.y - m)) + (expf(t.z - m) + expf(t.w - m));
    }
    for (int o = lpr >> 1; o > 0; o >>= 1) z += __shfl_xor(z, o, 64);
    const float lse = m + logf(z);
    for (int c = ll * 4; c < C; c += lpr * 4) {
      const float4 t = logits4(x, c, C);
      float4 o;
      o.x = (expf(t.x - lse) - (c == y ? 1.f : 0.f)) * invT;
      o.y = (expf(t.y - lse) - (c + 1 == y ? 1.f : 0.f)) * invT;
      o.z = (expf(t.z - lse) - (c + 2 == y ? 1.f : 0.f)) * invT;
      o.w = (expf(t.w - lse) - (c + 3 == y ? 1.f : 0.f)) * invT;
      *reinterpret_cast<float4*>(g + c) = o;
    }
    if (ll == 0) mine += (double)(lse - x[y]);
  }
  const double s = block_sum(mine, sh);
  if (threadIdx.x == 0) loss[blockIdx.x] = s;
}

// The end of an epoch in one launch (a launch each for every product's slices, the update, the loss and its copy cost 4 to 8 us apiece: 10 k
// vertices 156 -> 125 us an epoch with the products that read W in place).  Tensor t has the blocks from first[t] on, the last block has the loss.
struct StepItem {
  float* W;
  float* dW;                 // read, or written with the sum of the slices
  int64_t n;
  const float* P;            // slices of `pitch` values each, `stride` apart inside a slice, added in slice order as k_reduce_slices does
  int64_t pitch;
  int stride, slices;
};
struct StepBatch {
  int n;
  unsigned first[HT_SGD_MAX + 1];
  StepItem t[HT_SGD_MAX];
};
__global__ void __launch_bounds__(256) k_step(StepBatch b, float lr, LossParts L, float* __restrict__ loss) {
  if (blockIdx.x == b.first[b.n]) {
    __shared__ double sh[256];
    __shared__ unsigned long long shc[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < L.n_part; i += 256) s += L.part[i];
    s = block_sum(s, sh);
    const unsigned long long T = block_sum((int)threadIdx.x < L.n_count ? L.count[threadIdx.x] : 0ull, shc);
    if (threadIdx.x == 0) *loss = T > 0 ? (float)(s / (double)T) : 0.f;
    return;
  }
  int k = 0;
  while (k + 1 < b.n && blockIdx.x >= b.first[k + 1]) ++k;
  const StepItem it = b.t[k];
  const int64_t blk = blockIdx.x - b.first[k];
  if (it.slices == 0) {
    const int64_t i = blk * 256 + threadIdx.x;
    if (i < it.n) it.W[i] = it.W[i] - lr * it.dW[i];
    return;
  }
  // 64 elements; the four waves bring 64 slices at a time into LDS while the first one adds the 64 before them
  __shared__ float tile[2][64][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = blk * 64 + lane;
  const float* P = it.P + i * it.stride;
  float v[16];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int s = s0 + wave * 16 + q;
      v[q] = (s < it.slices && i < it.n) ? P[(int64_t)s * it.pitch] : 0.f;
    }
  };
  float s = 0.f;
  fetch(0);
  for (int s0 = 0, t = 0; s0 < it.slices; s0 += 64, t ^= 1) {
#pragma unroll
    for (int q = 0; q < 16; ++q) tile[t][wave * 16 + q][lane] = v[q];
    if (s0 + 64 < it.slices) fetch(s0 + 64);
    __syncthreads();   // (the other buffer was added before this barrier's turn came round)
    if (wave == 0) {
      const int m = (it.slices - s0) < 64 ? (it.slices - s0) : 64;
      for (int q = 0; q < m; ++q) s += tile[t][q][lane];
    }
  }
  if (wave == 0 && i < it.n) {
    it.dW[i] = s;
    it.W[i] = it.W[i] - lr * s;
  }
}

// n16 16-byte words from p16 (16-byte aligned), then the words of the ragged ends; a bounded grid
// that strides, so the launch also fits a HIP graph node at any size
__global__ void k_zero(uint4* __restrict__ p16, int64_t n16, uint32_t* __restrict__ head, int n_head,
                       uint32_t* __restrict__ tail, int n_tail, uint32_t v) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = t; i < n16; i += stride) p16[i] = make_uint4(v, v, v, v);
  if (t < n_head) head[t] = v;
  if (t < n_tail) tail[t] = v;
}

}  // namespace

int ht_relu_mask(ht_ctx* ctx, hipStream_t st, const float* dh, int64_t ld_dh, const float* ref, int64_t ld_ref,
                 float* dz, int64_t ld_dz, int64_t rows, int32_t cols) {
  if (rows <= 0 || cols <= 0) return HT_OK;
  const int cols4 = (cols + 3) & ~3;
  // one thread per 16-byte vector, as many rows a launch as it holds
  return ht_in_launches(rows, HT_LAUNCH_WAVES * 64 / (cols4 >> 2), [&](int64_t r, int64_t m) {
    const int64_t n = m * (cols4 >> 2);
    k_relu_mask<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(dh + r * ld_dh, ld_dh, ref + r * ld_ref, ld_ref, dz + r * ld_dz, ld_dz, m, cols4);
    HT_LAUNCH_CHECK(ctx);
    return (int)HT_OK;
  });
}

int ht_softmax_ce(ht_ctx* ctx, hipStream_t st, const float* logits, int64_t ld, const int32_t* labels, int64_t V,
                  int32_t C, float* grad, int64_t ld_g, LossParts* loss) {
  if (V <= 0 || C <= 0) return ht_set_err(ctx, HT_EINVAL, "loss: empty input");
  if ((ld & 3) || (ld_g & 3)) return ht_set_err(ctx, HT_ESHAPE, "loss: row pitch must be a multiple of 4");
  int lpr = 4;
  while (lpr < 64 && lpr * 4 < C) lpr *= 2;
  const unsigned nc = (unsigned)std::min<int64_t>((V + 255) / 256, COUNT_BLOCKS);
  const unsigned nb = (unsigned)std::min<int64_t>((V * lpr + 255) / 256, LOSS_BLOCKS);
  char* p = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_LOSS, (size_t)(COUNT_BLOCKS + LOSS_BLOCKS) * 8, (void**)&p));
  unsigned long long* cnt = (unsigned long long*)p;
  double* part = (double*)p + COUNT_BLOCKS;
  k_count_labelled<<<nc, 256, 0, st>>>(labels, V, cnt);
  HT_LAUNCH_CHECK(ctx);
  k_softmax_ce<<<nb, 256, 0, st>>>(logits, ld, labels, V, C, cnt, (int)nc, grad, ld_g, part, lpr);
  HT_LAUNCH_CHECK(ctx);
  *loss = LossParts{part, (int)nb, cnt, (int)nc};
  return HT_OK;
}

int ht_step(ht_ctx* ctx, hipStream_t st, const std::vector<ht_sgd_item>& items, float lr, const LossParts& parts, float* loss) {
  auto shared = [](const ht_sgd_item& a, const ht_sgd_item& b) { return a.W < b.W + b.n && b.W < a.W + a.n; };
  for (size_t i = 0; i < items.size(); ++i)
    for (size_t k = 0; k < i; ++k)
      if (shared(items[i], items[k])) HT_TRY(ht_flush_products(ctx, st));   // (parameters that share memory are updated one after the other)
  bool last = false;
  for (size_t i = 0; !last;) {
    StepBatch b{};
    for (; i < items.size() && b.n < HT_SGD_MAX; ++i) {
      const ht_sgd_item& it = items[i];
      if (it.n <= 0) continue;
      bool wait = false;
      for (int k = 0; k < b.n; ++k) wait = wait || shared(it, ht_sgd_item{b.t[k].W, nullptr, b.t[k].n});
      if (wait) break;
      StepItem s{it.W, const_cast<float*>(it.dW), it.n, nullptr, 0, 1, 0};
      for (const PendingTn& p : ctx->tn_pending) {
        for (int c = 0; c < 2; ++c)
          if (p.column[c] == it.dW) { s.P = p.P + c; s.stride = 4; s.pitch = p.n; s.slices = p.slices; }
        if (!p.column[0] && p.C == it.dW) { s.P = p.P; s.pitch = p.n; s.slices = p.slices; }
      }
      b.t[b.n] = s;
      b.first[b.n + 1] = b.first[b.n] + (unsigned)((it.n + (s.slices ? 63 : 255)) / (s.slices ? 64 : 256));
      ++b.n;
    }
    last = i >= items.size();
    const unsigned blocks = b.first[b.n] + (last ? 1 : 0);
    if (blocks == 0) continue;
    k_step<<<blocks, 256, 0, st>>>(b, lr, parts, loss);
    HT_LAUNCH_CHECK(ctx);
  }
  ctx->tn_pending.clear();
  ctx->tn_used = 0;
  ctx->tn_defer = false;
  return HT_OK;
}

int ht_fill_words(ht_ctx* ctx, hipStream_t st, void* p, size_t bytes, uint32_t value) {
  if (bytes == 0) return HT_OK;
  if (bytes & 3) return ht_set_err(ctx, HT_EINVAL, "fill: size must be a multiple of 4");
  if ((uintptr_t)p & 3) return ht_set_err(ctx, HT_EINVAL, "fill: pointer must be 4-byte aligned");
  const int64_t n = (int64_t)(bytes >> 2);
  uint32_t* w = (uint32_t*)p;
  int n_head = (int)((16 - ((uintptr_t)p & 15)) & 15) >> 2;   // words before the first 16-byte boundary
  if (n_head > n) n_head = (int)n;
  const int64_t n16 = (n - n_head) >> 2;
  const int n_tail = (int)(n - n_head - 4 * n16);
  int64_t blocks = (n16 + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (blocks < 1) blocks = 1;
  k_zero<<<(unsigned)blocks, 256, 0, st>>>((uint4*)(w + n_head), n16, w, n_head, w + n_head + 4 * n16, n_tail, value);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}
