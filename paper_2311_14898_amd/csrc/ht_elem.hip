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

// The loss in three launches whatever V is: labelled vertices per block; gradient rows and per-block loss sums; their total.
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

__global__ void __launch_bounds__(256) k_finish_loss(const double* __restrict__ part, int n, const unsigned long long* __restrict__ cnt,
                                                     int n_cnt, float* __restrict__ loss) {
  __shared__ double sh[256];
  __shared__ unsigned long long shc[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += part[i];
  s = block_sum(s, sh);
  const unsigned long long T = block_sum((int)threadIdx.x < n_cnt ? cnt[threadIdx.x] : 0ull, shc);
  if (threadIdx.x == 0) *loss = T > 0 ? (float)(s / (double)T) : 0.f;
}

// One launch for all parameters of a model (a launch each costs its 4 us whatever the size): tensor t has the blocks from
// first[t] on.
struct SgdBatch {
  int n;
  unsigned first[HT_SGD_MAX + 1];
  ht_sgd_item t[HT_SGD_MAX];
};
__global__ void k_sgd(SgdBatch b, float lr) {
  int k = 0;
  while (k + 1 < b.n && blockIdx.x >= b.first[k + 1]) ++k;
  const int64_t i = (int64_t)(blockIdx.x - b.first[k]) * blockDim.x + threadIdx.x;
  if (i < b.t[k].n) b.t[k].W[i] = b.t[k].W[i] - lr * b.t[k].dW[i];
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
                  int32_t C, float* grad, int64_t ld_g, float* loss_dev) {
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
  k_finish_loss<<<1, 256, 0, st>>>(part, (int)nb, cnt, (int)nc, loss_dev);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}

int ht_sgd(ht_ctx* ctx, hipStream_t st, const std::vector<ht_sgd_item>& items, float lr) {
  for (size_t i = 0; i < items.size();) {
    SgdBatch b{};
    for (; i < items.size() && b.n < HT_SGD_MAX; ++i) {
      const ht_sgd_item& it = items[i];
      if (it.n <= 0) continue;
      bool shared = false;      // (parameters that share memory are updated one after the other)
      for (int k = 0; k < b.n; ++k) shared = shared || (it.W < b.t[k].W + b.t[k].n && b.t[k].W < it.W + it.n);
      if (shared) break;
      b.t[b.n] = it;
      b.first[b.n + 1] = b.first[b.n] + (unsigned)((it.n + 255) / 256);
      ++b.n;
    }
    if (b.n == 0) continue;
    k_sgd<<<b.first[b.n], 256, 0, st>>>(b, lr);
    HT_LAUNCH_CHECK(ctx);
  }
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
