// Dense transform of the update stage (Eq. 2: linear + ReLU) and its gradient
// GEMMs (Sec. 2.3: grad W = a^T (ReLU'(aW) * grad h'), grad a = grad z W^T) on
// the fp32 matrix cores (v_mfma_f32_32x32x2_f32), LDS-tiled for 64-wide waves.  grad W with
// wide outputs runs on the bf16 matrix cores in fp32 precision (k_split_tn).
//
//   NN: C[M x N] = A[M x K] Bp        M = chunk rows (tall), K, N = layer widths
//   TN: C[K x N] = A[M x K]^T B[M x N] reduction over the tall M, cut into
//       slices whose partial tiles are added in slice order (no atomics).
// The small operand W is first packed into a zero-padded tile-aligned copy.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "ht_internal.h"

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int BK = 16;        // reduction depth of one LDS stage
constexpr int BM = 128;       // rows of A per block (NN) / output rows per block (TN)
// Rows up to which a product may read W as it is, a launch less (2.5 us and the gap before the next one).  Its single loads and bounds tests cost about
// 0.1 us a step of 16 of the reduction, in each round of blocks over the chip, so that it pays for short chains alone.  In place - packed (us), layers
// without edges, 300 | 3,000 | 10,000 | 20,000 | 32,768 rows: 128 x 256 -1.5 | -1.3 | -1.5 | -0.3 | +1.2, 256 x 256
// -0.3 | 0.0 | -1.0 | +1.0 | +3.7, 602 x 256 +3.7 | +3.3 | +2.8 | +8.6 | +10.5, 256 x 41 -1.4 | -0.7 | -1.4 | -1.7 | -2.2;
// the transpose, 256 columns to 128 +0.7 | +1.6 | 0.0 | +0.4 | +3.0, 129 to 300 -0.8 | -1.2 | -2.2 | +0.2 | +2.7.
constexpr int64_t HT_PACK_ROWS = 32768;
constexpr int HT_PACK_CHAIN = 192, HT_PACK_CHAIN_NARROW = 512;   // (up to 64 columns a block stores half as much of W at a step)
inline bool reads_w_in_place(int64_t M, int32_t K, int32_t N, bool transposed) {
  if (M > HT_PACK_ROWS) return false;
  const int64_t blocks = (M + BM - 1) / BM * (N > 64 ? (N + 127) / 128 : 1);
  return K * std::max<int64_t>(blocks, 256) <= 256 * (N <= 64 && !transposed ? HT_PACK_CHAIN_NARROW : HT_PACK_CHAIN);
}
// Partial tiles of an epoch's products up to which they are added up by its last launch (each keeps its own until then).  Beyond it the
// products take far longer than the launches that are saved.
constexpr size_t HT_DEFER_BYTES = (size_t)64 << 20;
constexpr int LDA_S = BK + 1; // LDS pitch of the row-major A tile (NN): odd, conflict-free column reads

__device__ __forceinline__ float4 ld4g(const float* p) { return *reinterpret_cast<const float4*>(p); }

// Pack W[K x N] (row-major, dense) into Bp[Kp x Np] zero-padded; transpose = 1 packs W^T.
__global__ void k_pack_b(const float* __restrict__ W, int K, int N, int transpose, float* __restrict__ Bp, int Kp,
                         int Np) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)Kp * Np) return;
  const int r = (int)(i / Np), c = (int)(i % Np);
  float v = 0.f;
  if (!transpose) {
    if (r < K && c < N) v = W[(int64_t)r * N + c];
  } else {  // Bp[r][c] = W[c][r], W is [N' x K'] = [c-range x r-range]
    if (r < N && c < K) v = W[(int64_t)c * N + r];
  }
  Bp[i] = v;
}

// C = A Bp (+ReLU).  A [M x K] pitch lda (columns >= K are never used as data),
// Bp [Kp x Np] padded, or W as it is: PACKED, AS_IS (W [K x N]) or TRANSPOSED (W [N x K]).  Block: 256 threads = WM x WN waves, wave tile
// (TI*32) x (TJ*32).
enum { PACKED, AS_IS, TRANSPOSED };
template <int BN, int WM, int WN, int TI, int TJ, int FORM>
__global__ void __launch_bounds__(256) k_gemm_nn(const float* __restrict__ A, int64_t lda,
                                                 const float* __restrict__ Bp, int Np, float* __restrict__ C,
                                                 int64_t ldc, int64_t M, int K, int N, int relu) {
  static_assert(WM * WN == 4 && WM * TI * 32 == BM && WN * TJ * 32 == BN, "tile shape");
  __shared__ float As[BM * LDA_S];
  __shared__ float Bs[BK * (BN + 4)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, half = lane >> 5;
  const int64_t m0 = (int64_t)blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;

  v16f acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // The tiles of step k0 + BK are fetched into registers while the matrix cores work on step k0.
  constexpr int NA = BM * 4 / 256, NB = BK * BN / 4 / 256;
  static_assert(NA * 256 == BM * 4 && NB * 256 == BK * BN / 4, "tile loads must divide among 256 threads");
  float4 ra[NA], rb[NB];
  // interior blocks (all BM rows exist) take their full K-steps without any bounds test
  const bool interior = m0 + BM <= M;
  auto fetch = [&](int k0) {
    if (interior && k0 + BK <= K) {
#pragma unroll
      for (int u = 0; u < NA; ++u) {
        const int f = tid + u * 256;
        const int row = f >> 2, kv = (f & 3) * 4;
        ra[u] = ld4g(A + (m0 + row) * lda + k0 + kv);
      }
    } else {
#pragma unroll
      for (int u = 0; u < NA; ++u) {
        const int f = tid + u * 256;
        const int row = f >> 2, kv = (f & 3) * 4;
        const int64_t gm = m0 + row;
        const int gk = k0 + kv;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (gm < M && gk < K) {
          v = ld4g(A + gm * lda + gk);
          if (gk + 1 >= K) v.y = 0.f;
          if (gk + 2 >= K) v.z = 0.f;
          if (gk + 3 >= K) v.w = 0.f;
        }
        ra[u] = v;
      }
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int f = tid + u * 256;
      if (FORM == PACKED) {
        const int kr = f / (BN / 4), nv = (f % (BN / 4)) * 4;
        rb[u] = ld4g(Bp + (int64_t)(k0 + kr) * Np + n0 + nv);
      } else {   // four columns of a row of W, or four rows of a column of its transpose: contiguous either way, at any alignment
        const int k = FORM == AS_IS ? k0 + f / (BN / 4) : k0 + (f & 3) * 4, n = FORM == AS_IS ? n0 + (f % (BN / 4)) * 4 : n0 + (f >> 2);
        const float* p = FORM == AS_IS ? Bp + (int64_t)k * N + n : Bp + (int64_t)n * K + k;
        const int left = k < K && n < N ? (FORM == AS_IS ? N - n : K - k) : 0;
        rb[u].x = left > 0 ? p[0] : 0.f;
        rb[u].y = left > 1 ? p[1] : 0.f;
        rb[u].z = left > 2 ? p[2] : 0.f;
        rb[u].w = left > 3 ? p[3] : 0.f;
      }
    }
  };
  auto stash = [&]() {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int f = tid + u * 256;
      const int row = f >> 2, kv = (f & 3) * 4;
      float* d = As + row * LDA_S + kv;
      d[0] = ra[u].x; d[1] = ra[u].y; d[2] = ra[u].z; d[3] = ra[u].w;
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int f = tid + u * 256;
      if (FORM == TRANSPOSED) {
        float* d = Bs + (f & 3) * 4 * (BN + 4) + (f >> 2);
        d[0] = rb[u].x; d[BN + 4] = rb[u].y; d[2 * (BN + 4)] = rb[u].z; d[3 * (BN + 4)] = rb[u].w;
      } else {
        const int kr = f / (BN / 4), nv = (f % (BN / 4)) * 4;
        *reinterpret_cast<float4*>(Bs + kr * (BN + 4) + nv) = rb[u];
      }
    }
  };
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
    stash();
    __syncthreads();
    if (k0 + BK < K) fetch(k0 + BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 2) {
      float af[TI], bf[TJ];
#pragma unroll
      for (int i = 0; i < TI; ++i) af[i] = As[(wm * TI * 32 + i * 32 + l32) * LDA_S + kk + half];
#pragma unroll
      for (int j = 0; j < TJ; ++j) bf[j] = Bs[(kk + half) * (BN + 4) + wn * TJ * 32 + j * 32 + l32];
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  // D layout of the 32x32 tile: lane holds column l32, rows (e/4)*8 + half*4 + e%4
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int gc = n0 + wn * TJ * 32 + j * 32 + l32;
      if (gc >= N) continue;
      float* cp = C + (m0 + wm * TI * 32 + i * 32 + half * 4) * ldc + gc;
      if (interior && relu < 2) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          float v = acc[i][j][e];
          if (relu) v = v > 0.f ? v : 0.f;
          cp[((e >> 2) * 8 + (e & 3)) * ldc] = v;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int64_t gr = m0 + wm * TI * 32 + i * 32 + (e >> 2) * 8 + half * 4 + (e & 3);
          if (gr < M) {
            float v = acc[i][j][e];
            if (relu & 1) v = v > 0.f ? v : 0.f;
            if (relu & 2) v += C[gr * ldc + gc];
            C[gr * ldc + gc] = v;
          }
        }
      }
    }
}

// C = A W (+ReLU), or A W^T, with the block's columns of W in LDS and the rows of A straight to registers, for widths that k_gemm_nn would pad
// (rows_shape).  A wave owns 32 rows x TJ tiles of 32 columns, takes strip after strip of rows, and waits for no other wave once W is there; its rows' pieces
// come NBUF steps of 32 values ahead, across strips.  Lane l32 + 32 half holds row l32 and the values 8 q + 4 half .. + 3 of a step (a load covers 32
// contiguous bytes of each row, a step its whole cache line); two exchanges between the halves of the wave turn four registers with the values 0 .. 3 | 4 .. 7
// into 0 | 1, 2 | 3, 4 | 5, 6 | 7, so that an element is summed up in the order of k_gemm_nn, to the same bits (0.5 % of a layer of 60 k rows, 67 x 129).  W lies in LDS as fours of every second value of the
// reduction, 0, 2, 4, 6 and 1, 3, 5, 7 of each eight: what a lane multiplies with them is one read.
// What bounds it: the fp32 matrix cores (1 M rows, 416 x 288 122 TFLOP/s of the 155 that an fp32 product of the vendor's reaches; 2.45 M, 256 x 256, which rows_shape leaves to k_gemm_nn,
// kept them 79 % busy, as k_gemm_nn does, and 85 without loads and stores), for narrow results the rows' reads (1 M x 64 x 20: 5 TB/s), and where W does not fit the LDS, reading the rows once
// for every tile or two.
constexpr int RS = 32;                       // values of a step
constexpr int ROWS_LDS = 160 << 10;          // LDS of a CU
constexpr int rows_lds(int K, int tj) { return (K + 7) / 8 * 2 * (tj * 32 + 1) * 16; }   // (a pitch of odd float4s: the transposed W is stored across rows)

template <int TJ, int NBUF, bool T>
__global__ void __launch_bounds__(512) k_rows_w(const float* __restrict__ A, int64_t lda, const float* __restrict__ W, float* __restrict__ C,
                                                int64_t ldc, int64_t M, int K, int N, int relu) {
  extern __shared__ float4 Bs[];
  constexpr int NT = TJ * 32, P = NT + 1;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int waves = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = blockIdx.y * NT, K4 = (K + 7) / 8 * 2;
  const int64_t strips = (M + 31) / 32, stride = (int64_t)gridDim.x * waves;
  int64_t strip = (int64_t)blockIdx.x * waves + wave;
  const int steps = (K + RS - 1) / RS;

  float4 buf[NBUF][4];
  auto row_of = [&](int64_t s) {   // (rows behind the last: the last again, not stored)
    const int64_t r = s * 32 + l32;
    return A + (r < M ? r : M - 1) * lda + half * 4;
  };
  auto fetch = [&](float4* b, const float* row, int c) {
    const float* p = row + c * RS;
    if ((c + 1) * RS <= K) {
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = ld4g(p + q * 8);
    } else {   // (what lies behind a row's last value is not looked at: it may be anything)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        int left = K - (c * RS + q * 8 + half * 4);
        asm volatile("" : "+v"(left));   // (or the conditions of every step's end are made before the loop, and kept)
        const float4 v = ld4g(p + (left > 0 ? q * 8 : (K - 1 - c * RS - half * 4) & ~3));
        auto kept = [&](float x, int i) { return __int_as_float(__float_as_int(x) & ((i - left) >> 31)); };
        b[q] = make_float4(kept(v.x, 0), kept(v.y, 1), kept(v.z, 2), kept(v.w, 3));
      }
    }
  };
  const float* row = row_of(strip < strips ? strip : strips - 1);
#pragma unroll
  for (int u = 0; u < NBUF; ++u)
    if (u < steps) fetch(buf[u], row, u);
  // W: fours along the reduction, one after the other along the columns of W, or eight along a row of its transpose, as it lies in memory
  const int n_w = (T ? (K4 + 7) / 8 * 8 : K4) * NT;
  const bool vec = T && (K & 3) == 0 && (reinterpret_cast<uintptr_t>(W) & 15) == 0;
  for (int i0 = tid; i0 < n_w; i0 += 4 * blockDim.x) {
    float4 v[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int i = i0 + x * blockDim.x, k = (T ? i / (8 * NT) * 8 + i % 8 : i / NT) * 4, n = n0 + (T ? i / 8 % NT : i % NT);
      v[x] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i >= n_w || n >= N || k >= K) continue;
      const float* p = T ? W + (int64_t)n * K + k : W + (int64_t)k * N + n;
      if (vec) {
        v[x] = ld4g(p);
      } else {
        const int d = T ? 1 : N;
        v[x].x = p[0];
        if (k + 1 < K) v[x].y = p[d];
        if (k + 2 < K) v[x].z = p[2 * (int64_t)d];
        if (k + 3 < K) v[x].w = p[3 * (int64_t)d];
      }
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int i = i0 + x * blockDim.x, k4 = T ? i / (8 * NT) * 8 + i % 8 : i / NT;
      if (i >= n_w || k4 >= K4) continue;
      float4* to = Bs + (k4 & ~1) * P + (T ? i / 8 % NT : i % NT);
      reinterpret_cast<float2*>(to)[k4 & 1] = make_float2(v[x].x, v[x].z);
      reinterpret_cast<float2*>(to + P)[k4 & 1] = make_float2(v[x].y, v[x].w);
    }
  }
  __syncthreads();
  for (; strip < strips; strip += stride) {
    v16f acc[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
    const int64_t m0 = strip * 32;
    const bool more = strip + stride < strips;
    const float* next = more ? row_of(strip + stride) : row;
    for (int c0 = 0; c0 < steps; c0 += NBUF) {
#pragma unroll
      for (int u = 0; u < NBUF; ++u) {
        const int c = c0 + u;
        if (c >= steps) break;
        const float4* B = Bs + (c * 8 + half) * P + l32;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (q > 0 && c * RS + q * 8 >= K) break;
          float4 b[TJ];
#pragma unroll
          for (int j = 0; j < TJ; ++j) b[j] = B[q * 2 * P + j * 32];
          const float4 v = buf[u][q];
          const auto xy = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.x), __float_as_uint(v.y), false, false);
          const auto zw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.z), __float_as_uint(v.w), false, false);
          const float4 a = make_float4(__uint_as_float(xy[0]), __uint_as_float(zw[0]), __uint_as_float(xy[1]), __uint_as_float(zw[1]));
#pragma unroll
          for (int j = 0; j < TJ; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b[j].x, acc[j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < TJ; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b[j].y, acc[j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < TJ; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b[j].z, acc[j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < TJ; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b[j].w, acc[j], 0, 0, 0);
        }
        // what takes this piece's place: of this strip, or of the next
        if (c + NBUF < steps) fetch(buf[u], row, c + NBUF);
        else if (more) fetch(buf[u], next, u);
      }
    }
    // D layout of a 32x32 tile: lane holds column l32, rows (e/4)*8 + half*4 + e%4
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int gc = n0 + j * 32 + l32;
      if (gc >= N) continue;
      float* cp = C + (m0 + half * 4) * ldc + gc;
      if (m0 + 32 <= M && relu < 2) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          float v = acc[j][e];
          if (relu) v = v > 0.f ? v : 0.f;
          cp[((e >> 2) * 8 + (e & 3)) * ldc] = v;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = (e >> 2) * 8 + (e & 3);
          if (m0 + half * 4 + r < M) {
            float v = acc[j][e];
            if (relu & 1) v = v > 0.f ? v : 0.f;
            if (relu & 2) v += cp[r * ldc];
            cp[r * ldc] = v;
          }
        }
      }
    }
    row = next;
  }
}

// MASKED: B counts where mask.ref is positive, and is 0 elsewhere (dz, where nothing else reads it: 2.45 M rows, 100 x 256, with a pass that writes it 2.61 ms, so 1.64; 233 k, 602 x
// 256 720 us, 668).
// Partial tile of C[K x N] = A[M x K]^T B[M x N] over the M-slice blockIdx.z (rows tab[2z] .. tab[2z + 1], or slice_rows each).
// P[slice][K x N] dense.  Block tile: BM output rows (k) x BN output columns.
// What bounds it is the loads of a step of 16 rows, PD steps of which are in flight: up to 64 columns two, wider ones, whose accumulators leave fewer registers, one.  us, loads
// with bounds tests one step ahead | without | two ahead | four | six, at rows x K x N: 2.45 M x 256 x 47 973 | - | 849 | 885 | 841, 1 M x 64 x 64 221 | - | 196 | 215 | 201, 60 k x 129
// x 60 42 | - | 35 | 37 | 38, 20 k x 50 x 33 17.0 | - | 16.5 | 17.8 | 17.8; wider: 20 k x 256 x 100 32 | 26 | 27 (| 27 three), 8 k x 200 x 100 22 | 19 | 20.
template <int BN, int WM, int WN, int TI, int TJ, int PD, bool MASKED>
__global__ void __launch_bounds__(256) k_gemm_tn(const float* __restrict__ A, int64_t lda,
                                                 const float* __restrict__ B, int64_t ldb, ReluMask mask, float* __restrict__ P,
                                                 int64_t M, int K, int N, int64_t slice_rows,
                                                 const int64_t* __restrict__ tab) {
  static_assert(WM * WN == 4 && WM * TI * 32 == BM && WN * TJ * 32 == BN, "tile shape");
  __shared__ float As[BK * (BM + 4)];
  __shared__ float Bs[BK * (BN + 4)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, half = lane >> 5;
  const int kc0 = blockIdx.x * BM;  // first output row (a column of A)
  const int n0 = blockIdx.y * BN;
  const int64_t ms = tab ? tab[2 * (int64_t)blockIdx.z] : (int64_t)blockIdx.z * slice_rows;
  const int64_t me = tab ? tab[2 * (int64_t)blockIdx.z + 1] : (ms + slice_rows) < M ? (ms + slice_rows) : M;

  v16f acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  constexpr int NA = BK * BM / 4 / 256, NB = BK * BN / 4 / 256;
  static_assert(NA * 256 == BK * BM / 4 && NB * 256 == BK * BN / 4, "tile loads must divide among 256 threads");
  // The tiles of PD steps are on their way at once.  Loads have no condition (outside the operands they read the last row, the last columns again), so that the
  // waits count only the loads of the step that is next; what lies outside is cleared on the way into LDS.
  float4 ra[PD][NA], rb[PD][NB], rm[MASKED ? PD : 1][NB];
  const bool full_a = kc0 + BM <= K, full_b = n0 + BN <= N;
  const int last_a = (K - 1) & ~3, last_b = (N - 1) & ~3;
  auto fetch = [&](int64_t mm0, float4* pa, float4* pb, float4* pm) {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int f = tid + u * 256, c = kc0 + (f % (BM / 4)) * 4;
      const int64_t r = mm0 + f / (BM / 4);
      pa[u] = ld4g(A + (r < me ? r : me - 1) * lda + (c < last_a ? c : last_a));
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int f = tid + u * 256, c = n0 + (f % (BN / 4)) * 4;
      const int64_t r = mm0 + f / (BN / 4);
      pb[u] = ld4g(B + (r < me ? r : me - 1) * ldb + (c < last_b ? c : last_b));
      if (MASKED) pm[u] = ld4g(mask.ref + (r < me ? r : me - 1) * mask.ld + (c < last_b ? c : last_b));
    }
  };
  auto inside = [&](float4 v, bool row, int c, int n) {
    const int left = row ? n - c : 0;
    return make_float4(left > 0 ? v.x : 0.f, left > 1 ? v.y : 0.f, left > 2 ? v.z : 0.f, left > 3 ? v.w : 0.f);
  };
  auto stash = [&](int64_t mm0, const float4* pa, const float4* pb, const float4* pm) {
    const bool full_m = mm0 + BK <= me;
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int f = tid + u * 256;
      const int mr = f / (BM / 4), cv = (f % (BM / 4)) * 4;
      *reinterpret_cast<float4*>(As + mr * (BM + 4) + cv) = full_m && full_a ? pa[u] : inside(pa[u], mm0 + mr < me, kc0 + cv, K);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int f = tid + u * 256;
      const int mr = f / (BN / 4), cv = (f % (BN / 4)) * 4;
      float4 v = pb[u];
      if (MASKED) v = make_float4(pm[u].x > 0.f ? v.x : 0.f, pm[u].y > 0.f ? v.y : 0.f, pm[u].z > 0.f ? v.z : 0.f, pm[u].w > 0.f ? v.w : 0.f);
      if (!(full_m && full_b)) v = inside(v, mm0 + mr < me, n0 + cv, N);
      *reinterpret_cast<float4*>(Bs + mr * (BN + 4) + cv) = v;
      if (MASKED && mask.to && mm0 + mr < me && n0 + cv < N) *reinterpret_cast<float4*>(mask.to + (mm0 + mr) * mask.to_ld + n0 + cv) = v;
    }
  };
  if (ms < me) {
#pragma unroll
    for (int u = 0; u < PD; ++u) fetch(ms + u * BK, ra[u], rb[u], rm[MASKED ? u : 0]);
  }
  for (int64_t m1 = ms; m1 < me; m1 += PD * BK) {
#pragma unroll
    for (int u = 0; u < PD; ++u) {
      const int64_t mm0 = m1 + u * BK;
      if (mm0 >= me) break;
      stash(mm0, ra[u], rb[u], rm[MASKED ? u : 0]);
      __syncthreads();
      fetch(mm0 + PD * BK, ra[u], rb[u], rm[MASKED ? u : 0]);
#pragma unroll
      for (int kk = 0; kk < BK; kk += 2) {
        float af[TI], bf[TJ];
#pragma unroll
        for (int i = 0; i < TI; ++i) af[i] = As[(kk + half) * (BM + 4) + wm * TI * 32 + i * 32 + l32];
#pragma unroll
        for (int j = 0; j < TJ; ++j) bf[j] = Bs[(kk + half) * (BN + 4) + wn * TJ * 32 + j * 32 + l32];
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i], bf[j], acc[i][j], 0, 0, 0);
      }
      __syncthreads();
    }
  }
  float* Ps = P + (int64_t)blockIdx.z * K * N;
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int gc = n0 + wn * TJ * 32 + j * 32 + l32;
      if (gc >= N) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int gr = kc0 + wm * TI * 32 + i * 32 + (e >> 2) * 8 + half * 4 + (e & 3);
        if (gr < K) Ps[(int64_t)gr * N + gc] = acc[i][j][e];
      }
    }
}

// ---- A^T B on the bf16 matrix cores, in fp32 precision.
// Every fp32 value is split into three bf16 values whose sum it is (x = x0 + x1 + x2, each the rounding of what the ones before
// leave: |x1| <= 2^-8 |x|, |x2| <= 2^-17 |x|), and eight of the nine partial products are added in fp32, smallest first; x2 y2 is
// below 2^-33 of the product.  (Without x1 y2 and x2 y1, up to 2^-24 of it together, single products were off by up to 1.75 x
// 2^-24, now by 1.002 x; in fp32 by 1 x.)  The operands are scaled by 2^24 first and the sums by 2^-48 at the end, both exact: the
// last part of every fp32 number, subnormal ones too, is then a normal bf16 (unscaled, factors below 2^-110 lost low bits).
// Eight 32x32x16 bf16 steps take 256 clocks where eight 32x32x2 fp32 steps take 512, and fewer fp32 sums are rounded.  Relative
// errors against fp64 (2-norm; fp32 products | these): 60,000 rows, 256 x 128 4.0e-7 | 2.9e-7, half of them masked 3.5e-7 | 2.9e-7,
// 233 k rows, 602 x 256 8.7e-7 | 3.4e-7 (with the small products summed apart: thousands of rows, rounded eight times per step).
// fp32 -> these: 2.45 M rows, 100 x 256 1.60 -> 1.28 ms, 256 x 256 2.84 -> 2.69; 1 M rows, 160 x 128 0.62 -> 0.53; 233 k rows,
// 602 x 256 0.73 -> 0.67; 116 k rows, 301 x 129 238 -> 197 us; 60 k rows, 129 x 67 69 -> 50.
// (A W and dZ W^T stay in fp32.  Split in the same way, with two sums, they are as exact, but take 2.72 ms instead of 2.88 and 2.97
// instead of 2.87 at 2.45 M rows, 256 x 256; with one sum, 2.47 and 2.54 ms, the matrix cores' rounding of small addends is
// felt: single products off by up to 2^-23, and sums over rows that a ReLU has masked 15 % further off than in fp32.)
// Values that are not finite, or whose scaled products are not (beyond about 2^80), would leave NaN where an fp32 product has an
// infinity or a number: a block whose tile holds anything but finite numbers computes it again on the fp32 matrix cores.  (233 k rows, 602 x 256:
// 0.8 ms; 1.4 with one NaN in A, 2.0 with whole columns of them: element by element they took 16 and 46.)
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
constexpr int SK = 32;                       // reduction depth of one LDS stage: two steps of 16
constexpr int SB = BM * 16;                  // bf16 per [128 rows][16] block of a stage [plane][step]

constexpr float SPLIT_SCALE = 0x1p24f, SPLIT_UNSCALE = 0x1p-48f;   // of each operand; of the sums

__device__ __forceinline__ void split3(float x, __bf16* p) {
  x *= SPLIT_SCALE;
  p[0] = (__bf16)x;
  const float r = x - (float)p[0];
  p[1] = (__bf16)r;
  p[2] = (__bf16)(r - (float)p[1]);
}
// a wave's 64 x 64 part of the block's 128 x 128; the seven small partial products have sums of their own
struct SplitTile {
  v16f acc[2][2], low[2][2];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = 0.f;
  }
  __device__ __forceinline__ void join() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] += low[i][j][e];
  }
  // one LDS stage; As, Bs: [plane][step][row][16]
  __device__ __forceinline__ void stage(const __bf16* As, const __bf16* Bs, int wm, int wn, int l32, int half) {
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      v8bf a[3][2], b[3][2];
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          a[p][i] = *reinterpret_cast<const v8bf*>(As + (p * 2 + st) * SB + (wm * 64 + i * 32 + l32) * 16 + half * 8);
          b[p][i] = *reinterpret_cast<const v8bf*>(Bs + (p * 2 + st) * SB + (wn * 64 + i * 32 + l32) * 16 + half * 8);
        }
      constexpr int PA[8] = {2, 1, 2, 0, 1, 1, 0, 0}, PB[8] = {1, 2, 0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            v16f& s = q < 7 ? low[i][j] : acc[i][j];
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[q]][i], b[PB[q]][j], s, 0, 0, 0);
          }
    }
  }
  __device__ __forceinline__ bool all_finite() const {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) ok = ok && fabsf(acc[i][j][e]) < INFINITY;
    return ok;
  }
  __device__ __forceinline__ void unscale() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] *= SPLIT_UNSCALE;
  }
  // The tile again on the fp32 matrix cores: a(row, k) and b(column, k) for k in [k0, k1), 0 outside the operands.  As, Bs: [BK][BM + 4]
  template <class FA, class FB>
  __device__ __forceinline__ void in_fp32(float* As, float* Bs, int64_t k0, int64_t k1, int wm, int wn, int l32, int half, FA a, FB b) {
    constexpr int P = BM + 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    const int c = threadIdx.x & (BM - 1), h = threadIdx.x >> 7;
    for (int64_t k = k0; k < k1; k += BK) {
#pragma unroll 1
      for (int u = h; u < BK; u += 2) {
        As[u * P + c] = k + u < k1 ? a(c, k + u) : 0.f;
        Bs[u * P + c] = k + u < k1 ? b(c, k + u) : 0.f;
      }
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < BK; kk += 2) {
        float af[2], bf[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          af[i] = As[(kk + half) * P + wm * 64 + i * 32 + l32];
          bf[i] = Bs[(kk + half) * P + wn * 64 + i * 32 + l32];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i], bf[j], acc[i][j], 0, 0, 0);
      }
      __syncthreads();
    }
  }
};
static_assert(BK * (BM + 4) * sizeof(float) <= 6 * SB * sizeof(__bf16), "the fp32 stages fit where the split ones were");

// Partial tile of C[K x N] = A^T B over a slice of rows, as k_gemm_tn
template <bool MASKED>
__global__ void __launch_bounds__(256, 2) k_split_tn(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, ReluMask mask,
                                                  float* __restrict__ P, int64_t M, int K, int N, int64_t slice_rows,
                                                  const int64_t* __restrict__ tab) {
  __shared__ __attribute__((aligned(16))) __bf16 As[6 * SB];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[6 * SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, half = lane >> 5;
  const int kc0 = blockIdx.x * BM, n0 = blockIdx.y * 128;
  const int64_t ms = tab ? tab[2 * (int64_t)blockIdx.z] : (int64_t)blockIdx.z * slice_rows;
  const int64_t me = tab ? tab[2 * (int64_t)blockIdx.z + 1] : (ms + slice_rows) < M ? (ms + slice_rows) : M;
  // a thread takes one column of either operand and 16 rows: its values are consecutive along the reduction, as the LDS layout
  // wants them, and a wave's loads cover 256 consecutive bytes of a row
  // (the row is the same in all lanes: scalar base, 32-bit lane offset)
  const int c = tid & 127, st = __builtin_amdgcn_readfirstlane(tid >> 7);
  const bool has_a = kc0 + c < K, has_b = n0 + c < N;
  const unsigned ca = has_a ? kc0 + c : 0, cb = has_b ? n0 + c : 0;
  float ra[16], rb[16], rm[MASKED ? 16 : 1];
  auto fetch = [&](int64_t mm) {
    const int64_t r0 = mm + st * 16;
    // (row pointers that step along: kept for all rows of a stage, they take more scalar registers than there are)
    const float *pa = A + r0 * lda, *pb = B + r0 * ldb, *pm = MASKED ? mask.ref + r0 * mask.ld : nullptr;
    asm volatile("" : "+s"(pa), "+s"(pb), "+s"(pm));
    const int64_t left = me - r0;
    if (left >= 16) {
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        ra[u] = pa[ca];
        rb[u] = pb[cb];
        if (MASKED) rm[u] = pm[cb];
        pa += lda;
        pb += ldb;
        if (MASKED) pm += mask.ld;
      }
    } else {
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        ra[u] = u < left ? pa[ca] : 0.f;
        rb[u] = u < left ? pb[cb] : 0.f;
        if (MASKED) rm[u] = u < left ? pm[cb] : 0.f;
        pa += lda;
        pb += ldb;
        if (MASKED) pm += mask.ld;
      }
    }
  };
  auto masked = [&] {   // (when the loads are there, not where they are issued)
    if (MASKED)
#pragma unroll
      for (int u = 0; u < 16; ++u) rb[u] = rm[u] > 0.f ? rb[u] : 0.f;
  };
  auto put = [&](const float* v, bool has, __bf16* S) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v8bf o[3];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        __bf16 p[3];
        split3(has ? v[h * 8 + u] : 0.f, p);
        o[0][u] = p[0];
        o[1][u] = p[1];
        o[2][u] = p[2];
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) *reinterpret_cast<v8bf*>(S + (q * 2 + st) * SB + c * 16 + h * 8) = o[q];
    }
  };
  SplitTile t;
  t.clear();
  if (ms < me) fetch(ms);
  for (int64_t mm = ms; mm < me; mm += SK) {
    put(ra, has_a, As);
    masked();
    put(rb, has_b, Bs);
    __syncthreads();
    if (mm + SK < me) fetch(mm + SK);
    t.stage(As, Bs, wm, wn, l32, half);
    __syncthreads();
  }
  t.join();
  if (__syncthreads_or(!t.all_finite()))
    t.in_fp32(reinterpret_cast<float*>(As), reinterpret_cast<float*>(Bs), ms, me, wm, wn, l32, half,
              [&](int r, int64_t m) { return kc0 + r < K ? A[m * lda + kc0 + r] : 0.f; },
              [&](int q, int64_t m) { return n0 + q < N && (!MASKED || mask.ref[m * mask.ld + n0 + q] > 0.f) ? B[m * ldb + n0 + q] : 0.f; });
  else
    t.unscale();
  float* Ps = P + (int64_t)blockIdx.z * K * N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int gc = n0 + wn * 64 + j * 32 + l32;
      if (gc >= N) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int gr = kc0 + wm * 64 + i * 32 + (e >> 2) * 8 + half * 4 + (e & 3);
        if (gr < K) Ps[(int64_t)gr * N + gc] = t.acc[i][j][e];
      }
    }
}

// C[i] (+)= the slices' partial sums, one after the other in slice order.  The adds of one element are a chain, the loads are
// not: a block takes E elements, its four waves bring 4,096 values at a time into LDS (16 loads in flight per lane) while E
// lanes add those before them.  (One thread per element that loads as it adds took 43 us where this takes 15.)  What bounds it: the loads that the blocks there are
// have in flight, so tiles of few elements go 16 to a block: a layer of 1 M vertices, 64 x 64 (3,906 slices, 69 us of it) 3.084 -> 3.047 ms.
// Large ones stay at 64, whose reads are whole cache lines: an epoch of 233 k vertices, 602-256-41 12.63 | 12.65 ms with 64 | 16.
template <int E>
__global__ void __launch_bounds__(256) k_reduce_slices(const float* __restrict__ P, int64_t n, int slices, int accumulate,
                                                       float* __restrict__ C) {
  constexpr int AT_ONCE = 256 / E, STAGE = 16 * AT_ONCE, PITCH = STAGE + 4;
  __shared__ __attribute__((aligned(16))) float tile[2][E][PITCH];
  const int e = threadIdx.x % E, sl = threadIdx.x / E;
  const int64_t i = (int64_t)blockIdx.x * E + e;
  const bool adds = threadIdx.x < E && i < n;
  float v[16];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int k = s0 + q * AT_ONCE + sl;
      v[q] = (k < slices && i < n) ? P[(int64_t)k * n + i] : 0.f;
    }
  };
  float s = accumulate && adds ? C[i] : 0.f;
  fetch(0);
  for (int s0 = 0, b = 0; s0 < slices; s0 += STAGE, b ^= 1) {
#pragma unroll
    for (int q = 0; q < 16; ++q) tile[b][e][q * AT_ONCE + sl] = v[q];
    if (s0 + STAGE < slices) fetch(s0 + STAGE);
    __syncthreads();   // (the other buffer was added before this barrier's turn came round)
    if (adds) {
      const int m = slices - s0;
      if (m >= STAGE) {
#pragma unroll 4
        for (int k = 0; k < STAGE; k += 4) {
          const float4 x = *reinterpret_cast<const float4*>(&tile[b][e][k]);
          s += x.x;
          s += x.y;
          s += x.z;
          s += x.w;
        }
      } else {
        for (int k = 0; k < m; ++k) s += tile[b][e][k];
      }
    }
  }
  if (adds) C[i] = s;
}

constexpr int REDUCE_WIDE = 512;   // blocks of 64 elements from which those are taken
void launch_reduce(hipStream_t st, const float* P, int64_t n, int slices, int accumulate, float* C) {
  if (n >= REDUCE_WIDE * 64) k_reduce_slices<64><<<(unsigned)((n + 63) / 64), 256, 0, st>>>(P, n, slices, accumulate, C);
  else k_reduce_slices<16><<<(unsigned)((n + 15) / 16), 256, 0, st>>>(P, n, slices, accumulate, C);
}

// The first two of every four values, each a vector of its own (the same sums).
__global__ void __launch_bounds__(256) k_reduce_columns(const float* __restrict__ P, int64_t n, int slices, float* __restrict__ c0, float* __restrict__ c1) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n / 4) return;
  float a = 0.f, b = 0.f;
  for (int s = 0; s < slices; ++s) {
    a += P[(int64_t)s * n + i * 4];
    b += P[(int64_t)s * n + i * 4 + 1];
  }
  c0[i] = a;
  c1[i] = b;
}

// Slices of a reduction over M rows: as many as fill the GPU with `tiles` output tiles each, not below 256 rows; a slice is a
// multiple of the step.  `alone` (one row group, nothing beside it): down to 64 rows until there is a block per CU.  A slice is
// a chain of loads, about 1.7 us per step of 16 rows, and slices add partial tiles to write and read: 10,000 rows, 64 x 32:
// 28 -> 10 us; beyond a block per CU the chain is hidden by other blocks and only the partial tiles would grow.
struct SliceRule {
  int tiles;
  bool alone = false;
  __host__ __device__ void cut(int64_t M, int64_t* rows, int64_t* slices) const {
    int64_t s = (1024 + tiles - 1) / tiles;
    int64_t most = (M + 255) / 256;
    if (alone) {
      const int64_t per_cu = (256 + tiles - 1) / tiles, finest = (M + 63) / 64;
      const int64_t fine = finest < per_cu ? finest : per_cu;
      if (fine > most) most = fine;
    }
    if (s > most) s = most;
    if (s < 1) s = 1;
    int64_t r = (M + s - 1) / s;
    r = (r + BK - 1) / BK * BK;
    *rows = r;
    *slices = (M + r - 1) / r;
  }
};

// tab[2 z], tab[2 z + 1]: rows of slice z; a block per row group, its slices behind those of the groups before it
__global__ void __launch_bounds__(256) k_slice_table(const int64_t* __restrict__ groups, SliceRule rule, int64_t* __restrict__ tab) {
  __shared__ int64_t before;
  const int g = blockIdx.x;
  if (threadIdx.x == 0) before = 0;
  __syncthreads();
  int64_t mine = 0, rows, n;
  for (int q = threadIdx.x; q < g; q += 256) {
    rule.cut(groups[2 * q + 1] - groups[2 * q], &rows, &n);
    mine += n;
  }
  if (mine) atomicAdd((unsigned long long*)&before, (unsigned long long)mine);
  __syncthreads();
  const int64_t r0 = groups[2 * g], r1 = groups[2 * g + 1];
  rule.cut(r1 - r0, &rows, &n);
  for (int64_t z = threadIdx.x; z < n; z += 256) {
    tab[2 * (before + z)] = r0 + z * rows;
    tab[2 * (before + z) + 1] = r0 + (z + 1) * rows < r1 ? r0 + (z + 1) * rows : r1;
  }
}

inline int round_up(int x, int m) { return (x + m - 1) / m * m; }

template <int FORM>
int launch_nn(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* Bp, int Np, float* C, int64_t ldc, int64_t M, int K, int N,
              int relu) {
  const unsigned gx = (unsigned)((M + BM - 1) / BM);
  if (N > 64) k_gemm_nn<128, 2, 2, 2, 2, FORM><<<dim3(gx, (unsigned)((N + 127) / 128)), 256, 0, st>>>(A, lda, Bp, Np, C, ldc, M, K, N, relu);
  else k_gemm_nn<64, 4, 1, 1, 2, FORM><<<dim3(gx, 1), 256, 0, st>>>(A, lda, Bp, Np, C, ldc, M, K, N, relu);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}

// Products whose columns, in tiles of 32, are at most four fifths of what k_gemm_nn's blocks of 64 or 128 would compute go through k_rows_w.  us, k_gemm_nn (with
// its packed W) | k_rows_w, at rows x K x N: 10 k x 64 x 32 5.8 | 4.7, 60 k x 67 x 129 40.4 | 23.4, 60 k x 129 x 67 34.3 | 25.0, 116 k x 301 x 129 165 | 135, 233 k x 256 x
// 20 79 | 49, 300 k x 129 x 67 113 | 97, 1 M x 64 x 20 85 | 68.  Beyond the line: 300 k x 64 x 300 187 | 195, 233 k x 256 x 41 85 | 89, 1 M x 64 x 64 112 | 120, 2.45 M x 100 x 256
// 1,415 | 1,430 (the memory's rate or, in long runs, the power that fp32 matrix cores draw).
// Where W's columns do not fit the LDS together the rows are read once for every tile or two.  That pays while it spares enough products: 5 of 8 tiles, 300 k x 602 x 160 744 | 621, 2.45 M x
// 1216 x 132 12,599 | 9,397; 6 of 8, 1 M x 800 x 192 3,234 | 3,016; 9 of 12, 1 M x 602 x 288 3,894 | 3,567.  Not with 3 of 4 tiles over many rows: 424 x 70 and 602 x 96, 60 k rows
// 81 | 66 and 103 | 86, 300 k 308 | 293 and 411 | 398, 600 k 540 | 571 and 749 | 779, 2.45 M 2,115 | 2,308 and 2,956 | 3,120.
// An element is summed up in the same order by both, so that a row does not depend on how many are multiplied at once.
constexpr int64_t ROWS_THRICE = 400000;   // rows up to which they are read three times for the sake of a quarter of the products
struct RowsShape {
  int tj = 0, waves = 0;     // tj 0: k_gemm_nn's
  unsigned gx = 0, gy = 0;
};
RowsShape rows_shape(int64_t M, int K, int N) {
  RowsShape s;
  const int tiles = (N + 31) / 32, blocks = N > 64 ? (N + 127) / 128 * 4 : 2;
  int best = blocks * 4 / 5;
  for (int tj = 1; tj <= 5 && rows_lds(K, tj) <= ROWS_LDS; ++tj) {
    const int n = (tiles + tj - 1) / tj * tj;
    if (n <= best) best = n, s.tj = tj;
  }
  if (tiles == 3 && s.tj == 1 && M > ROWS_THRICE) s.tj = 0;
  if (!s.tj) return s;
  const int64_t strips = (M + 31) / 32;
  while (s.tj > 1 && strips * ((tiles + s.tj - 1) / s.tj) < 1024) --s.tj;   // (a wave for every SIMD)
  s.gy = (unsigned)((tiles + s.tj - 1) / s.tj);
  // eight waves a CU in two blocks, or in one where W takes most of the LDS: more waves do not help (their strips come round by round), fewer wait for their loads
  const int per_cu = 2 * rows_lds(K, s.tj) <= ROWS_LDS ? 2 : 1;
  s.waves = strips * s.gy < 1024 ? 2 : 8 / per_cu;
  s.gx = (unsigned)std::min<int64_t>((strips + s.waves - 1) / s.waves, std::max(1u, 256u * per_cu * (8 / per_cu / s.waves) / s.gy));
  return s;
}
template <int TJ, int NBUF, bool T>
int launch_rows(ht_ctx* ctx, hipStream_t st, const RowsShape& s, const float* A, int64_t lda, const float* W, float* C, int64_t ldc, int64_t M, int K,
                int N, int relu) {
  const int lds = rows_lds(K, TJ);
  // The limit belongs to the kernel on its device, for all contexts and threads: raised to all of the LDS, once, and never lowered (by the bytes of each call it could fall
  // between another thread's raising it and its launch).
  static std::atomic<uint64_t> raised{0};   // a bit for each device
  const uint64_t bit = ctx->device < 64 ? 1ull << ctx->device : 0;
  if (lds > (64 << 10) && !(raised.load(std::memory_order_relaxed) & bit)) {
    HT_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_rows_w<TJ, NBUF, T>), hipFuncAttributeMaxDynamicSharedMemorySize, ROWS_LDS));
    raised.fetch_or(bit, std::memory_order_relaxed);
  }
  k_rows_w<TJ, NBUF, T><<<dim3(s.gx, s.gy), s.waves * 64, lds, st>>>(A, lda, W, C, ldc, M, K, N, relu);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}
template <bool T>
int rows_w(ht_ctx* ctx, hipStream_t st, const RowsShape& s, const float* A, int64_t lda, const float* W, float* C, int64_t ldc, int64_t M, int K, int N,
           int relu) {
  switch (s.tj) {
    case 1: return launch_rows<1, 4, T>(ctx, st, s, A, lda, W, C, ldc, M, K, N, relu);
    case 2: return launch_rows<2, 4, T>(ctx, st, s, A, lda, W, C, ldc, M, K, N, relu);
    case 3: return launch_rows<3, 2, T>(ctx, st, s, A, lda, W, C, ldc, M, K, N, relu);
    case 4: return launch_rows<4, 2, T>(ctx, st, s, A, lda, W, C, ldc, M, K, N, relu);
    default: return launch_rows<5, 2, T>(ctx, st, s, A, lda, W, C, ldc, M, K, N, relu);
  }
}

// C = A W (+ReLU), or A W^T: out of a padded copy of W in the context's scratch, or of W itself.
int gemm_nn(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* W, bool transposed, float* C, int64_t ldc, int64_t M, int32_t K,
            int32_t N, int relu) {
  if (lda & 3) return ht_set_err(ctx, HT_ESHAPE, "gemm: row pitch must be a multiple of 4");
  if (M <= 0 || N <= 0) return HT_OK;
  const RowsShape shape = rows_shape(M, K, N);
  if (shape.tj)
    return transposed ? rows_w<true>(ctx, st, shape, A, lda, W, C, ldc, M, K, N, relu) : rows_w<false>(ctx, st, shape, A, lda, W, C, ldc, M, K, N, relu);
  if (reads_w_in_place(M, K, N, transposed))
    return transposed ? launch_nn<TRANSPOSED>(ctx, st, A, lda, W, 0, C, ldc, M, K, N, relu)
                      : launch_nn<AS_IS>(ctx, st, A, lda, W, 0, C, ldc, M, K, N, relu);
  const int Kp = round_up(K, BK), Np = round_up(N, 128);
  float* Bp = nullptr;
  HT_TRY(ht_scratch(ctx, HT_S_PACKW, (size_t)Kp * Np * 4, (void**)&Bp));
  k_pack_b<<<(unsigned)(((int64_t)Kp * Np + 255) / 256), 256, 0, st>>>(W, transposed ? N : K, transposed ? K : N, transposed, Bp, Kp, Np);
  HT_LAUNCH_CHECK(ctx);
  return launch_nn<PACKED>(ctx, st, A, lda, Bp, Np, C, ldc, M, K, N, relu);
}

}  // namespace

// scratch slots: 0 = packed W, 1 = TN partial tiles
// Bp = the zero-padded, tile-aligned copy of W [K x N] that the NN kernels read ([round_up(K, 16) x round_up(N, 128)], in
// the context's scratch); *Np its row pitch.
int ht_pack_w(ht_ctx* ctx, hipStream_t st, const float* W, int32_t K, int32_t N, float** Bp, int* Np) {
  const int Kp = round_up(K, BK), Npp = round_up(N, 128);
  HT_TRY(ht_scratch(ctx, HT_S_PACKW, (size_t)Kp * Npp * 4, (void**)Bp));
  k_pack_b<<<(unsigned)(((int64_t)Kp * Npp + 255) / 256), 256, 0, st>>>(W, K, N, 0, *Bp, Kp, Npp);
  HT_LAUNCH_CHECK(ctx);
  *Np = Npp;
  return HT_OK;
}

int ht_gemm_nn(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, float* C, int64_t ldc,
               int64_t M, int32_t K, int32_t N, int relu) {
  return gemm_nn(ctx, st, A, lda, B, false, C, ldc, M, K, N, relu);
}

int ht_gemm_nt(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, float* C, int64_t ldc,
               int64_t M, int32_t N, int32_t K, int accumulate) {
  // C[M x K] = A[M x N] (B[K x N])^T : reduction over N, output width K
  return gemm_nn(ctx, st, A, lda, B, true, C, ldc, M, N, K, accumulate ? 2 : 0);
}

namespace {

int tn_tiles(int32_t K, int32_t N) { return ((K + BM - 1) / BM) * (N > 64 ? (N + 127) / 128 : 1); }

// Which grad W goes through k_split_tn: both sides of the tile filled, and enough rows, or enough work in all, that its deeper stages
// and longer prologue pay.  us in fp32 | split, at rows x K x N.  Beyond the line: 60 k x 129 x 67 69 | 50, 60 k x 256 x 128 57 | 56,
// 20 k x 256 x 256 51 | 49, 9 k x 602 x 256 66 | 55.  Before it: 20 k x 256 x 128 29 | 31, 9 k x 256 x 256 27 | 31,
// 4 k x 256 x 256 20 | 22, 1 k x 256 x 256 17 | 19.
bool use_split_tn(int64_t rows, int32_t K, int32_t N) {
  return K > 64 && N > 64 && (rows >= 32768 || (double)rows * K * N >= 1e9);
}

}  // namespace

// One block reads each value of B, so that writing it masked costs no read twice.  (Wider A: as much memory traffic as k_relu_mask and a product that reads what it wrote.)
// A layer of 1 M vertices, 64 x 64, forward and backward 3.04 -> 2.96 ms; of 20 k, 64 x 32 111 us either way.
bool ht_gemm_tn_writes(int64_t rows, int32_t K, int32_t N) { return K <= BM && !use_split_tn(rows, K, N); }

namespace {

size_t pad256(size_t b) { return (b + 255) & ~(size_t)255; }

// rows: destination rows behind all slices
int launch_tn(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t M, int32_t K,
              int32_t N, int64_t slice_rows, int64_t slices, const int64_t* tab, int64_t rows, int accumulate, TnLater* later, ReluMask mask) {
  const int64_t kn = (int64_t)K * N;
  float* P = nullptr;
  const size_t bytes = pad256((size_t)(slices * kn) * 4);
  const bool leave = later && ctx->tn_defer && !accumulate && ctx->tn_used + bytes <= ctx->scratch_bytes[HT_S_TNPART];
  if (leave) {
    P = (float*)((char*)ctx->scratch[HT_S_TNPART] + ctx->tn_used);
  } else {
    HT_TRY(ht_flush_products(ctx, st));     // (the partial tiles of this one go where theirs are)
    HT_TRY(ht_scratch(ctx, HT_S_TNPART, bytes, (void**)&P));
  }
  dim3 grid((unsigned)((K + BM - 1) / BM), (unsigned)(N > 64 ? (N + 127) / 128 : 1), (unsigned)slices);
  auto launch = [&](auto masked) {
    constexpr bool MASKED = decltype(masked)::value;
    if (use_split_tn(rows, K, N))
      k_split_tn<MASKED><<<grid, 256, 0, st>>>(A, lda, B, ldb, mask, P, M, K, N, slice_rows, tab);
    else if (N > 64)
      k_gemm_tn<128, 2, 2, 2, 2, 1, MASKED><<<grid, 256, 0, st>>>(A, lda, B, ldb, mask, P, M, K, N, slice_rows, tab);
    else
      k_gemm_tn<64, 4, 1, 1, 2, 2, MASKED><<<grid, 256, 0, st>>>(A, lda, B, ldb, mask, P, M, K, N, slice_rows, tab);
  };
  mask.ref ? launch(std::true_type{}) : launch(std::false_type{});
  HT_LAUNCH_CHECK(ctx);
  if (leave) {
    ctx->tn_used += bytes;
    ctx->tn_pending.push_back(PendingTn{P, kn, (int)slices, C, {later->column[0], later->column[1]}});
    later->left = true;
    return HT_OK;
  }
  launch_reduce(st, P, kn, (int)slices, accumulate, C);
  HT_LAUNCH_CHECK(ctx);
  return HT_OK;
}

}  // namespace

int ht_gemm_tn(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, int64_t ldb, float* C,
               int64_t M, int32_t K, int32_t N, int accumulate, TnLater* later, ReluMask mask) {
  if ((lda & 3) || (ldb & 3) || (mask.ld & 3)) return ht_set_err(ctx, HT_ESHAPE, "gemm: row pitch must be a multiple of 4");
  if (K <= 0 || N <= 0) return HT_OK;
  if (M <= 0) {
    if (!accumulate) HT_TRY(ht_fill_zero(ctx, st, C, (size_t)K * N * 4));
    return HT_OK;
  }
  int64_t rows, slices;
  SliceRule{tn_tiles(K, N), true}.cut(M, &rows, &slices);
  return launch_tn(ctx, st, A, lda, B, ldb, C, M, K, N, rows, slices, nullptr, M, accumulate, later, mask);
}

size_t ht_gemm_tn_bytes(int64_t M, int32_t K, int32_t N) {
  int64_t rows, slices;
  SliceRule{tn_tiles(K, N), true}.cut(std::max<int64_t>(M, 1), &rows, &slices);
  return (size_t)(slices * K * N) * 4;
}

namespace {

// [g0, g1) and its slices: the row groups that one launch of ht_gemm_tn_groups takes
size_t next_groups(const SliceRule& rule, int32_t K, int32_t N, const std::vector<int64_t>& groups, size_t g0, int64_t* slices) {
  const int64_t most = std::max<int64_t>(1024, std::min<int64_t>(32768, ((int64_t)1 << 30) / ((int64_t)K * N * 4)));   // slices per launch
  size_t g1 = g0;
  *slices = 0;
  for (; g1 < groups.size() / 2; ++g1) {
    int64_t rows, n;
    rule.cut(groups[2 * g1 + 1] - groups[2 * g1], &rows, &n);
    if (g1 > g0 && *slices + n > most) break;
    *slices += n;
  }
  return g1;
}

}  // namespace

void ht_gemm_groups_wants(int32_t K, int32_t N, const std::vector<int64_t>& groups, std::vector<ScratchWant>* want) {
  const size_t G = groups.size() / 2;
  if (G <= 1) {
    want->push_back({HT_S_TNPART, ht_gemm_tn_bytes(G ? groups[1] - groups[0] : 0, K, N)});
    return;
  }
  const SliceRule rule{tn_tiles(K, N)};
  for (size_t g0 = 0; g0 < G;) {
    int64_t slices;
    g0 = next_groups(rule, K, N, groups, g0, &slices);
    want->push_back({HT_S_TNPART, (size_t)(slices * K * N) * 4});
    want->push_back({HT_S_TNTAB, (size_t)slices * 16});
  }
}

size_t ht_gemm_groups_bytes(int32_t K, int32_t N, const std::vector<int64_t>& groups) {
  std::vector<ScratchWant> want;
  ht_gemm_groups_wants(K, N, groups, &want);
  size_t bytes = 0;
  for (const ScratchWant& w : want) bytes += w.slot == HT_S_TNPART ? pad256(w.bytes) : 0;
  return bytes;
}

int ht_defer_products(ht_ctx* ctx, const std::vector<size_t>& bytes) {
  ctx->tn_pending.clear();
  ctx->tn_used = 0;
  ctx->tn_defer = false;
  size_t all = 0;
  for (size_t b : bytes) all += pad256(b);
  if (all > HT_DEFER_BYTES || !ht_may_spend(ctx)) return HT_OK;
  const int rc = ht_scratch_all(ctx, {{HT_S_TNPART, all}});
  ctx->tn_defer = rc == HT_OK;
  return rc == HT_ENOMEM ? (int)HT_OK : rc;
}

int ht_flush_products(ht_ctx* ctx, hipStream_t st, bool drop) {
  for (const PendingTn& p : ctx->tn_pending) {
    if (drop) break;
    if (p.column[0]) {
      k_reduce_columns<<<(unsigned)((p.n / 4 + 255) / 256), 256, 0, st>>>(p.P, p.n, p.slices, p.column[0], p.column[1]);
    } else {
      launch_reduce(st, p.P, p.n, p.slices, 0, p.C);
    }
    HT_LAUNCH_CHECK(ctx);
  }
  ctx->tn_pending.clear();
  ctx->tn_used = 0;
  if (drop) ctx->tn_defer = false;
  return HT_OK;
}

// The row groups' sums one after the other, as ht_gemm_tn called once per group would add them, in as few launches as the
// partial tiles' memory allows.
int ht_gemm_tn_groups(ht_ctx* ctx, hipStream_t st, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int32_t K,
                      int32_t N, const std::vector<int64_t>& groups, const int64_t* d_groups, TnLater* later, ReluMask mask) {
  const size_t G = groups.size() / 2;
  if (G <= 1) {
    const int64_t r0 = G ? groups[0] : 0;
    return ht_gemm_tn(ctx, st, A + r0 * lda, lda, B + r0 * ldb, ldb, C, G ? groups[1] - r0 : 0, K, N, 0, later,
                      ReluMask{mask.ref ? mask.ref + r0 * mask.ld : nullptr, mask.ld, mask.to ? mask.to + r0 * mask.to_ld : nullptr, mask.to_ld});
  }
  if ((lda & 3) || (ldb & 3) || (mask.ld & 3)) return ht_set_err(ctx, HT_ESHAPE, "gemm: row pitch must be a multiple of 4");
  if (K <= 0 || N <= 0) return HT_OK;
  const SliceRule rule{tn_tiles(K, N)};
  int64_t all = 0;
  for (size_t k = 0; k < G; ++k) all += groups[2 * k + 1] - groups[2 * k];
  for (size_t g0 = 0; g0 < G;) {
    int64_t total;
    const size_t g1 = next_groups(rule, K, N, groups, g0, &total);
    int64_t* tab = nullptr;
    HT_TRY(ht_scratch(ctx, HT_S_TNTAB, (size_t)total * 16, (void**)&tab));
    k_slice_table<<<(unsigned)(g1 - g0), 256, 0, st>>>(d_groups + 2 * g0, rule, tab);
    HT_LAUNCH_CHECK(ctx);
    HT_TRY(launch_tn(ctx, st, A, lda, B, ldb, C, 0, K, N, 0, total, tab, all, g0 > 0, g1 == G ? later : nullptr, mask));
    g0 = g1;
  }
  return HT_OK;
}
