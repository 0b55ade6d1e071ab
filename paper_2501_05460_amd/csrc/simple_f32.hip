// fp32 mode of the encode stage: bounds-checked kernels with fp32 storage and
// fp32 accumulation (the products on the fp32 matrix instruction).  This mode
// exists for the small fp32 configuration, whose time is the latency chain of
// its 23 short launches, and as the on-device numerical reference of the bf16
// MFMA path.
#include <cmath>
#include <type_traits>

#include "kernels.h"

namespace epd {

// ---------------------------------------------------------------- im2col ----
// A[t*N + y*g + x][(c*p + dy)*p + dx] = tiles[t][c][p*y + dy][p*x + dx]
__global__ void k_f32_im2col(const float* __restrict__ tiles, float* __restrict__ A, int S, int p,
                             int g, int Kp, long total) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  int e = (int)(i % Kp);
  long row = i / Kp;
  int N = g * g;
  long t = row / N;
  int n = (int)(row % N);
  int y = n / g, x = n % g;
  int c = e / (p * p), r = e % (p * p);
  int dy = r / p, dx = r % p;
  A[i] = tiles[((t * 3 + c) * S + (p * y + dy)) * (long)S + (p * x + dx)];
}

void f32_im2col(const float* tiles, float* A, int T, int S, int p, hipStream_t st) {
  int g = S / p, Kp = 3 * p * p;
  long total = (long)T * g * g * Kp;
  if (total == 0) return;
  int bs = 256;
  k_f32_im2col<<<dim3((unsigned)((total + bs - 1) / bs)), dim3(bs), 0, st>>>(tiles, A, S, p, g, Kp, total);
}

// ------------------------------------------------------------------ GEMM ----
// C[M,N] = A[M,K] * W[N,K]^T on v_mfma_f32_16x16x4_f32.  One workgroup per 16 R x 16 R tile; its four waves split K
// (whole 16-element chunks, a share of ceil(chunks / 4) each) and their partial tiles are added in LDS.
// The launches of the small configuration are bound by one wave's chain of loads and multiply-adds, so the
// contraction is cut in four and the tile is 16 x 16 while larger ones would leave CUs idle (M = 256, N = 192,
// K = 768, one slice of the tiny configuration: 192 workgroups with chains of 48 instructions; 36 us with one thread's
// chain of 768 multiply-adds through LDS tiles, 8 us now).  Large launches are bound by the operand bytes a tile asks its
// CU's cache for, 64 x 64 tiles for half as many per product as 32 x 32 ones (M = 16384, N = 4096, K = 1024, in us: 3600 |
// 2040 | 1520 on 16 | 32 | 64-wide tiles, 2640 through LDS tiles of 64 x 64 on the vector unit).  Operands come straight from global memory: lane l holds
// row l % 16, elements 4 (l / 16) .. + 3 of a chunk (one 16-byte load), and instruction e of a chunk multiplies
// element e of all four groups, the same four elements of both operands.  An element's sum is ordered by K alone, so its
// bits do not depend on the tile or the batch.
constexpr int F32_GROUP = 6;   // most chunks loaded ahead as one batch
// NORM: the rows of A are normalised on the way in (LayerNorm / RMSNorm over their K elements).  A share of the
// contraction then has to fit one batch of loads (K <= 64 F32_GROUP): a wave holds its part of the rows, the statistics
// meet in LDS, twice (mean, then squared deviations), and the normalised row never goes to memory: the launch of its own
// (5 us of which the work is less than one) is gone.  Bits depend on K alone here too (multiply-adds are written out: all
// tile sizes have to contract alike).
template <int N, typename F>
__device__ __forceinline__ void for_const(F f) {
  if constexpr (N > 0) { for_const<N - 1>(f); f(std::integral_constant<int, N - 1>{}); }
}
struct F32Norm { const float* gamma; const float* beta; int rms; float eps; };
template <int EPI, int R, bool VEC, bool NORM = false>
__global__ __launch_bounds__(256, R == 4 ? 2 : 1) void k_f32_gemm(const F32Norm norm, const float* __restrict__ A, int lda,
                                                  const float* __restrict__ W,
                                                  const float* __restrict__ bias, float* C, int ldc,
                                                  const float* __restrict__ pos, int n_pos, int M,
                                                  int N, int K, const int* __restrict__ row_map,
                                                  int block_tokens, SliceRows xrows) {
  constexpr int T = 16 * R;
  constexpr int G = R == 4 ? 1 : R == 2 ? 2 : F32_GROUP;   // chunks loaded ahead as one batch: enough products to cover the next one's loads, and two workgroups' registers
  constexpr int IB = R == 4 ? 1 : R;          // 16-row blocks of the tile whose partial sums meet in LDS at a time
  __shared__ float part[4][16 * IB * T];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, q = lane >> 4;
  const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
  const int chunks = (K + 15) / 16, share = (chunks + 3) / 4;
  const int c_begin = __builtin_amdgcn_readfirstlane(wave * share), c_end = min(chunks, c_begin + share);
  auto load = [&](const float* base, long ld, int row, int rows, int c) -> f32x4 {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    const int k = c * 16 + 4 * q;
    if (c < c_end && row < rows) {
      const float* p = base + (long)row * ld + k;
      if (VEC) {
        if (k < K) v = *reinterpret_cast<const f32x4*>(p);   // K % 4 == 0
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (k + e < K) v[e] = p[e];
      }
    }
    return v;
  };
  f32x4 acc[R][R];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // NORM holds the whole share of its rows, set 0 only
  f32x4 a[NORM ? 1 : 2][NORM ? F32_GROUP : G][R], w[2][G][R];
  auto fetch_a = [&](auto set, int c0, int n) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int g = 0; g < (NORM ? F32_GROUP : G); ++g)
#pragma unroll
      for (int i = 0; i < R; ++i)
        if (g < n) a[S][g][i] = load(A, lda, m0 + 16 * i + r16, M, c0 + g);
  };
  auto fetch_w = [&](auto set, int c0) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int i = 0; i < R; ++i) w[S][g][i] = load(W, K, n0 + 16 * i + r16, N, c0 + g);
  };
  // chunks g0 .. g0 + G - 1 of operand set A against weight set S, the first n of them: the others lie past the share and are zeros (K = 192
  // fills half a batch; M = 256, us, all | n of them: N = 768 with a norm 6.3 | 5.7, N = 192 3.5 | 3.3; M = 1024 12.5 | 11.0, 5.2 | 4.7)
  auto multiply = [&](auto set_a, auto set_w, int g0, int n) {
    constexpr int SA = decltype(set_a)::value, S = decltype(set_w)::value;
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (G == 1 || g < n) {   // uniform
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < R; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[SA][g0 + g][i][e], w[S][g][j][e], acc[i][j], 0, 0, 0);
      }
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  fetch_a(S0{}, c_begin, F32_GROUP);
  fetch_w(S0{}, c_begin);
  if constexpr (NORM) {
    __shared__ float red[2][4][T];
    float mean[R], rstd[R];
    // sum over a row: this lane's elements, the lanes of the row in this wave, the four waves
    auto row_sum = [&](int pass, float (&x)[R]) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        auto add = [](float a, float b) { return a + b; };
        x[i] = with_lane_32(with_lane_16(x[i], add), add);
        if (q == 0) red[pass][wave][16 * i + r16] = x[i];
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int r = 16 * i + r16;
        x[i] = (red[pass][0][r] + red[pass][1][r]) + (red[pass][2][r] + red[pass][3][r]);
      }
    };
    auto in_row = [&](int g) { return c_begin + g < c_end && (c_begin + g) * 16 + 4 * q < K; };   // K % 4 == 0
    float s1[R], s2[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      s1[i] = s2[i] = 0.f;
#pragma unroll
      for (int g = 0; g < F32_GROUP; ++g) s1[i] += (a[0][g][i][0] + a[0][g][i][1]) + (a[0][g][i][2] + a[0][g][i][3]);
    }
    if (!norm.rms) row_sum(0, s1);   // uniform
#pragma unroll
    for (int i = 0; i < R; ++i) {
      mean[i] = norm.rms ? 0.f : s1[i] / K;
#pragma unroll
      for (int g = 0; g < F32_GROUP; ++g)
        if (in_row(g)) {
#pragma unroll
          for (int e = 0; e < 4; ++e) { const float d = a[0][g][i][e] - mean[i]; s2[i] = fmaf(d, d, s2[i]); }
        }
    }
    row_sum(1, s2);
#pragma unroll
    for (int i = 0; i < R; ++i) rstd[i] = 1.0f / sqrtf(s2[i] / K + norm.eps);
#pragma unroll
    for (int g = 0; g < F32_GROUP; ++g)
      if (in_row(g)) {
        const int k = (c_begin + g) * 16 + 4 * q;
        const f32x4 gm = *reinterpret_cast<const f32x4*>(norm.gamma + k);
        const f32x4 bt = norm.rms ? f32x4{0.f, 0.f, 0.f, 0.f} : *reinterpret_cast<const f32x4*>(norm.beta + k);
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) a[0][g][i][e] = fmaf((a[0][g][i][e] - mean[i]) * rstd[i], gm[e], bt[e]);
      }
  }
  if constexpr (NORM) {
    static_assert(F32_GROUP % G == 0, "whole batches");
    for_const<F32_GROUP / G>([&](auto b_) {
      constexpr int b = decltype(b_)::value;
      if constexpr ((b + 1) * G < F32_GROUP) fetch_w(std::integral_constant<int, 1 - b % 2>{}, c_begin + (b + 1) * G);
      multiply(S0{}, std::integral_constant<int, b % 2>{}, b * G, c_end - c_begin - b * G);
    });
  } else {
    for (int c = c_begin; c < c_end; c += 2 * G) {
      fetch_a(S1{}, c + G, G);
      fetch_w(S1{}, c + G);
      multiply(S0{}, S0{}, 0, c_end - c);
      if (c + G >= c_end) break;
      fetch_a(S0{}, c + 2 * G, G);
      fetch_w(S0{}, c + 2 * G);
      multiply(S1{}, S1{}, 0, c_end - c - G);
    }
  }
  // result register e of lane l: row 4 (l / 16) + e, column l % 16
#pragma unroll
  for (int ib = 0; ib < R; ib += IB) {
    if (ib > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[wave][(16 * i + 4 * q + e) * T + 16 * j + r16] = acc[ib + i][j][e];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < IB * R; ++u) {
      const int idx = tid + 256 * u;
      const int r = m0 + 16 * ib + idx / T, c = n0 + idx % T;
      if (r >= M || c >= N) continue;
      const float v = ((part[0][idx] + part[1][idx]) + (part[2][idx] + part[3][idx])) + (bias ? bias[c] : 0.f);
      // paged output: row r of the product lives in block row_map[r / block_tokens]
      const long orow = row_map ? (long)row_map[r / block_tokens] * block_tokens + r % block_tokens : r;
      const long o = orow * ldc + c;
      if (EPI == EPI_BIAS_RESIDUAL) {
        C[o] += v;
      } else if (EPI == EPI_BIAS_POS) {
        C[xrows.row(r) * ldc + c] = v + pos[(long)(r % n_pos) * N + c];   // patch embedding: through the slice layout
      } else {
        C[o] = apply_act<EPI>(v);
      }
    }
  }
}

static int f32_cu_count() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, v = 0;
    n = (hipGetDevice(&dev) == hipSuccess &&
         hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) ? v : 256;
  }
  return n;
}

// The tile's side in units of 16: the smallest of the times estimated for M rows, N columns and K, in us (fitted to 132
// launches of M 256 to 16384, K 192 to 4304: the tile taken is 0.7 % behind the fastest on average).  16 x 16 and 32 x 32
// tiles come in such numbers that the time grows with their count, 64 x 64 tiles in rounds.
static int f32_tile(int M, int N, int K, bool norm) {
  const double cus = f32_cu_count(), k = K;
  const double t32 = (double)((N + 31) / 32) * ((M + 31) / 32) / cus, rounds = ceil((double)((N + 63) / 64) * ((M + 63) / 64) / cus);
  const double us[3] = {norm ? 4.0 + 0.0078 * k + t32 * (2.0 + 0.0155 * k) : 4.5 + 0.0025 * k + t32 * (1.0 + 0.0145 * k),
                        norm ? 4.5 + 0.0130 * k + fmax(0.75, t32) * (3.1 + 0.0026 * k) : 6.0 + 0.0030 * k + fmax(0.75, t32) * (0.5 + 0.0088 * k),
                        norm ? 8.0 + 0.0100 * k + rounds * (9.0 + 0.0100 * k) : 6.0 + rounds * (4.0 + 0.0215 * k)};
  return us[0] <= us[1] && us[0] <= us[2] ? 1 : us[1] <= us[2] ? 2 : 4;
}

template <int R, bool VEC>
static void f32_gemm_r(int epi, const float* A, int lda, const float* W, const float* bias, float* C, int ldc,
                       const float* pos, int n_pos, int M, int N, int K, hipStream_t st, const int* row_map,
                       int block_tokens, SliceRows xrows) {
  dim3 grid((N + 16 * R - 1) / (16 * R), (M + 16 * R - 1) / (16 * R)), block(256);
  switch (epi) {
    case EPI_BIAS: k_f32_gemm<EPI_BIAS, R, VEC><<<grid, block, 0, st>>>(F32Norm{}, A, lda, W, bias, C, ldc, pos, n_pos, M, N, K, row_map, block_tokens, xrows); break;
    case EPI_BIAS_GELU_ERF: k_f32_gemm<EPI_BIAS_GELU_ERF, R, VEC><<<grid, block, 0, st>>>(F32Norm{}, A, lda, W, bias, C, ldc, pos, n_pos, M, N, K, row_map, block_tokens, xrows); break;
    case EPI_BIAS_GELU_TANH: k_f32_gemm<EPI_BIAS_GELU_TANH, R, VEC><<<grid, block, 0, st>>>(F32Norm{}, A, lda, W, bias, C, ldc, pos, n_pos, M, N, K, row_map, block_tokens, xrows); break;
    case EPI_BIAS_RESIDUAL: k_f32_gemm<EPI_BIAS_RESIDUAL, R, VEC><<<grid, block, 0, st>>>(F32Norm{}, A, lda, W, bias, C, ldc, pos, n_pos, M, N, K, row_map, block_tokens, xrows); break;
    default: k_f32_gemm<EPI_BIAS_POS, R, VEC><<<grid, block, 0, st>>>(F32Norm{}, A, lda, W, bias, C, ldc, pos, n_pos, M, N, K, row_map, block_tokens, xrows); break;
  }
}

void f32_gemm(int epi, const float* A, int lda, const float* W, const float* bias, float* C, int ldc,
              const float* pos, int n_pos, int M, int N, int K, hipStream_t st, const int* row_map,
              int block_tokens, SliceRows xrows) {
  if (M == 0 || N == 0) return;
  const bool vec = K % 4 == 0 && lda % 4 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15) == 0;
  const int r = f32_tile(M, N, K, false);
#define F32_GEMM(VEC)                                                                                                   \
  if (r == 1) f32_gemm_r<1, VEC>(epi, A, lda, W, bias, C, ldc, pos, n_pos, M, N, K, st, row_map, block_tokens, xrows);       \
  else if (r == 2) f32_gemm_r<2, VEC>(epi, A, lda, W, bias, C, ldc, pos, n_pos, M, N, K, st, row_map, block_tokens, xrows);  \
  else f32_gemm_r<4, VEC>(epi, A, lda, W, bias, C, ldc, pos, n_pos, M, N, K, st, row_map, block_tokens, xrows);
  if (vec) { F32_GEMM(true) } else { F32_GEMM(false) }
#undef F32_GEMM
}

bool f32_norm_gemm_fits(int lda, int K, const float* A, const float* W, const float* gamma, const float* beta) {
  return K <= 4 * F32_GROUP * 16 && K % 4 == 0 && lda % 4 == 0 &&
         (((uintptr_t)A | (uintptr_t)W | (uintptr_t)gamma | (uintptr_t)beta) & 15) == 0;
}

void f32_norm_gemm(int epi, int kind, const float* gamma, const float* beta, float eps, const float* A, int lda, const float* W,
                   const float* bias, float* C, int ldc, int M, int N, int K, hipStream_t st) {
  if (M == 0 || N == 0) return;
  const F32Norm nm{gamma, beta, kind == 1 ? 1 : 0, eps};
  const int r = f32_tile(M, N, K, true), t = 16 * r;
  const dim3 grid((N + t - 1) / t, (M + t - 1) / t), block(256);
  const SliceRows xr{0, 0, 0};
#define F32_NORM_GEMM(EPI)                                                                                              \
  if (r == 1) k_f32_gemm<EPI, 1, true, true><<<grid, block, 0, st>>>(nm, A, lda, W, bias, C, ldc, nullptr, 1, M, N, K, nullptr, 1, xr);      \
  else if (r == 2) k_f32_gemm<EPI, 2, true, true><<<grid, block, 0, st>>>(nm, A, lda, W, bias, C, ldc, nullptr, 1, M, N, K, nullptr, 1, xr); \
  else k_f32_gemm<EPI, 4, true, true><<<grid, block, 0, st>>>(nm, A, lda, W, bias, C, ldc, nullptr, 1, M, N, K, nullptr, 1, xr);
  switch (epi) {
    case EPI_BIAS_GELU_ERF: F32_NORM_GEMM(EPI_BIAS_GELU_ERF) break;
    case EPI_BIAS_GELU_TANH: F32_NORM_GEMM(EPI_BIAS_GELU_TANH) break;
    default: F32_NORM_GEMM(EPI_BIAS) break;
  }
#undef F32_NORM_GEMM
}

// ------------------------------------------------------------------ norm ----
// Logical row R of `dim` elements lives at in + (R / groups) * ld_in + (R % groups) * dim
// (groups > 1: per-head norm inside a wider row).  One wave per row.
__global__ __launch_bounds__(256) void k_f32_norm(int kind, const float* in, long ld_in, float* out,
                                                  long ld_out, const float* __restrict__ gamma,
                                                  const float* __restrict__ beta, long rows, int dim,
                                                  int groups, float eps) {
  long R = (long)blockIdx.x * 4 + threadIdx.x / 64;
  if (R >= rows) return;
  int lane = threadIdx.x % 64;
  const float* x = in + (R / groups) * ld_in + (R % groups) * (long)dim;
  float* y = out + (R / groups) * ld_out + (R % groups) * (long)dim;
  float s = 0.f;
  float mean = 0.f;
  if (kind == 0) {
    for (int i = lane; i < dim; i += 64) s += x[i];
    mean = wave_sum(s) / dim;
  }
  float q = 0.f;
  for (int i = lane; i < dim; i += 64) {
    float d = x[i] - mean;
    q += d * d;
  }
  float rstd = 1.0f / sqrtf(wave_sum(q) / dim + eps);
  for (int i = lane; i < dim; i += 64) {
    float v = (x[i] - mean) * rstd * gamma[i];
    if (kind == 0) v += beta[i];
    y[i] = v;
  }
}

void f32_norm(int kind, const float* in, long ld_in, float* out, long ld_out, const float* gamma,
              const float* beta, long rows, int dim, int groups, float eps, hipStream_t st) {
  if (rows == 0) return;
  k_f32_norm<<<dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st>>>(kind, in, ld_in, out, ld_out, gamma,
                                                                    beta, rows, dim, groups, eps);
}

// ------------------------------------------------------------- attention ----
// One block per (query, head, slice): logits of the slice's N keys in LDS,
// block-wide max and sum, then one thread per output channel.
__global__ __launch_bounds__(128) void k_f32_attention(const float* __restrict__ q, long ld_q, int q_shared,
                                                       const float* __restrict__ k,
                                                       const float* __restrict__ v, long ld,
                                                       float* __restrict__ o, long ldo, int N, int hd,
                                                       float scale) {
  extern __shared__ float sm[];
  float* sc = sm;          // [N]
  float* sq = sm + N;      // [hd]
  __shared__ float red[2];
  const int tid = threadIdx.x;
  const int qi = blockIdx.x, h = blockIdx.y, t = blockIdx.z;
  const long row0 = (long)t * N;
  const long qrow = q_shared ? qi : row0 + qi;
  const long orow = (long)t * gridDim.x + qi;
  for (int d = tid; d < hd; d += 128) sq[d] = q[qrow * ld_q + h * hd + d];
  __syncthreads();
  float mx = -INFINITY;
  for (int j = tid; j < N; j += 128) {
    const float* kr = k + (row0 + j) * ld + h * hd;
    float acc = 0.f;
    for (int d = 0; d < hd; ++d) acc = fmaf(sq[d], kr[d], acc);
    acc *= scale;
    sc[j] = acc;
    mx = fmaxf(mx, acc);
  }
  mx = wave_max(mx);
  if (tid % 64 == 0) red[tid / 64] = mx;
  __syncthreads();
  mx = fmaxf(red[0], red[1]);
  __syncthreads();
  float sum = 0.f;
  for (int j = tid; j < N; j += 128) {
    float e = expf(sc[j] - mx);
    sc[j] = e;
    sum += e;
  }
  sum = wave_sum(sum);
  if (tid % 64 == 0) red[tid / 64] = sum;
  __syncthreads();
  float inv = 1.0f / (red[0] + red[1]);
  for (int d = tid; d < hd; d += 128) {
    float acc = 0.f;
    for (int j = 0; j < N; ++j) acc = fmaf(sc[j], v[(row0 + j) * ld + h * hd + d], acc);
    o[orow * ldo + h * hd + d] = acc * inv;
  }
}

// The same on v_mfma_f32_16x16x4_f32: one workgroup per 16 queries of one (slice, head).  The query-per-block kernel
// above reads every key and value once per query and its time is one thread's chain over head dim and keys; here 16
// queries share them and the four waves split the keys of the first product and, at head dim 64, of the second, else its head
// dim.  What bounds it is the chain of one workgroup: one slice of the tiny configuration (256 tokens, 3 heads of 64, 48 workgroups)
// 30 us with the kernel above, 11.1 with four-byte loads of the values and the softmax through LDS shuffles one logit at a time, 8.3 now
// (1024 tokens 34.0 -> 26.4; of 11.1 us the second product took 4.6, the softmax 2.6, the first product 2.5).  Values asked for
// ahead of the first product: 9.0.  The logits [16][keys] stay in LDS; keys past N count as weight zero and their rows are not read.
// hd % 16 == 0, rows 16-byte aligned.
// A lane's operand registers as in the GEMM: row l % 16, elements 4 (l / 16) .. + 3 of a 16-element chunk.
constexpr int F32_ATTN_MAX_KEYS = 2048;   // 16 rows of logits in LDS
constexpr int F32_ATTN_PART = 4 * 16 * 64;   // head dim 64: the waves' shares of the output
// HC: head dim / 16 when it is compiled in (the loads of a wave's keys and values are then issued as batches: 15.3 -> 11.8 us),
// 0: any, and head dim 64 where values or output rows are not 16-byte aligned.
template <int HC>
__global__ __launch_bounds__(256) void k_f32_attention_mfma(const float* __restrict__ q, long ld_q, int q_shared,
                                                            const float* __restrict__ k, const float* __restrict__ v,
                                                            long ld, float* __restrict__ o, long ldo, int n_q, int N, int hd,
                                                            float scale) {
  extern __shared__ float sm[];
  const int NP = (N + 15) / 16 * 16, LD = NP + 4;   // + 4: rows start 4 banks apart
  float* inv = sm + 16 * LD;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, g = lane >> 4;
  const int q0 = blockIdx.x * 16, h = blockIdx.y, t = blockIdx.z;
  const long row0 = (long)t * N;
  const int qi = min(q0 + r16, n_q - 1);   // rows past n_q repeat the last query, never stored
  const float* qp = q + ((q_shared ? 0 : row0) + qi) * ld_q + (long)h * hd + 4 * g;
  // logits: wave w takes key blocks w, w + 4, ..; result register e = query 4 g + e, key l % 16
  constexpr int HCR = HC > 0 ? HC : 1, KB = HC > 0 ? 4 : 1;   // key blocks of a wave loaded together
  f32x4 qr[HCR];
  if constexpr (HC > 0) {
#pragma unroll
    for (int d = 0; d < HC; ++d) qr[d] = *reinterpret_cast<const f32x4*>(qp + 16 * d);
  }
  for (int kb0 = wave * 16; kb0 < NP; kb0 += 64 * KB) {
    f32x4 acc[KB], kr[KB][HCR];
    if constexpr (HC > 0) {
#pragma unroll
      for (int b = 0; b < KB; ++b) {
        const int key = kb0 + 64 * b + r16;
        const float* kp = k + (row0 + (key < N ? key : 0)) * ld + (long)h * hd + 4 * g;
#pragma unroll
        for (int d = 0; d < HC; ++d) kr[b][d] = *reinterpret_cast<const f32x4*>(kp + 16 * d);
      }
    }
#pragma unroll
    for (int b = 0; b < KB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (HC > 0) {
#pragma unroll
      for (int d = 0; d < HC; ++d)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int b = 0; b < KB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(qr[d][e], kr[b][d][e], acc[b], 0, 0, 0);
    } else {
      const float* kp = k + (row0 + (kb0 + r16 < N ? kb0 + r16 : 0)) * ld + (long)h * hd + 4 * g;
#pragma unroll 4
      for (int d = 0; d < hd; d += 16) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(qp + d), b = *reinterpret_cast<const f32x4*>(kp + d);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc[0], 0, 0, 0);
      }
    }
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      const int key = kb0 + 64 * b + r16;
      if (key < NP) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sm[(4 * g + e) * LD + key] = key < N ? acc[b][e] * scale : -INFINITY;
      }
    }
  }
  // Output, head dim 64: wave w takes keys 64 u + 16 w .. + 15 of every group of 64 and all of the head dim: a lane loads 16 bytes of a
  // key's row and supplies them as column l % 16 of four blocks, feature 4 (l % 16) + c in block c.  (The chain of a 16-key block
  // over the groups is the one that the four chains of a wave per head-dim block below have: the same bits.)  The values of
  // the first 256 keys are on their way during the softmax.
  constexpr int VG = HC > 0 ? 4 : 0;
  f32x4 vpre[VG > 0 ? VG : 1][4];
  auto vrows = [&](int u, f32x4 (&b)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = 64 * u + 16 * wave + 4 * g + e;
      b[e] = j < N ? *reinterpret_cast<const f32x4*>(v + (row0 + j) * ld + (long)h * hd + 4 * r16) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  if constexpr (HC > 0) {
#pragma unroll
    for (int u = 0; u < VG; ++u) vrows(u, vpre[u]);
  }
  __syncthreads();
  // softmax: 16 threads per query, 16 logits of each at a time; exchanges inside a row of 16 lanes (turning by 8, 4, 2 and 1 adds what
  // the exchange with lane ^ 8, ^ 4, ^ 2 and ^ 1 does)
  {
    float* row = sm + (tid >> 4) * LD;
    const int j0 = tid & 15;
    float x[16], mx = -INFINITY;
    auto fetch = [&](int b) {
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = b + 16 * i < NP ? row[b + 16 * i + j0] : -INFINITY;   // NP % 16 == 0: uniform
    };
    for (int b = 0; b < NP; b += 256) {
      fetch(b);
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, x[i]);
    }
    mx = fmaxf(mx, row_turn<8>(mx));
    mx = fmaxf(mx, row_turn<4>(mx));
    mx = fmaxf(mx, row_turn<2>(mx));
    mx = fmaxf(mx, row_turn<1>(mx));
    float sum = 0.f;
    for (int b = 0; b < NP; b += 256) {
      if (NP > 256) fetch(b);
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (b + 16 * i < NP) {
          x[i] = expf(x[i] - mx);
          row[b + 16 * i + j0] = x[i];
          sum += x[i];
        }
    }
    sum += row_turn<8>(sum);
    sum += row_turn<4>(sum);
    sum += row_turn<2>(sum);
    sum += row_turn<1>(sum);
    if (j0 == 0) inv[tid >> 4] = 1.0f / sum;
  }
  __syncthreads();
  if constexpr (HC > 0) {
    static_assert(HC == 4, "four blocks of 16 columns, 16 bytes a lane");
    f32x4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto group = [&](int u, const f32x4 (&b)[4]) {
      const int j = 64 * u + 16 * wave + 4 * g;
      const f32x4 a = 64 * u + 16 * wave < NP ? *reinterpret_cast<const f32x4*>(sm + r16 * LD + j) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e][c], acc[c], 0, 0, 0);
    };
#pragma unroll
    for (int u = 0; u < VG; ++u) {
      if (64 * u < NP) group(u, vpre[u]);   // uniform
    }
    for (int u = VG; 64 * u < NP; ++u) {
      f32x4 b[4];
      vrows(u, b);
      group(u, b);
    }
    // register e of block c: query 4 (l / 16) + e, feature 4 (l % 16) + c.  The waves' shares meet in LDS.
    float* part = inv + 16;   // [4 waves][16 queries][64]
#pragma unroll
    for (int e = 0; e < 4; ++e) *reinterpret_cast<f32x4*>(part + (wave * 16 + 4 * g + e) * 64 + 4 * r16) = f32x4{acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
    __syncthreads();
    const int qr = tid >> 4, d = (tid & 15) * 4;
    const f32x4 p0 = *reinterpret_cast<const f32x4*>(part + qr * 64 + d), p1 = *reinterpret_cast<const f32x4*>(part + (16 + qr) * 64 + d),
                p2 = *reinterpret_cast<const f32x4*>(part + (32 + qr) * 64 + d), p3 = *reinterpret_cast<const f32x4*>(part + (48 + qr) * 64 + d);
    if (q0 + qr < n_q) {
      const float f = inv[qr];
      f32x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = ((p0[e] + p1[e]) + (p2[e] + p3[e])) * f;
      *reinterpret_cast<f32x4*>(o + ((long)t * n_q + q0 + qr) * ldo + (long)h * hd + d) = r;
    }
  } else {
    // wave w takes head-dim blocks w, w + 4, ..; lane l supplies keys 4 (l / 16) + e of column l % 16
    for (int d0 = wave * 16; d0 < hd; d0 += 64) {
      const float* vp = v + row0 * ld + (long)h * hd + d0 + r16;
      f32x4 acc[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int j0 = 0; j0 < NP; j0 += 64) {   // four chains, one per 16-key block of a group of 64 keys
        float b[4][4];
        f32x4 a[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int j1 = j0 + 16 * c + 4 * g;
#pragma unroll
          for (int e = 0; e < 4; ++e) b[c][e] = j1 + e < N ? vp[(long)(j1 + e) * ld] : 0.f;
          a[c] = j1 < NP ? *reinterpret_cast<const f32x4*>(sm + r16 * LD + j1) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][e], b[c][e], acc[c], 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = q0 + 4 * g + e;
        if (row < n_q) o[((long)t * n_q + row) * ldo + (long)h * hd + d0 + r16] = ((acc[0][e] + acc[1][e]) + (acc[2][e] + acc[3][e])) * inv[4 * g + e];
      }
    }
  }
}

// the rows of logits of more than 1020 keys take more than the 64 KiB a launch may ask for by default
hipError_t f32_attention_init() {
  constexpr int most = (int)((16 * (F32_ATTN_MAX_KEYS + 4) + 16 + F32_ATTN_PART) * sizeof(float));
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_f32_attention_mfma<4>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, most);
  return e != hipSuccess ? e : hipFuncSetAttribute(reinterpret_cast<const void*>(&k_f32_attention_mfma<0>),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, most);
}

void f32_attention(const float* q, long ld_q, int n_q, int q_shared, const float* k, const float* v, long ld,
                   float* o, long ldo, int T, int N, int H, int hd, float scale, hipStream_t st) {
  if (T == 0) return;
  const bool aligned = ld_q % 4 == 0 && ld % 4 == 0 && (((uintptr_t)q | (uintptr_t)k) & 15) == 0;
  if (hd % 16 == 0 && N <= F32_ATTN_MAX_KEYS && aligned) {
    const bool by_64 = hd == 64 && ldo % 4 == 0 && (((uintptr_t)v | (uintptr_t)o) & 15) == 0;
    const size_t smem = (size_t)(16 * ((N + 15) / 16 * 16 + 4) + 16 + (by_64 ? F32_ATTN_PART : 0)) * sizeof(float);
    const dim3 grid((n_q + 15) / 16, H, T);
    if (by_64) k_f32_attention_mfma<4><<<grid, dim3(256), smem, st>>>(q, ld_q, q_shared, k, v, ld, o, ldo, n_q, N, hd, scale);
    else k_f32_attention_mfma<0><<<grid, dim3(256), smem, st>>>(q, ld_q, q_shared, k, v, ld, o, ldo, n_q, N, hd, scale);
    return;
  }
  const size_t smem = (size_t)(N + hd) * sizeof(float);
  k_f32_attention<<<dim3(n_q, H, T), dim3(128), smem, st>>>(q, ld_q, q_shared, k, v, ld, o, ldo, N, hd, scale);
}

__global__ void k_f32_add_rows(const float* __restrict__ in, const float* __restrict__ add, int add_rows,
                               float* __restrict__ out, int dim, long total) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  out[i] = in[i] + add[((i / dim) % add_rows) * dim + i % dim];
}

void f32_add_rows(const float* in, const float* add, int add_rows, float* out, long rows, int dim, hipStream_t st) {
  long total = rows * dim;
  if (total == 0) return;
  k_f32_add_rows<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st>>>(in, add, add_rows, out, dim, total);
}

// --------------------------------------------------------- pixel shuffle ----
// out[t*N/4 + Y*(g/2) + X][(dy*2 + dx)*D + c] = in[row of patch t*N + (2Y+dy)*g + (2X+dx)][c]
__global__ void k_f32_shuffle(const float* __restrict__ in, SliceRows srows, float* __restrict__ out, int g, int D,
                              long total) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  int D4 = 4 * D;
  int e = (int)(i % D4);
  long m = i / D4;
  int h = g / 2;
  long t = m / (h * h);
  int mm = (int)(m % (h * h));
  int Y = mm / h, X = mm % h;
  int blk = e / D, c = e % D;
  int dy = blk / 2, dx = blk % 2;
  long src = srows.row(t * g * g + (long)(2 * Y + dy) * g + (2 * X + dx));
  out[i] = in[src * D + c];
}

void f32_shuffle(const float* in, SliceRows src, float* out, int T, int g, int D, hipStream_t st) {
  long total = (long)T * (g * g / 4) * 4 * D;
  if (total == 0) return;
  k_f32_shuffle<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st>>>(in, src, out, g, D, total);
}

__global__ void k_f32_take_rows(const float* __restrict__ in, SliceRows srows, float* __restrict__ out, int D, long total) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  out[i] = in[srows.row(i / D) * D + i % D];
}

void f32_take_rows(const float* in, SliceRows src, float* out, long rows, int D, hipStream_t st) {
  long total = rows * D;
  if (total == 0) return;
  k_f32_take_rows<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st>>>(in, src, out, D, total);
}

}  // namespace epd
