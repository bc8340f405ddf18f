// Kernels of the learned-guess network: a per-rank-index MLP n_in -> w -> w -> n_out with SiLU
// hidden activations, trained in FP32 (forward, backward, Adam) and run for inference in BF16 on
// MFMA with FP32 accumulation.
//
// Training pieces:
//   sgemm        C = op(A) op(B) on 64 x 64 tiles (FP32 VALU, LDS-staged), with fused epilogues:
//                bias + SiLU (keeps the pre-activation for the backward pass, or not in a pass
//                that is only a forward one), bias only, or a product with SiLU'(Z) (the backward
//                pass through an activation)
//   normalize    x_n = (x - mu) / sd per input column
//   mse_grad     dY = 2 (y_n - (t - mu) / sd) / (rows n_out) and per-block partial loss sums
//   colsum       bias gradients
//   adam         bias-corrected Adam update (Kingma and Ba, 2015)
//   init         Glorot-uniform weights from a counter-based generator (SplitMix64 of the index)
// A network of the guess network's class (width 256, at most 16 inputs and outputs) trains in three
// launches instead: train_rows (all of a row tile's forward and backward pass), train_w2 (the
// 256 x 256 weight gradient) and train_update (sums of the partials and the Adam step).
// Inference: one kernel evaluates all three layers of its rows with v_mfma_f32_16x16x16_bf16,
// keeping the activations in LDS.
// Parameter layout (FP32, one flat vector): W1 [n_in][w], b1 [w], W2 [w][w], b2 [w], W3 [w][n_out],
// b3 [n_out].
#include <mutex>

#include "internal.h"

namespace thc {
namespace {

constexpr int TPB = 256;

__device__ inline float silu_f(float z) { return z / (1.0f + __expf(-z)); }
__device__ inline float silu_grad_f(float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

constexpr int BM = 64, BN = 64, BK = 16;

// C[M][N] = op(A) op(B) (+ epilogue).  A is [M][K] (or [K][M] if TA), B is [K][N] (or [N][K] if TB).
template <bool TA, bool TB, int EPI>
__global__ __launch_bounds__(TPB) void sgemm_kernel(int64_t M, int64_t N, int64_t K, const float* __restrict__ A,
                                                    int64_t lda, const float* __restrict__ B, int64_t ldb,
                                                    float* __restrict__ C, int64_t ldc, const float* __restrict__ bias,
                                                    float* __restrict__ Z, int64_t ldz) {
  __shared__ float As[BK][BM + 1];
  __shared__ float Bs[BK][BN + 1];
  const int t = threadIdx.x;
  const int64_t m0 = (int64_t)blockIdx.y * BM, n0 = (int64_t)blockIdx.x * BN;
  const int tr = t / 16, tc = t % 16;  // thread owns rows tr + 16 i, cols tc + 16 j
  float acc[4][4] = {};
  for (int64_t k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
    for (int q = 0; q < (BM * BK) / TPB; ++q) {
      const int e = t + TPB * q;
      int mm, kk;
      if (TA) { mm = e % BM; kk = e / BM; } else { kk = e % BK; mm = e / BK; }
      const int64_t m = m0 + mm, k = k0 + kk;
      As[kk][mm] = (m < M && k < K) ? (TA ? A[k * lda + m] : A[m * lda + k]) : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < (BN * BK) / TPB; ++q) {
      const int e = t + TPB * q;
      int nn, kk;
      if (TB) { kk = e % BK; nn = e / BK; } else { nn = e % BN; kk = e / BN; }
      const int64_t n = n0 + nn, k = k0 + kk;
      Bs[kk][nn] = (n < N && k < K) ? (TB ? B[n * ldb + k] : B[k * ldb + n]) : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][tr + 16 * i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tc + 16 * j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t m = m0 + tr + 16 * i, n = n0 + tc + 16 * j;
      if (m >= M || n >= N) continue;
      float x = acc[i][j];
      if (EPI == 1) {  // bias + SiLU; the pre-activation goes to Z
        x += bias[n];
        Z[m * ldz + n] = x;
        x = silu_f(x);
      } else if (EPI == 4) {  // bias + SiLU, pre-activation not kept (forward pass only)
        x = silu_f(x + bias[n]);
      } else if (EPI == 2) {  // bias only
        x += bias[n];
      } else if (EPI == 3) {  // times SiLU'(Z)
        x *= silu_grad_f(Z[m * ldz + n]);
      }
      C[m * ldc + n] = x;
    }
}

__global__ void normalize_kernel(int64_t rows, int64_t cols, const float* __restrict__ X, const float* __restrict__ mu,
                                 const float* __restrict__ sd, float* __restrict__ Xn) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < rows * cols; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = e % cols;
    Xn[e] = (X[e] - mu[c]) / sd[c];
  }
}

__global__ void denorm_kernel(int64_t rows, int64_t cols, const float* __restrict__ Yn, const float* __restrict__ mu,
                              const float* __restrict__ sd, float* __restrict__ Y) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < rows * cols; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = e % cols;
    Y[e] = Yn[e] * sd[c] + mu[c];
  }
}

// dY = 2 (y_n - t_n) / (rows cols), t_n = (t - mu) / sd; part[block] = sum of (y_n - t_n)^2 over the block
__global__ void mse_grad_kernel(int64_t rows, int64_t cols, const float* __restrict__ Yn, const float* __restrict__ T,
                                const float* __restrict__ mu, const float* __restrict__ sd, float* __restrict__ dY,
                                double* __restrict__ part) {
  __shared__ double red[TPB];
  const int64_t n = rows * cols;
  const float scale = 2.0f / (float)n;
  double s = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = e % cols;
    const float d = Yn[e] - (T[e] - mu[c]) / sd[c];
    dY[e] = scale * d;
    s += (double)d * (double)d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = TPB / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void sum_parts_kernel(int64_t nparts, const double* __restrict__ part, double denom, float* __restrict__ out) {
  __shared__ double red[TPB];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < nparts; i += blockDim.x) s += part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = TPB / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (float)(red[0] / denom);
}

// out[n] = sum_r D[r][n]  (one workgroup per column)
__global__ void colsum_kernel(int64_t rows, int64_t cols, const float* __restrict__ D, float* __restrict__ out) {
  __shared__ float red[TPB];
  const int64_t n = blockIdx.x;
  float s = 0.0f;
  for (int64_t r = threadIdx.x; r < rows; r += blockDim.x) s += D[r * cols + n];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = TPB / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[n] = red[0];
}

// Per column of D[rows][cols]: mean and standard deviation (FP64 sums); a column whose spread is
// below 1e-6 of its scale gets sd = 1, so constant inputs standardize to zero.
__global__ void colstats_kernel(int64_t rows, int64_t cols, const float* __restrict__ D, float* __restrict__ mu,
                                float* __restrict__ sd) {
  __shared__ double r1[TPB], r2[TPB];
  const int64_t n = blockIdx.x;
  double s1 = 0.0, s2 = 0.0;
  for (int64_t r = threadIdx.x; r < rows; r += blockDim.x) {
    const double x = D[r * cols + n];
    s1 += x;
    s2 += x * x;
  }
  r1[threadIdx.x] = s1;
  r2[threadIdx.x] = s2;
  __syncthreads();
  for (int h = TPB / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      r1[threadIdx.x] += r1[threadIdx.x + h];
      r2[threadIdx.x] += r2[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double m = r1[0] / (double)rows;
    const double var = fmax(r2[0] / (double)rows - m * m, 0.0);
    const double d = sqrt(var);
    mu[n] = (float)m;
    sd[n] = (float)(d > 1e-6 * fmax(1.0, fabs(m)) ? d : 1.0);
  }
}

__global__ void adam_kernel(int64_t n, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[e];
    const float mi = b1 * m[e] + (1.0f - b1) * gi;
    const float vi = b2 * v[e] + (1.0f - b2) * gi * gi;
    m[e] = mi;
    v[e] = vi;
    p[e] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

__device__ inline uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// weights of layer l: U(-a, a), a = sqrt(6 / (fan_in + fan_out)); biases zero
__global__ void init_kernel(int64_t n_in, int64_t w, int64_t n_out, uint64_t seed, float* __restrict__ p) {
  const int64_t s1 = n_in * w, s2 = s1 + w, s3 = s2 + w * w, s4 = s3 + w, s5 = s4 + w * n_out, total = s5 + n_out;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    float a = 0.0f;
    if (e < s1) a = sqrtf(6.0f / (float)(n_in + w));
    else if (e >= s2 && e < s3) a = sqrtf(6.0f / (float)(2 * w));
    else if (e >= s4 && e < s5) a = sqrtf(6.0f / (float)(w + n_out));
    const double u = (double)(splitmix64(seed * 0x100000001B3ull + (uint64_t)e) >> 11) * (1.0 / 9007199254740992.0);
    p[e] = a == 0.0f ? 0.0f : a * (float)(2.0 * u - 1.0);
  }
}

// ---------------------------------------------------------------------------------------------
// BF16 inference: RT tiles of 16 rows per workgroup, all three layers, activations in LDS.  The four
// waves share the rows and take four of the sixteen column blocks each, so one tile of 16 rows
// already spreads over a CU's four matrix cores.  A prediction (some hundred to a few thousand rows)
// is bound by latency: the weights are packed in the order of the MFMA operands, a lane's pieces of
// two k-steps in one 16-byte load, and a wave's share of W2 (32 such loads) is in flight before the
// first layer starts.  1240 rows: 31.5 us with every wave reading all weights in 2-byte pieces.
// Every output sums the same products in the same order whatever RT is.
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

__device__ inline short to_bf16(float x) {  // round to nearest even
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const uint32_t r = u + 0x7FFFu + ((u >> 16) & 1u);
  return (short)(r >> 16);
}

constexpr int IW = 256;  // hidden width of the inference kernel
constexpr int KIN = 16;  // padded input width
constexpr int NOUT = 16; // padded output width
constexpr int NB = IW / 16, KP = IW / 32;  // column blocks; pairs of k-steps

__device__ inline bf16x4 half_of(bf16x8 v, int h) {
  return h ? __builtin_shufflevector(v, v, 4, 5, 6, 7) : __builtin_shufflevector(v, v, 0, 1, 2, 3);
}

// Wb: bf16 weights as MFMA B operands (lane l of a fragment: column l % 16, k = 4 (l / 16) + 0..3):
// W1 [16 column blocks][lane][4]; W2 [16 column blocks][8 pairs of k-steps][lane][2][4];
// W3 [8 pairs][lane][2][4] (zero padded).  bias fp32 [IW] | [IW] | [NOUT]
template <int RT>
__global__ __launch_bounds__(TPB) void infer_kernel(int64_t rows, int64_t n_in, int64_t n_out,
                                                   const float* __restrict__ X, const float* __restrict__ mu_in,
                                                   const float* __restrict__ sd_in, const short* __restrict__ Wb,
                                                   const float* __restrict__ bias, const float* __restrict__ mu_out,
                                                   const float* __restrict__ sd_out, float* __restrict__ Y) {
  constexpr int NW = 4, CB = NB / NW;           // waves, column blocks per wave
  __shared__ short act1[RT][16][IW + 8], act2[RT][16][IW + 8];  // bf16 activations, padded rows
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * (16 * RT);
  const bf16x4* W1 = (const bf16x4*)Wb + (CB * w) * 64 + lane;
  const bf16x8* W2 = (const bf16x8*)(Wb + KIN * IW) + (CB * w) * KP * 64 + lane;
  const bf16x8* W3 = (const bf16x8*)(Wb + KIN * IW + IW * IW) + lane;
  const float* b1 = bias;
  const float* b2 = b1 + IW;
  const float* b3 = b2 + IW;

  bf16x4 w1[CB];
  bf16x8 w2[CB][KP];
#pragma unroll
  for (int c = 0; c < CB; ++c) w1[c] = W1[c * 64];
#pragma unroll
  for (int c = 0; c < CB; ++c)
#pragma unroll
    for (int q = 0; q < KP; ++q) w2[c][q] = W2[(c * KP + q) * 64];

  // layer 1: one k-step; A fragment of the normalized input: row lr, k = 4 lk .. 4 lk + 3
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    bf16x4 xa;
    const int64_t r = r0 + 16 * rt + lr;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = 4 * lk + j;
      float x = 0.0f;
      if (r < rows && k < n_in) x = (X[r * n_in + k] - mu_in[k]) / sd_in[k];
      xa[j] = to_bf16(x);
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int n = 16 * (CB * w + c) + lr;
      const f4 acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(xa, w1[c], f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) act1[rt][4 * lk + j][n] = to_bf16(silu_f(acc[j] + b1[n]));
    }
  }
  __syncthreads();
  // layer 2: 16 k-steps
  f4 acc2[RT][CB];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CB; ++c) acc2[rt][c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < NB; ++ks)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const bf16x4 a = *(const bf16x4*)&act1[rt][lr][16 * ks + 4 * lk];
#pragma unroll
      for (int c = 0; c < CB; ++c)
        acc2[rt][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, half_of(w2[c][ks / 2], ks & 1), acc2[rt][c], 0, 0, 0);
    }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int n = 16 * (CB * w + c) + lr;
#pragma unroll
      for (int j = 0; j < 4; ++j) act2[rt][4 * lk + j][n] = to_bf16(silu_f(acc2[rt][c][j] + b2[n]));
    }
  __syncthreads();
  // layer 3: one column block (n_out <= 16), 16 k-steps; wave w takes row tiles w, w + 4, ...
  for (int rt = w; rt < RT; rt += NW) {
    f4 acc3 = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < NB; ++ks) {
      const bf16x4 a = *(const bf16x4*)&act2[rt][lr][16 * ks + 4 * lk];
      acc3 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, half_of(W3[(ks / 2) * 64], ks & 1), acc3, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t r = r0 + 16 * rt + 4 * lk + j;
      if (r < rows && lr < n_out) Y[r * n_out + lr] = (acc3[j] + b3[lr]) * sd_out[lr] + mu_out[lr];
    }
  }
}

// bf16 copy of the weights in the inference kernel's padded operand order, fp32 biases alongside
__global__ void pack_bf16_kernel(int64_t n_in, int64_t n_out, const float* __restrict__ p, short* __restrict__ Wb,
                                 float* __restrict__ bias) {
  const int64_t s1 = n_in * IW, s2 = s1 + IW, s3 = s2 + IW * IW, s4 = s3 + IW;
  const int64_t total = KIN * IW + IW * IW + IW * NOUT;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    float x = 0.0f;
    if (e < KIN * IW) {
      const int64_t j = e & 3, lane = (e >> 2) & 63, nb = e >> 8, k = 4 * (lane >> 4) + j;
      if (k < n_in) x = p[k * IW + 16 * nb + (lane & 15)];
    } else {
      const int64_t f = e < KIN * IW + IW * IW ? e - KIN * IW : e - KIN * IW - IW * IW;
      const int64_t j = f & 3, h = (f >> 2) & 1, lane = (f >> 3) & 63, q = (f >> 9) % KP, nb = f / (512 * KP);
      const int64_t k = 16 * (2 * q + h) + 4 * (lane >> 4) + j, c = lane & 15;
      if (e < KIN * IW + IW * IW) x = p[s2 + k * IW + 16 * nb + c];
      else if (c < n_out) x = p[s4 + k * n_out + c];
    }
    Wb[e] = to_bf16(x);
  }
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < 2 * IW + NOUT; e += (int64_t)gridDim.x * blockDim.x) {
    float x = 0.0f;
    if (e < IW) x = p[s1 + e];
    else if (e < 2 * IW) x = p[s3 + (e - IW)];
    else if (e - 2 * IW < n_out) x = p[s4 + IW * n_out + (e - 2 * IW)];
    bias[e] = x;
  }
}

// ---------------------------------------------------------------------------------------------
// Training of a network of the guess network's class: width 256, n_in <= 16, n_out <= 16, FP32.
// The separate products left the chip idle: a weight gradient has K = rows but at most 16 output
// tiles (722 us each at 4096 rows, on 4 to 16 workgroups).
constexpr int TR = 16, TNT = 512, TNW = TNT / 64;  // rows per tile, threads and waves of train_rows
constexpr int HP = IW + 4;                         // LDS row pitch of an activation tile

__device__ inline f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// Forward pass, loss gradient and backward pass of tiles of 16 rows (a workgroup walks tiles
// blockIdx.x, + gridDim.x, ...), on v_mfma_f32_16x16x4f32 with W2 read from L2 as the MFMA B operand
// (8- and 16-byte loads; the k of a step and the columns of a tile are taken in the order in which
// such a load delivers them) and the tile's activations as A from LDS.  Eight waves, 32 columns each.
// Written for every row: H1 (first hidden activations) and D2 (gradient at the second layer's
// pre-activations), the operands of dW2; for the workgroup: its sums for the other parameters,
// part[workgroup][dW1 | db1 | db2 | dW3 | db3], and its loss sum.  16 rows a tile rather than 32: a
// minibatch of 4096 rows is then one tile per CU, and the chain of one tile is what it waits for.
template <int NO>
__global__ __launch_bounds__(TNT) void train_rows_kernel(int64_t rows, int n_in, int n_out, const float* __restrict__ X,
                                                         const float* __restrict__ T, const float* __restrict__ mu_in,
                                                         const float* __restrict__ sd_in,
                                                         const float* __restrict__ mu_out,
                                                         const float* __restrict__ sd_out, const float* __restrict__ p,
                                                         float* __restrict__ H1, float* __restrict__ D2,
                                                         float* __restrict__ part, double* __restrict__ lpart) {
  __shared__ __attribute__((aligned(16))) float hA[TR][HP], hB[TR][HP];
  __shared__ float xs[TR][KIN], dys[TR][NO], red[TNW][TR][NO];
  __shared__ double lred[TR * NO];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, lr = lane & 15, lk = lane >> 4;
  const float *W1 = p, *b1 = W1 + n_in * IW, *W2 = b1 + IW, *b2 = W2 + IW * IW, *W3 = b2 + IW, *b3 = W3 + IW * n_out;
  // layer 1 and its gradient: thread = column c and eight of the tile's rows
  const int c = t & (IW - 1), rh = (t >> 8) * 8;
  float w1[KIN], gw1[KIN], gb1 = 0.0f;
#pragma unroll
  for (int k = 0; k < KIN; ++k) {
    w1[k] = k < n_in ? W1[k * IW + c] : 0.0f;
    gw1[k] = 0.0f;
  }
  const float b1c = b1[c];
  // layers 2 and 3: this lane's columns of the second layer
  const int col = 32 * w + 2 * lr;
  float w3[2][NO], gw3[2][NO], gb2[2] = {0.0f, 0.0f}, b2c[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    b2c[q] = b2[col + q];
#pragma unroll
    for (int j = 0; j < NO; ++j) {
      w3[q][j] = j < n_out ? W3[(col + q) * n_out + j] : 0.0f;
      gw3[q][j] = 0.0f;
    }
  }
  const float scale = 2.0f / (float)(rows * n_out);
  float gb3 = 0.0f;
  double loss = 0.0;

  for (int64_t tile = blockIdx.x; tile * TR < rows; tile += gridDim.x) {
    const int64_t r0 = tile * TR;
    if (t < TR * KIN) {
      const int r = t / KIN, k = t % KIN;
      xs[r][k] = (r0 + r < rows && k < n_in) ? (X[(r0 + r) * n_in + k] - mu_in[k]) / sd_in[k] : 0.0f;
    }
    __syncthreads();
    float z1[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float x = 0.0f;
#pragma unroll
      for (int k = 0; k < KIN; ++k) x = __builtin_fmaf(xs[rh + r][k], w1[k], x);
      z1[r] = x + b1c;
      const float h = silu_f(z1[r]);
      hA[rh + r][c] = h;
      if (r0 + rh + r < rows) H1[(r0 + rh + r) * IW + c] = h;
    }
    __syncthreads();
    f4 acc[2] = {f4{0, 0, 0, 0}, f4{0, 0, 0, 0}};
#pragma unroll 4
    for (int ks = 0; ks < IW / 16; ++ks) {
      const f4 a = *(const f4*)&hA[lr][16 * ks + 4 * lk];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const f2 b = *(const f2*)&W2[(16 * ks + 4 * lk + s) * IW + col];
        acc[0] = mfma4(a[s], b.x, acc[0]);
        acc[1] = mfma4(a[s], b.y, acc[1]);
      }
    }
    // element r of acc[q]: row 4 lk + r, column col + q
    float z2[2][4], h2[2][4];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z2[q][r] = acc[q][r] + b2c[q];
        h2[q][r] = silu_f(z2[q][r]);
      }
#pragma unroll
    for (int j = 0; j < NO; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float y = h2[0][r] * w3[0][j] + h2[1][r] * w3[1][j];
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) y += __shfl_xor(y, off, 64);
        if (lr == 0) red[w][4 * lk + r][j] = y;
      }
    __syncthreads();
    if (t < TR * NO) {
      const int r = t / NO, j = t % NO;
      float d = 0.0f;
      if (r0 + r < rows && j < n_out) {
        float y = 0.0f;
#pragma unroll
        for (int q = 0; q < TNW; ++q) y += red[q][r][j];
        d = y + b3[j] - (T[(r0 + r) * n_out + j] - mu_out[j]) / sd_out[j];
      }
      loss += (double)d * (double)d;
      dys[r][j] = scale * d;
      gb3 += scale * d;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      f2 d2;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float x = 0.0f;
#pragma unroll
        for (int j = 0; j < NO; ++j) {
          const float dy = dys[4 * lk + r][j];
          x = __builtin_fmaf(dy, w3[q][j], x);
          gw3[q][j] = __builtin_fmaf(h2[q][r], dy, gw3[q][j]);
        }
        d2[q] = x * silu_grad_f(z2[q][r]);
        gb2[q] += d2[q];
      }
      *(f2*)&hB[4 * lk + r][col] = d2;
      if (r0 + 4 * lk + r < rows) *(f2*)&D2[(r0 + 4 * lk + r) * IW + col] = d2;
    }
    __syncthreads();
    acc[0] = acc[1] = f4{0, 0, 0, 0};
#pragma unroll 4
    for (int ks = 0; ks < IW / 16; ++ks) {
      const f4 a = *(const f4*)&hB[lr][16 * ks + 4 * lk];
      const f4 u = *(const f4*)&W2[(32 * w + lr) * IW + 16 * ks + 4 * lk];
      const f4 v = *(const f4*)&W2[(32 * w + 16 + lr) * IW + 16 * ks + 4 * lk];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        acc[0] = mfma4(a[s], u[s], acc[0]);
        acc[1] = mfma4(a[s], v[s], acc[1]);
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) hA[4 * lk + r][32 * w + 16 * q + lr] = acc[q][r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float d1 = hA[rh + r][c] * silu_grad_f(z1[r]);
      gb1 += d1;
#pragma unroll
      for (int k = 0; k < KIN; ++k) gw1[k] = __builtin_fmaf(xs[rh + r][k], d1, gw1[k]);
    }
    __syncthreads();  // xs and hA are free for the next tile
  }

  const int n1 = (n_in + 1) * IW;  // dW1, db1
  float* out = part + (int64_t)blockIdx.x * (n1 + IW + (IW + 1) * n_out);
  if (rh) {
#pragma unroll
    for (int k = 0; k < KIN; ++k) hA[k][c] = gw1[k];
    hB[0][c] = gb1;
  }
  if (t < TR * NO) {
    lred[t] = loss;
    red[0][t / NO][t % NO] = gb3;
  }
  __syncthreads();
  if (!rh) {
#pragma unroll
    for (int k = 0; k < KIN; ++k)
      if (k < n_in) out[k * IW + c] = gw1[k] + hA[k][c];
    out[n_in * IW + c] = gb1 + hB[0][c];
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float x = gb2[q];
    x += __shfl_xor(x, 16, 64);
    x += __shfl_xor(x, 32, 64);
    if (lk == 0) out[n1 + col + q] = x;
#pragma unroll
    for (int j = 0; j < NO; ++j) {
      float g = gw3[q][j];
      g += __shfl_xor(g, 16, 64);
      g += __shfl_xor(g, 32, 64);
      if (lk == 0 && j < n_out) out[n1 + IW + (col + q) * n_out + j] = g;
    }
  }
  if (t < n_out) {
    float x = 0.0f;
    for (int r = 0; r < TR; ++r) x += red[0][r][t];
    out[n1 + IW + IW * n_out + t] = x;
  }
  if (t == 0) {
    double x = 0.0;
    for (int k = 0; k < TR * NO; ++k) x += lred[k];
    lpart[blockIdx.x] = x;
  }
}

// dW2 = H1^T D2 over the rows, cut into gridDim.y row ranges: part[range][256][256].  A workgroup owns
// a 64 x 64 tile, its four waves every fourth step of four rows, added up through LDS; a lane's
// 16-byte load of a row of H1 (D2) feeds the A (B) operands of four MFMA tiles, so nothing is staged.
__global__ __launch_bounds__(TPB) void train_w2_kernel(int64_t rows, int64_t per, const float* __restrict__ H1,
                                                       const float* __restrict__ D2, float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) float sum[4][64][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
  const int k0 = (blockIdx.x >> 2) * 64, n0 = (blockIdx.x & 3) * 64;
  const int64_t beg = (int64_t)blockIdx.y * per, end = beg + per < rows ? beg + per : rows;
  f4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f4{0, 0, 0, 0};
#pragma unroll 4
  for (int64_t r = beg + 4 * w; r < end; r += 16) {
    const bool ok = r + lk < end;
    const f4 zero = f4{0, 0, 0, 0};
    const f4 a = ok ? *(const f4*)&H1[(r + lk) * IW + k0 + 4 * lr] : zero;
    const f4 b = ok ? *(const f4*)&D2[(r + lk) * IW + n0 + 4 * lr] : zero;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = mfma4(a[i], b[j], acc[i][j]);
  }
  // element r of acc[i][j]: k = k0 + 4 (4 lk + r) + i, n = n0 + 4 lr + j
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *(f4*)&sum[w][4 * (4 * lk + r) + i][4 * lr] = f4{acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]};
  __syncthreads();
  float* out = part + (int64_t)blockIdx.y * IW * IW;
  for (int e = threadIdx.x; e < 64 * 16; e += TPB) {
    const int k = e >> 4, n = (e & 15) * 4;
    const f4 x = *(const f4*)&sum[0][k][n] + *(const f4*)&sum[1][k][n] + *(const f4*)&sum[2][k][n] + *(const f4*)&sum[3][k][n];
    *(f4*)&out[(k0 + k) * IW + n0 + n] = x;
  }
}

// The gradient from the partials of train_rows (nw workgroups) and train_w2 (ns ranges), the loss, and
// the Adam step (lr > 0).  Blocks 0..255: a row of dW2, one element a thread; then blocks of 32 other
// parameters, eight threads each (every eighth workgroup's partial).
__global__ __launch_bounds__(TPB) void train_update_kernel(int n_in, int n_out, int nw, int ns,
                                                           const float* __restrict__ part,
                                                           const float* __restrict__ part2,
                                                           const double* __restrict__ lpart, double denom,
                                                           float* __restrict__ loss, float* __restrict__ p,
                                                           float* __restrict__ g, float* __restrict__ m,
                                                           float* __restrict__ v, float lr, float b1, float b2, float eps,
                                                           float c1, float c2) {
  __shared__ float red[8][32];
  const int n1 = (n_in + 1) * IW, no = n1 + IW + (IW + 1) * n_out;  // parameters outside W2
  int64_t e = -1;
  float x = 0.0f;
  if (blockIdx.x < IW) {
    const int64_t k = (int64_t)blockIdx.x * IW + threadIdx.x;
#pragma unroll 8
    for (int s = 0; s < ns; ++s) x += part2[(int64_t)s * IW * IW + k];
    e = n1 + k;
  } else {
    const int tp = threadIdx.x & 31, tg = threadIdx.x >> 5, q = (blockIdx.x - IW) * 32 + tp;
    if (q < no)
#pragma unroll 8
      for (int s = tg; s < nw; s += 8) x += part[(int64_t)s * no + q];
    red[tg][tp] = x;
    __syncthreads();
    if (tg == 0 && q < no) {
      for (int k = 1; k < 8; ++k) x += red[k][tp];
      e = q < n1 ? q : q + IW * IW;
    }
    if (blockIdx.x == IW && tg == 1) {  // the loss, by one half wave
      double s = 0.0;
      for (int k = tp; k < nw; k += 32) s += lpart[k];
      for (int off = 16; off > 0; off >>= 1) s += __shfl_xor(s, off, 32);
      if (tp == 0) loss[0] = (float)(s / denom);
    }
  }
  if (e < 0) return;
  g[e] = x;
  if (lr > 0.0f) {
    const float mi = b1 * m[e] + (1.0f - b1) * x;
    const float vi = b2 * v[e] + (1.0f - b2) * x * x;
    m[e] = mi;
    v[e] = vi;
    p[e] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

// Workgroups of 16 rows up to this many (every CU busy twice over); past that four row tiles share
// one read of the weights.
constexpr int64_t INFER_FEW = 512;
constexpr int64_t TRAIN_WGS = 512;    // most workgroups of train_rows (partials per parameter)
constexpr int64_t TRAIN_RANGES = 32;  // most row ranges of train_w2 (16 tiles each: two workgroups a CU)

unsigned nblk(int64_t n) {
  int64_t b = (n + TPB - 1) / TPB;
  if (b < 1) b = 1;
  if (b > 4096) b = 4096;
  return (unsigned)b;
}

}  // namespace

// Scratch of the allocation-free FP32 forward pass: the activations of one call live in this
// file-scope device array (MLP_SCRATCH_FLOATS floats, 32 MiB), which every GPU the library runs on
// holds until the process ends.  In host code `scratch` is only a stand-in for the symbol, not a
// device address: kernels get the address that mlp_scratch_resolve looked up for the device.
static __device__ __align__(256) float scratch[MLP_SCRATCH_FLOATS];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
float* scratch_at[MAX_DEVICES] = {};  // device address of `scratch` per device id, once resolved
}  // namespace

hipError_t mlp_scratch_resolve(float** out) {
  *out = nullptr;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_at[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    scratch_at[dev] = static_cast<float*>(p);
  }
  *out = scratch_at[dev];
  return hipSuccess;
}

hipError_t mlp_sgemm(bool tA, bool tB, int epi, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                     const float* B, int64_t ldb, float* C, int64_t ldc, const float* bias, float* Z, int64_t ldz,
                     hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if ((M + BM - 1) / BM > 65535) return hipErrorInvalidValue;
  dim3 grid((unsigned)((N + BN - 1) / BN), (unsigned)((M + BM - 1) / BM));
#define SG(TA, TB, E) hipLaunchKernelGGL((sgemm_kernel<TA, TB, E>), grid, dim3(TPB), 0, s, M, N, K, A, lda, B, ldb, C, ldc, bias, Z, ldz)
  if (!tA && !tB) {
    if (epi == 1) SG(false, false, 1); else if (epi == 2) SG(false, false, 2); else if (epi == 4) SG(false, false, 4);
    else SG(false, false, 0);
  } else if (tA && !tB) {
    SG(true, false, 0);
  } else if (!tA && tB) {
    if (epi == 3) SG(false, true, 3); else SG(false, true, 0);
  } else {
    return hipErrorInvalidValue;
  }
#undef SG
  return hipGetLastError();
}

hipError_t mlp_normalize(int64_t rows, int64_t cols, const float* X, const float* mu, const float* sd, float* Xn,
                         hipStream_t s) {
  hipLaunchKernelGGL(normalize_kernel, dim3(nblk(rows * cols)), dim3(TPB), 0, s, rows, cols, X, mu, sd, Xn);
  return hipGetLastError();
}

hipError_t mlp_denorm(int64_t rows, int64_t cols, const float* Yn, const float* mu, const float* sd, float* Y,
                      hipStream_t s) {
  hipLaunchKernelGGL(denorm_kernel, dim3(nblk(rows * cols)), dim3(TPB), 0, s, rows, cols, Yn, mu, sd, Y);
  return hipGetLastError();
}

hipError_t mlp_mse_grad(int64_t rows, int64_t cols, const float* Yn, const float* T, const float* mu, const float* sd,
                        float* dY, double* part, int64_t nparts, float* loss, hipStream_t s) {
  const unsigned nb = (unsigned)std::min<int64_t>(nparts, nblk(rows * cols));
  hipLaunchKernelGGL(mse_grad_kernel, dim3(nb), dim3(TPB), 0, s, rows, cols, Yn, T, mu, sd, dY, part);
  hipLaunchKernelGGL(sum_parts_kernel, dim3(1), dim3(TPB), 0, s, (int64_t)nb, part, (double)(rows * cols), loss);
  return hipGetLastError();
}

hipError_t mlp_colsum(int64_t rows, int64_t cols, const float* D, float* out, hipStream_t s) {
  if (cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(colsum_kernel, dim3((unsigned)cols), dim3(TPB), 0, s, rows, cols, D, out);
  return hipGetLastError();
}

hipError_t mlp_colstats(int64_t rows, int64_t cols, const float* D, float* mu, float* sd, hipStream_t s) {
  if (cols <= 0 || rows <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(colstats_kernel, dim3((unsigned)cols), dim3(TPB), 0, s, rows, cols, D, mu, sd);
  return hipGetLastError();
}

hipError_t mlp_adam(int64_t n, float* p, const float* g, float* m, float* v, float lr, float b1, float b2, float eps,
                    int64_t step, hipStream_t s) {
  const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3(nblk(n)), dim3(TPB), 0, s, n, p, g, m, v, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t mlp_init(int64_t n_in, int64_t w, int64_t n_out, uint64_t seed, float* p, hipStream_t s) {
  const int64_t total = n_in * w + w + w * w + w + w * n_out + n_out;
  hipLaunchKernelGGL(init_kernel, dim3(nblk(total)), dim3(TPB), 0, s, n_in, w, n_out, seed, p);
  return hipGetLastError();
}

bool mlp_infer_supported(int64_t n_in, int64_t w, int64_t n_out) {
  return w == IW && n_in >= 1 && n_in <= KIN && n_out >= 1 && n_out <= NOUT;
}
int64_t mlp_bf16_weights(int64_t) { return KIN * IW + IW * IW + IW * NOUT; }
int64_t mlp_bf16_biases() { return 2 * IW + NOUT; }

hipError_t mlp_pack_bf16(int64_t n_in, int64_t n_out, const float* p, short* Wb, float* bias, hipStream_t s) {
  hipLaunchKernelGGL(pack_bf16_kernel, dim3(nblk(KIN * IW + IW * IW + IW * NOUT)), dim3(TPB), 0, s, n_in, n_out, p, Wb,
                     bias);
  return hipGetLastError();
}

hipError_t mlp_infer_bf16(int64_t rows, int64_t n_in, int64_t n_out, const float* X, const float* mu_in,
                          const float* sd_in, const short* Wb, const float* bias, const float* mu_out,
                          const float* sd_out, float* Y, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const bool few = rows <= 16 * INFER_FEW;
  const int64_t per = few ? 16 : 64, nb = (rows + per - 1) / per;
  if (nb > 2147483647LL) return hipErrorInvalidValue;
  if (few)
    hipLaunchKernelGGL(infer_kernel<1>, dim3((unsigned)nb), dim3(TPB), 0, s, rows, n_in, n_out, X, mu_in, sd_in, Wb,
                       bias, mu_out, sd_out, Y);
  else
    hipLaunchKernelGGL(infer_kernel<4>, dim3((unsigned)nb), dim3(TPB), 0, s, rows, n_in, n_out, X, mu_in, sd_in, Wb,
                       bias, mu_out, sd_out, Y);
  return hipGetLastError();
}

// Workgroups of train_rows, row ranges of dW2 (256 rows, 16 MFMA steps a wave, or more each) and the length
// of the workgroups' partials (the ranges' start 16 bytes aligned behind them).
static int64_t train_wgs(int64_t rows) { return std::min<int64_t>((rows + TR - 1) / TR, TRAIN_WGS); }
static int64_t train_ranges(int64_t rows) { return std::min<int64_t>((rows + 255) / 256, TRAIN_RANGES); }
static int64_t train_part_floats(int64_t rows, int64_t n_in, int64_t n_out) {
  return (train_wgs(rows) * ((n_in + 2) * IW + (IW + 1) * n_out) + 3) / 4 * 4;
}
int64_t mlp_train_floats(int64_t rows, int64_t n_in, int64_t n_out) {
  return train_part_floats(rows, n_in, n_out) + train_ranges(rows) * IW * IW;
}

hipError_t mlp_train(int64_t rows, int64_t n_in, int64_t n_out, const float* X, const float* T, const float* mu_in,
                     const float* sd_in, const float* mu_out, const float* sd_out, float* p, float* H1, float* D2,
                     float* part, double* lpart, float* loss, float* g, float* m, float* v, float lr, float b1,
                     float b2, float eps, int64_t step, hipStream_t s) {
  if (rows < 1 || !mlp_infer_supported(n_in, IW, n_out)) return hipErrorInvalidValue;
  const int nw = (int)train_wgs(rows);
  const int64_t want = train_ranges(rows);
  const int64_t per = ((rows + want - 1) / want + 15) / 16 * 16, ns = (rows + per - 1) / per;
  float* part2 = part + train_part_floats(rows, n_in, n_out);
#define ROWS(NO) hipLaunchKernelGGL(train_rows_kernel<NO>, dim3((unsigned)nw), dim3(TNT), 0, s, rows, (int)n_in, (int)n_out, X, T, mu_in, sd_in, mu_out, sd_out, p, H1, D2, part, lpart)
  if (n_out <= 2) ROWS(2); else ROWS(NOUT);
#undef ROWS
  hipLaunchKernelGGL(train_w2_kernel, dim3(16, (unsigned)ns), dim3(TPB), 0, s, rows, per, H1, D2, part2);
  const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
  const int64_t others = (n_in + 2) * IW + (IW + 1) * n_out;
  hipLaunchKernelGGL(train_update_kernel, dim3((unsigned)(IW + (others + 31) / 32)), dim3(TPB), 0, s, (int)n_in, (int)n_out,
                     nw, (int)ns, part, part2, lpart, (double)(rows * n_out), loss, p, g, m, v, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace thc
