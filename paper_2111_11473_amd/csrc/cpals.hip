// Kernels of the weighted CP-ALS (paper Sec. II.c-d, Appendix I): the reductions that finish the
// matricized-tensor-times-Khatri-Rao products after their matrix-product part, and the column-wise
// steps of the block preconditioned conjugate gradients that solve S U = B for every row of a
// factor at once (S the n x n Hadamard product of Gram matrices, preconditioned by its diagonal;
// U, B stored [n][m], column c one right-hand side).
//
// One CG iteration is the product S P in K slices (gemm_f64) and three passes over [n][m]: the sum
// of the slices with the partial p.q, the step with the partial r.r and r.z, and the new direction.
// Z = R / d is never stored.  Every pass cuts the rows into `splits` ranges so that a few columns
// still fill the chip, and leaves one partial per range and column ([splits][m], fixed order); the
// next pass adds them up for its own columns.  What bounds an iteration is launches (four, 4-7 us
// each) and, for many columns, the product.  At n = 1000 and 20 to 600 columns an iteration took
// ~700 us when each column's dot product was one thread's walk down the rows (250 us a dot, three
// of them) and the host read the residuals every iteration.
//
// Convergence is decided on the device: flag[k] says whether iteration k of a batch has to run; the
// direction pass of iteration k sets flag[k + 1] if some column is still above its tolerance, and
// the passes of an iteration whose flag is 0 do nothing.  The host reads the flags once a batch.
#include "internal.h"

namespace thc {
namespace {

constexpr int TPB = 256;

unsigned grid_of(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + TPB - 1) / TPB, 65536)); }

// out[r][c] = w[r]^2 X[r][c] (w null: a copy)
__global__ void weighted_rows_kernel(int64_t m, int64_t n, const double* __restrict__ w, const double* __restrict__ X,
                                     double* __restrict__ out) {
  for (int64_t e = (int64_t)blockIdx.x * TPB + threadIdx.x; e < m * n; e += (int64_t)gridDim.x * TPB) {
    const double s = w ? w[e / n] : 1.0;
    out[e] = s * s * X[e];
  }
}

// T[i][j][c] (I x J x n); over_j: out[c][i] = sum_j V[j][c] T[i][j][c]; else out[c][j] = sum_i V[i][c] T[i][j][c]
__global__ void mttkrp_reduce_kernel(int64_t I, int64_t J, int64_t n, const double* __restrict__ T,
                                     const double* __restrict__ V, bool over_j, double* __restrict__ out) {
  const int64_t rows = over_j ? I : J, len = over_j ? J : I;
  for (int64_t e = (int64_t)blockIdx.x * TPB + threadIdx.x; e < rows * n; e += (int64_t)gridDim.x * TPB) {
    const int64_t r = e / n, c = e % n;
    double s = 0.0;
    if (over_j)
      for (int64_t j = 0; j < len; ++j) s += V[j * n + c] * T[(r * J + j) * n + c];
    else
      for (int64_t i = 0; i < len; ++i) s += V[i * n + c] * T[(i * J + r) * n + c];
    out[c * rows + r] = s;
  }
}

// sum of (w1_i w2_j w3_k A_ijk)^2, one partial per block
__global__ void wnorm2_kernel(int64_t I, int64_t J, int64_t K, const double* __restrict__ A,
                              const double* __restrict__ w1, const double* __restrict__ w2,
                              const double* __restrict__ w3, double* __restrict__ part) {
  __shared__ double red[TPB];
  double s = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * TPB + threadIdx.x; e < I * J * K; e += (int64_t)gridDim.x * TPB) {
    const int64_t k = e % K, ij = e / K, j = ij % J, i = ij / J;
    const double w = (w1 ? w1[i] : 1.0) * (w2 ? w2[j] : 1.0) * (w3 ? w3[k] : 1.0);
    const double x = w * A[e];
    s += x * x;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = TPB / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

constexpr int CC = 64, CR = TPB / CC;  // columns and row lanes of a block of the CG passes

// Sum over the splits of one column's partials: each of the block's row lanes takes every CR-th.
__device__ inline double split_sum(const double* __restrict__ part, int64_t m, int64_t c, double (&red)[CR][CC]) {
  const int tc = threadIdx.x % CC, tr = threadIdx.x / CC, splits = gridDim.y;
  double s = 0.0;
  if (c < m)
#pragma unroll 4
    for (int k = tr; k < splits; k += CR) s += part[(int64_t)k * m + c];
  __syncthreads();
  red[tr][tc] = s;
  __syncthreads();
  s = red[0][tc];
#pragma unroll
  for (int k = 1; k < CR; ++k) s += red[k][tc];
  return s;
}
// Element e of a matrix held as ns slices.
__device__ inline double slice_sum(const double* __restrict__ X, int64_t nm, int ns, int64_t e) {
  double q = 0.0;
#pragma unroll 4
  for (int k = 0; k < ns; ++k) q += X[(int64_t)k * nm + e];
  return q;
}
// The block's row lanes of one column added up, by row lane 0, into part[split][c].
__device__ inline void put_partial(double x, double (&red)[CR][CC], int64_t m, int64_t c, double* __restrict__ part) {
  const int tc = threadIdx.x % CC, tr = threadIdx.x / CC;
  __syncthreads();
  red[tr][tc] = x;
  __syncthreads();
  if (tr == 0 && c < m) {
    double s = red[0][tc];
#pragma unroll
    for (int k = 1; k < CR; ++k) s += red[k][tc];
    part[(int64_t)blockIdx.y * m + c] = s;
  }
}
// Rows r0 <= r < r1 of split blockIdx.y, walked by row lane in steps of CR; column c of the thread.
struct CgPos {
  int64_t c, r, r1;
};
__device__ inline CgPos cg_pos(int64_t n) {
  const int64_t per = (n + gridDim.y - 1) / gridDim.y, r0 = (int64_t)blockIdx.y * per;
  return {(int64_t)blockIdx.x * CC + threadIdx.x % CC, r0 + threadIdx.x / CC, r0 + per < n ? r0 + per : n};
}

// R = B - sum of the ns slices of S U;  P = R / d;  partials of r.(r / d) and b.b
__global__ __launch_bounds__(TPB) void cg_start_kernel(int64_t n, int64_t m, int ns, const double* __restrict__ SU,
                                                       const double* __restrict__ B, const double* __restrict__ d,
                                                       double* __restrict__ R, double* __restrict__ P,
                                                       double* __restrict__ rz, double* __restrict__ bb) {
  __shared__ double red[CR][CC];
  const CgPos at = cg_pos(n);
  double sz = 0.0, sb = 0.0;
  if (at.c < m)
#pragma unroll 4
    for (int64_t r = at.r; r < at.r1; r += CR) {
      const int64_t e = r * m + at.c;
      const double b = B[e], x = b - slice_sum(SU, n * m, ns, e), z = x / d[r];
      R[e] = x;
      P[e] = z;
      sz += x * z;
      sb += b * b;
    }
  put_partial(sz, red, m, at.c, rz);
  put_partial(sb, red, m, at.c, bb);
}

// Q = sum of the ns slices of S P;  partials of p.q
__global__ __launch_bounds__(TPB) void cg_pq_kernel(int64_t n, int64_t m, int ns, const double* __restrict__ SP,
                                                    const double* __restrict__ P, double* __restrict__ Q,
                                                    double* __restrict__ pq, const int* __restrict__ flag) {
  if (*flag == 0) return;
  __shared__ double red[CR][CC];
  const CgPos at = cg_pos(n);
  double s = 0.0;
  if (at.c < m)
#pragma unroll 4
    for (int64_t r = at.r; r < at.r1; r += CR) {
      const int64_t e = r * m + at.c;
      const double q = slice_sum(SP, n * m, ns, e);
      Q[e] = q;
      s += P[e] * q;
    }
  put_partial(s, red, m, at.c, pq);
}

// alpha_c = rz_c / pq_c (0 where pq_c is 0);  U += alpha p;  R -= alpha q;  partials of r.r and r.(r / d)
__global__ __launch_bounds__(TPB) void cg_step_kernel(int64_t n, int64_t m, const double* __restrict__ rz,
                                                      const double* __restrict__ pq, const double* __restrict__ P,
                                                      const double* __restrict__ Q, const double* __restrict__ d,
                                                      double* __restrict__ U, double* __restrict__ R,
                                                      double* __restrict__ rr, double* __restrict__ rz_new,
                                                      const int* __restrict__ flag) {
  if (*flag == 0) return;
  __shared__ double red[CR][CC];
  const CgPos at = cg_pos(n);
  double sr = 0.0, sz = 0.0;
  const double num = split_sum(rz, m, at.c, red), den = split_sum(pq, m, at.c, red);
  const double a = den != 0.0 ? num / den : 0.0;
  if (at.c < m) {
#pragma unroll 4
    for (int64_t r = at.r; r < at.r1; r += CR) {
      const int64_t e = r * m + at.c;
      U[e] += a * P[e];
      const double x = R[e] - a * Q[e];
      R[e] = x;
      sr += x * x;
      sz += x * (x / d[r]);
    }
  }
  put_partial(sr, red, m, at.c, rr);
  put_partial(sz, red, m, at.c, rz_new);
}

// P = R / d + (rz_new / rz_old) P  (beta 0 where rz_old is 0); the first row split of every column
// block sets flag[1] if a column's |r| is above tol |b|
__global__ __launch_bounds__(TPB) void cg_dir_kernel(int64_t n, int64_t m, double tol, const double* __restrict__ rz_new,
                                                     const double* __restrict__ rz_old, const double* __restrict__ rr,
                                                     const double* __restrict__ bb, const double* __restrict__ R,
                                                     const double* __restrict__ d, double* __restrict__ P,
                                                     int* __restrict__ flag) {
  if (flag[0] == 0) return;
  __shared__ double red[CR][CC];
  const CgPos at = cg_pos(n);
  if (blockIdx.y == 0) {
    const double res = sqrt(split_sum(rr, m, at.c, red)), lim = tol * sqrt(split_sum(bb, m, at.c, red));
    if (at.c < m && !(res <= lim)) flag[1] = 1;  // every writer stores the same value
  }
  const double old = split_sum(rz_old, m, at.c, red), now = split_sum(rz_new, m, at.c, red);
  const double b = old != 0.0 ? now / old : 0.0;
  if (at.c >= m) return;
#pragma unroll 4
  for (int64_t r = at.r; r < at.r1; r += CR) {
    const int64_t e = r * m + at.c;
    P[e] = R[e] / d[r] + b * P[e];
  }
}

__global__ void cg_flags_kernel(int count, int* __restrict__ flag) {
  for (int k = threadIdx.x; k < count; k += blockDim.x) flag[k] = k == 0;
}

__global__ void diag_kernel(int64_t n, const double* __restrict__ S, double* __restrict__ d) {
  for (int64_t r = (int64_t)blockIdx.x * TPB + threadIdx.x; r < n; r += (int64_t)gridDim.x * TPB) d[r] = S[r * n + r];
}

}  // namespace

#define CP_LAUNCH(kernel, n, ...)                                                      \
  do {                                                                                 \
    hipLaunchKernelGGL(kernel, dim3(grid_of(n)), dim3(TPB), 0, s, __VA_ARGS__);       \
    return hipGetLastError();                                                          \
  } while (0)

hipError_t cp_weighted_rows(int64_t m, int64_t n, const double* w, const double* X, double* out, hipStream_t s) {
  CP_LAUNCH(weighted_rows_kernel, m * n, m, n, w, X, out);
}
hipError_t cp_mttkrp_reduce(int64_t I, int64_t J, int64_t n, const double* T, const double* V, bool over_j,
                            double* out, hipStream_t s) {
  CP_LAUNCH(mttkrp_reduce_kernel, (over_j ? I : J) * n, I, J, n, T, V, over_j, out);
}
int64_t cp_wnorm2_parts(int64_t I, int64_t J, int64_t K) { return (int64_t)grid_of(I * J * K); }
hipError_t cp_wnorm2(int64_t I, int64_t J, int64_t K, const double* A, const double* w1, const double* w2,
                     const double* w3, double* part, hipStream_t s) {
  CP_LAUNCH(wnorm2_kernel, I * J * K, I, J, K, A, w1, w2, w3, part);
}
// Row ranges of the CG passes: four rows a thread (their loads in flight together) for up to 64 ranges.
// At n = 1000 and 20 to 600 columns 15 ranges of 17 rows a thread took 31, 15 and 18 us a pass.
int cp_cg_splits(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(64, n / (4 * CR))); }
static dim3 cg_grid(int64_t n, int64_t m) { return dim3((unsigned)((m + CC - 1) / CC), (unsigned)cp_cg_splits(n)); }
hipError_t cp_cg_start(int64_t n, int64_t m, int ns, const double* SU, const double* B, const double* d, double* R,
                       double* P, double* rz, double* bb, hipStream_t s) {
  hipLaunchKernelGGL(cg_start_kernel, cg_grid(n, m), dim3(TPB), 0, s, n, m, ns, SU, B, d, R, P, rz, bb);
  return hipGetLastError();
}
hipError_t cp_cg_pq(int64_t n, int64_t m, int ns, const double* SP, const double* P, double* Q, double* pq,
                    const int* flag, hipStream_t s) {
  hipLaunchKernelGGL(cg_pq_kernel, cg_grid(n, m), dim3(TPB), 0, s, n, m, ns, SP, P, Q, pq, flag);
  return hipGetLastError();
}
hipError_t cp_cg_step(int64_t n, int64_t m, const double* rz, const double* pq, const double* P, const double* Q,
                      const double* d, double* U, double* R, double* rr, double* rz_new, const int* flag,
                      hipStream_t s) {
  hipLaunchKernelGGL(cg_step_kernel, cg_grid(n, m), dim3(TPB), 0, s, n, m, rz, pq, P, Q, d, U, R, rr, rz_new, flag);
  return hipGetLastError();
}
hipError_t cp_cg_dir(int64_t n, int64_t m, double tol, const double* rz_new, const double* rz_old, const double* rr,
                     const double* bb, const double* R, const double* d, double* P, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(cg_dir_kernel, cg_grid(n, m), dim3(TPB), 0, s, n, m, tol, rz_new, rz_old, rr, bb, R, d, P, flag);
  return hipGetLastError();
}
hipError_t cp_cg_flags(int count, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(cg_flags_kernel, dim3(1), dim3(64), 0, s, count, flag);
  return hipGetLastError();
}
hipError_t cp_diag(int64_t n, const double* S, double* d, hipStream_t s) { CP_LAUNCH(diag_kernel, n, n, S, d); }

}  // namespace thc
