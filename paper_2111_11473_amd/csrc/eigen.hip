// Set-up linear algebra on the device: the 64 x 64 diagonal blocks of the Cholesky factorizations
// and the symmetric eigenproblem of the working basis.  The eigenproblem runs as
//   1. Householder reduction to a tridiagonal matrix, one launch per column (tridiag_step_kernel);
//   2. Q from compact WY blocks of 64 reflectors (products; their triangular factors here);
//   3. the implicit QL iteration on the tridiagonal, on the host (a serial chain of about
//      1.7 n^2 / 2 plane rotations; hostla.h), whose rotations stream to the device and are applied
//      to Q while the host goes on (rotate_kernel);
//   4. columns gathered in the order of their eigenvalues.
// n = 400: 7.6 ms (reduction 3.1, Q 1.3, rotations 3, of which 2.1 overlap the host's QL); on the host
// with threads it took 110 ms, of which most went to starting them twice a column.
#include "internal.h"

namespace thc {
namespace {

// Sum over the 64 lanes of a wavefront, in every lane.
__device__ inline double wave_sum(double x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// ---- Cholesky factor and inverse of one diagonal block (kb <= 64), or the inverse alone ----
// One workgroup: lane = column, each wavefront 16 rows, the block and its growing inverse in registers.
// The elimination runs without square roots (A = L' D L'^T; rows and columns are scaled at the end):
// a column step passes column k (by symmetry also row k) and row k of the inverse through LDS, two
// copies, one barrier a step.  What bounds it is the chain of 64 steps (barrier, LDS, reciprocal): 62 us
// a block, which stays on the device (through the host: four transfers a block, each waited for).
//   chol: A[0:kb, 0:kb] <- L, X <- L^-1 (kb x kb), status[0] = blk + 1 at the first pivot <= 0 (or
//         NaN) if no earlier block has set it.
//   else: X <- M^-1 for the lower triangular M with the elements of A below the diagonal and dval on it.
__global__ __launch_bounds__(256) void diag_block_kernel(int kb, double* A, int64_t lda, double* X, bool chol,
                                                         double dval, double* status, double blk) {
  __shared__ __align__(16) double col[2][64], xrow[2][64], diag[64];
  const int tx = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double a[16], x[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 16 * w + r;
    const bool in = i < kb && tx < kb;
    a[r] = in ? A[(int64_t)i * lda + tx] : (i == tx ? 1.0 : 0.0);
    x[r] = i == tx ? 1.0 : 0.0;
  }
  for (int k = 0; k < 64; ++k) {
    const int b = k & 1;
    if (tx == k) {
#pragma unroll
      for (int r = 0; r < 16; ++r) col[b][16 * w + r] = a[r];
    }
    if (w == k >> 4) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if ((k & 15) == r) xrow[b][tx] = x[r];
    }
    __syncthreads();
    double d = chol ? col[b][k] : (k < kb ? dval : 1.0);
    if (!(d > 0.0)) {
      if (threadIdx.x == 0 && status[0] == 0.0) status[0] = blk + 1.0;
      d = 1.0;
    }
    if (threadIdx.x == 0) diag[k] = d;
    if (16 * w + 15 <= k) continue;
    const double inv = 1.0 / d;
    const double xk = xrow[b][tx] * inv;
    const double lj = chol && tx > k ? col[b][tx] * inv : 0.0;
    // (rows up to k of the remainder change too, above the diagonal, where nothing is read)
    if (16 * w > k) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const double li = col[b][16 * w + r];
        a[r] -= li * lj;
        x[r] -= li * xk;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const double li = r > (k & 15) ? col[b][16 * w + r] : 0.0;
        a[r] -= li * lj;
        x[r] -= li * xk;
      }
    }
  }
  __syncthreads();
  const double cs = chol ? 1.0 / sqrt(diag[tx]) : 0.0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 16 * w + r;
    if (i >= kb || tx >= kb) continue;
    const double d = diag[i], sd = sqrt(d);
    if (chol) A[(int64_t)i * lda + tx] = tx < i ? a[r] * cs : (tx == i ? sd : 0.0);
    X[(int64_t)i * kb + tx] = tx <= i ? x[r] / (chol ? sd : d) : 0.0;
  }
}

// ---- out = (A + A^T) / 2 with 32 x 32 tiles ----
__global__ __launch_bounds__(256) void symmetrize_kernel(int64_t n, const double* A, double* out) {
  __shared__ double t[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t r0 = (int64_t)blockIdx.y * 32, c0 = (int64_t)blockIdx.x * 32;
  for (int r = ty; r < 32; r += 8)
    if (c0 + r < n && r0 + tx < n) t[r][tx] = A[(c0 + r) * n + r0 + tx];
  __syncthreads();
  for (int r = ty; r < 32; r += 8)
    if (r0 + r < n && c0 + tx < n) out[(r0 + r) * n + c0 + tx] = 0.5 * (A[(r0 + r) * n + c0 + tx] + t[tx][r]);
}

// ---- one column of the Householder reduction ----
// Launch k applies the rank-2 update of column k - 1 to rows and columns > k, forms the reflector of
// column k and p = 2 A v, in one pass over the trailing matrix.  What the update needs of its
// predecessor is v (row k - 1 of V), p, and the partial sums of v . p by row block (K = v . p,
// q = p - K v, A <- A - v q^T - q v^T).  Row k of the updated matrix (= column k) gives the reflector;
// every workgroup forms it for itself, so a column is one launch without a grid-wide wait.  Each
// workgroup owns TR rows; a thread takes columns k + 1 + t, + 256, ...
// What bounds it: the latency of the launch and its chain (partials -> row k -> norm -> rows), 7.8 us
// a column at n = 400; for n in the thousands, the one read and write of the trailing matrix.
constexpr int TR = 8;

__global__ __launch_bounds__(256) void tridiag_step_kernel(int64_t n, int64_t k, double* A, double* V, const double* p0,
                                                           const double* part0, int64_t npart0, double* p1,
                                                           double* part1, double* d, double* e) {
  __shared__ double red[4], acc_s[TR][256 + 8];
  const int t = threadIdx.x;
  const bool prev = k > 0;
  const double* vp = V + (k - 1) * n;  // read only if prev
  double K = 0.0, vk = 0.0, qk = 0.0;
  if (prev) {
    for (int64_t b = t & 63; b < npart0; b += 64) K += part0[b];
    K = wave_sum(K);
    vk = vp[k];
    qk = p0[k] - K * vk;
  }
  const double* Ak = A + k * n;
  auto updated = [&](int64_t j) {  // row k after the update
    double a = Ak[j];
    if (prev) {
      const double v = vp[j];
      a -= vk * (p0[j] - K * v) + qk * v;
    }
    return a;
  };
  const bool first = blockIdx.x == 0 && t == 0;
  if (k == n - 2) {  // the last 2 x 2 block: no reflector
    if (first) {
      d[k] = updated(k);
      e[k] = updated(k + 1);
      double a = A[(n - 1) * n + n - 1];
      if (prev) {
        const double v = vp[n - 1];
        a -= 2.0 * v * (p0[n - 1] - K * v);
      }
      d[n - 1] = a;
      e[n - 1] = 0.0;
    }
    return;
  }
  double sig = 0.0;
  for (int64_t j = k + 1 + t; j < n; j += 256) {
    const double x = updated(j);
    sig += x * x;
  }
  sig = wave_sum(sig);
  if ((t & 63) == 0) red[t >> 6] = sig;
  const double x0 = updated(k + 1);
  __syncthreads();
  const double xn = sqrt((red[0] + red[1]) + (red[2] + red[3]));
  const double alpha = x0 > 0.0 ? -xn : xn;
  // |x - alpha e_1| = sqrt(2 xn (xn + |x0|)); a zero column has v = 0 (the identity)
  const double inv = xn > 0.0 ? 1.0 / (sqrt(2.0 * xn) * sqrt(xn + fabs(x0))) : 0.0;
  if (first) {
    d[k] = updated(k);
    e[k] = xn > 0.0 ? alpha : 0.0;
  }
  // rows i0 .. i0 + TR - 1 of the trailing matrix
  const int64_t i0 = k + 1 + (int64_t)blockIdx.x * TR;
  double vi[TR], qi[TR], acc[TR];
#pragma unroll
  for (int r = 0; r < TR; ++r) {
    const int64_t i = min(i0 + r, n - 1);
    vi[r] = prev ? vp[i] : 0.0;
    qi[r] = prev ? p0[i] - K * vi[r] : 0.0;
    acc[r] = 0.0;
  }
  for (int64_t j = k + 1 + t; j < n; j += 256) {
    double vj = 0.0, qj = 0.0;
    if (prev) {
      vj = vp[j];
      qj = p0[j] - K * vj;
    }
    const double v = (Ak[j] - (prev ? vk * qj + qk * vj : 0.0) - (j == k + 1 ? alpha : 0.0)) * inv;
    if (blockIdx.x == 0) V[k * n + j] = v;
#pragma unroll
    for (int r = 0; r < TR; ++r) {
      if (i0 + r >= n) break;
      double* a = A + (i0 + r) * n + j;
      const double x = *a - (vi[r] * qj + qi[r] * vj);
      *a = x;
      acc[r] += x * v;
    }
  }
  if (blockIdx.x == 0)
    for (int64_t j = t; j <= k; j += 256) V[k * n + j] = 0.0;
#pragma unroll
  for (int r = 0; r < TR; ++r) acc_s[r][t] = acc[r];
  __syncthreads();
  const int r = t >> 5, u = t & 31;
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 8; ++c) s += acc_s[r][u + 32 * c];
  for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (u == 0) {
    const int64_t i = i0 + r;
    double vp1 = 0.0;
    if (i < n) {
      p1[i] = 2.0 * s;
      vp1 = (updated(i) - (i == k + 1 ? alpha : 0.0)) * inv * (2.0 * s);
    }
    acc_s[r][256] = vp1;
  }
  __syncthreads();
  if (t == 0) {
    double z = 0.0;
#pragma unroll
    for (int c = 0; c < TR; ++c) z += acc_s[c][256];
    part1[blockIdx.x] = z;
  }
}

// ---- plane rotations of the QL sweeps, applied to the rows of Z ----
// Z (n x n) holds Q^T; rotation (i, c, s) takes rows i, i + 1 to (c z_i - s z_i+1, s z_i + c z_i+1).
// Columns are independent: a lane keeps one.  Rotations come in groups of ROT_K sweeps that all run
// downwards; sweep s of a group acts on pair top - t + s in step t, right after sweep s - 1 has passed
// that pair, so a group reads and writes each element once and works on a window of ROT_K + 1 elements
// in registers (their names rotate: the steps are unrolled by ROT_K + 1).  A group's table is
// [step][sweep](c, s) with the identity where a sweep has no rotation; a step's 16 pairs are broadcast
// from LDS a step ahead.  Bound by the 64 FP64 instructions of a step (256 cycles): 67 us for a group of
// 16 sweeps at n = 400 (9.5 ns a rotation; 16 ns when each pair was read just before its use), against
// about 50 us that the host takes to make it.
constexpr int K = ROT_K, U = ROT_K + 1;

__global__ __launch_bounds__(64) void rotate_kernel(int n, double* Z, const double* table) {
  __shared__ double2 rot[(U + 1) * K];  // a tile's table and a step that is only read ahead
  const int lane = threadIdx.x;
  // lanes past the last column repeat it (the same values to the same places)
  double* Zc = Z + min((int)blockIdx.x * 64 + lane, n - 1);
  const int64_t* hdr = (const int64_t*)table;
  const int groups = (int)hdr[0], top = n - 2;
  for (int g = 0; g < groups; ++g) {
    const int bot = (int)hdr[1 + 3 * g], tiles = (int)hdr[2 + 3 * g];
    const double2* R = (const double2*)(table + hdr[3 + 3 * g]);
    // rows below the group's lowest are read (down to row 0) and meet the identity only; not stored
    double w[U], nx[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      w[u] = 0.0;
      nx[u] = Zc[(int64_t)max(top - u, 0) * n];
    }
    w[U - 1] = Zc[(int64_t)(top + 1) * n];
    double2 pre[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) pre[q] = R[min(q * 64 + lane, U * K - 1)];
    for (int tl = 0; tl < tiles; ++tl) {
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 5; ++q)
        if (q * 64 + lane < U * K) rot[q * 64 + lane] = pre[q];
      __syncthreads();
      const int64_t next = (int64_t)min(tl + 1, tiles - 1) * (U * K);
#pragma unroll
      for (int q = 0; q < 5; ++q) pre[q] = R[next + min(q * 64 + lane, U * K - 1)];
      const int t0 = top - tl * U;
      double2 q0[K], q1[K];
#pragma unroll
      for (int s = 0; s < K; ++s) q0[s] = rot[s];
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int s = 0; s < K; ++s) q1[s] = rot[(u + 1) * K + s];
        w[u] = nx[u];
        nx[u] = Zc[(int64_t)max(t0 - U - u, 0) * n];
#pragma unroll
        for (int s = 0; s < K; ++s) {
          const int i0 = (u - s + 2 * U) % U, i1 = (u - s - 1 + 2 * U) % U;
          const double a0 = w[i0], a1 = w[i1];
          w[i1] = __builtin_fma(q0[s].y, a0, q0[s].x * a1);  // a0 comes last: one FMA a rotation on the chain
          w[i0] = __builtin_fma(q0[s].x, a0, -(q0[s].y * a1));
        }
        const int el = t0 - u + K;
        if (el >= bot && el <= top + 1) Zc[(int64_t)el * n] = w[(u + 1) % U];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < K; ++s) q0[s] = q1[s];
      }
    }
  }
}

// ---- out[i][j] = Z[idx[j]][i] (idx held as doubles) with 32 x 32 tiles ----
__global__ __launch_bounds__(256) void gather_columns_kernel(int64_t n, const double* Z, const double* idx, double* out) {
  __shared__ double t[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t r0 = (int64_t)blockIdx.y * 32, c0 = (int64_t)blockIdx.x * 32;
  for (int r = ty; r < 32; r += 8)
    if (c0 + r < n && r0 + tx < n) t[r][tx] = Z[(int64_t)idx[c0 + r] * n + r0 + tx];
  __syncthreads();
  for (int r = ty; r < 32; r += 8)
    if (r0 + r < n && c0 + tx < n) out[(r0 + r) * n + c0 + tx] = t[tx][r];
}

}  // namespace

hipError_t eig_chol_block(int kb, double* A, int64_t lda, double* X, double* status, int64_t blk, hipStream_t s) {
  diag_block_kernel<<<1, 256, 0, s>>>(kb, A, lda, X, true, 0.0, status, (double)blk);
  return hipGetLastError();
}

hipError_t eig_tri_inverse(int kb, const double* M, double dval, double* X, hipStream_t s) {
  diag_block_kernel<<<1, 256, 0, s>>>(kb, const_cast<double*>(M), kb, X, false, dval, nullptr, 0.0);
  return hipGetLastError();
}

hipError_t eig_symmetrize(int64_t n, const double* A, double* out, hipStream_t s) {
  const unsigned t = (unsigned)((n + 31) / 32);
  symmetrize_kernel<<<dim3(t, t), 256, 0, s>>>(n, A, out);
  return hipGetLastError();
}

int64_t eig_tridiag_scratch(int64_t n) { return 2 * n + 2 * ((n + TR - 1) / TR); }

hipError_t eig_tridiag(int64_t n, double* A, double* V, double* d, double* e, double* scratch, hipStream_t s) {
  const int64_t np = (n + TR - 1) / TR;
  double* p[2] = {scratch, scratch + n};
  double* part[2] = {scratch + 2 * n, scratch + 2 * n + np};
  int64_t blocks0 = 0;
  for (int64_t k = 0; k + 1 < n; ++k) {
    const int64_t blocks = k == n - 2 ? 1 : (n - k - 1 + TR - 1) / TR;
    tridiag_step_kernel<<<(unsigned)blocks, 256, 0, s>>>(n, k, A, V, p[(k + 1) & 1], part[(k + 1) & 1], blocks0,
                                                         p[k & 1], part[k & 1], d, e);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    blocks0 = blocks;
  }
  return hipSuccess;
}

hipError_t eig_rotate(int64_t n, double* Z, const double* table, hipStream_t s) {
  rotate_kernel<<<(unsigned)((n + 63) / 64), 64, 0, s>>>((int)n, Z, table);
  return hipGetLastError();
}

hipError_t eig_gather_columns(int64_t n, const double* Z, const double* idx, double* out, hipStream_t s) {
  const unsigned t = (unsigned)((n + 31) / 32);
  gather_columns_kernel<<<dim3(t, t), 256, 0, s>>>(n, Z, idx, out);
  return hipGetLastError();
}

}  // namespace thc
