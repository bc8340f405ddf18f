// The three-way product of the quartic T2^2 algorithm (paper Alg. 6):
//   H^XYZ += sum_I ( E_I^XY F_I^XZ + E_I^XZ F_I^XY ) G_I^YZ
// Each factor carries two of the three output indices, so this is not a matrix product over I.
//
// Symmetry.  The bracket t_I(X; Y, Z) = E^XY F^XZ + E^XZ F^XY is symmetric in Y <-> Z, so for
// Y != Z one t serves both H^XYZ (times G^YZ) and H^XZY (times G^ZY).
//
// Where (Y, Z) sit.  A wave's 64 lanes hold a 16 x 16 block of (Y, Z), four Y and one Z a lane, and its X are
// in registers: G^YZ is an ordinary register that serves every X.
// FP64 (vector ALU; it shares its throughput with the FP64 matrix instructions, and forming the bracket
// with v_mfma_f64_16x16x4f64, two of its four k padding, took 1.06 us a point and generation): E^Z and F^Z
// are the lane's own, E^Y and F^Y are broadcast by DPP over the 16 lanes that share them, sixteen values to a
// register pair.  At P = 1000: 0.95 us a grid point and generation of 512 tiles (the copies alone 0.76, the
// arithmetic alone 0.79) against 0.97-0.99 with lanes over X and G broadcast, which copied 26 KB a stage
// three deep instead of 20 KB four deep.
// FP32 (mixed precision): at fixed X and I the bracket is a product of rank 2 over (Y, Z);
// v_mfma_f32_16x16x1f32 forms it for four X at a time, so two of them replace the 32 vector instructions
// of 1024 brackets, and a wave reads 24 values a lane per 4096 brackets instead of the 96 of a 4 x 4 x 4 patch
// per lane.  At P = 800: 1.08 -> 0.89 us a grid point and generation (copies alone 0.66, arithmetic alone
// 0.67).
// Both are bound by the copies -- E and F rows and G blocks from beyond the L2: with every point in the L2 the
// copies take 0.37 us -- and by the arithmetic at a clock of 2.0-2.1 GHz (2.35 without the copies).
//
// Work decomposition.  A workgroup of four waves owns one 16 x 16 block pair (Yb <= Zb) and a slice of
// X: 32 X in FP64, 64 in FP32.  A wave owns a quarter of them (8 or 16) and the whole block pair: lane
// l holds Z = l % 16 and Y = 4 (l / 16) + r; 32 accumulators and as many mirror accumulators in FP64, 64 and 64 in
// FP32.  For Yb < Zb it accumulates both H^XYZ and its mirror H^XZY; a diagonal
// block (Yb == Zb) covers every ordered pair inside itself directly and keeps no mirror.
//
// Operand staging.  Per I the workgroup's rows -- E^XY, F^XY for its 16 Y, E^XZ, F^XZ for its 16 Z, 256
// bytes of X each -- and its two G blocks are copied by buffer loads straight into LDS, NS stages deep
// (NS - 1 values of I in flight), and each wave waits only for its own copies of the next stage before
// the barrier.  The 16-byte granule g of row r lands at g ^ r, so sixteen lanes that read the same
// granule of sixteen rows touch every bank once; the G blocks land in the order in which the lanes read
// them.
// Tile order comes from a host-built table: runs of `slots` tiles (the workgroups resident on one
// XCD) that share an X tile and a compact patch of (Y, Z) blocks are placed at workgroup ids b with
// b % 8 = that XCD, so tiles sharing operand rows run on one XCD at about the same time and share
// them through its L2.  The table is launched one generation (8 runs, every slot of the device)
// at a time, so the workgroups of a run start together and cannot drift apart by more than one
// tile's lifetime; consecutive generations walk the grid points in opposite directions, so a
// generation starts on the points its predecessor read last (still in the last-level cache).
// One workgroup per tile measured faster than a persistent grid walking the table.
// Layouts (Y, Z ranks zero-padded to Pp, a multiple of 16; X restricted to a block of Xb ranks, a
// multiple of 64 and at most Pp rounded up to 64):
//   E, F: [Xb/64][ldi][Pp][64] (E_I^XY at [X/64][I][Y][X%64]);
//   G: [I][Pp/16][Pp/16][16][16] (G_I^YZ at [I][Y/16][Z/16][Y%16][Z%16]);
//   H: [Pp][Pp][Xb] (H^XYZ at [Y][Z][X]), FP64 always.
#include <algorithm>
#include <utility>
#include <vector>

#include "internal.h"

namespace thc {
namespace {

constexpr int XT = 64;                     // X per tile of E, F
constexpr int BY = 16;                     // Y (and Z) block edge
constexpr int RSRC_W3 = 0x00020000;        // raw 32-bit buffer access
constexpr uint32_t EMPTY = 0x80000000u;

typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16 __attribute__((ext_vector_type(16)));

// A stage (bytes): E^Y and F^Y (16 rows of 256 bytes each) and G^YZ, then F^Z, E^Z and G^ZY.
template <typename T>
struct Geo {
  static constexpr bool F64 = sizeof(T) == 8;
  static constexpr int ROW_B = 256;                     // bytes of X per row and workgroup
  static constexpr int XW = ROW_B / (int)sizeof(T);     // X per workgroup: 32 or 64
  static constexpr int NZS = XT / XW;                   // workgroups per X tile
  static constexpr int REG_B = BY * ROW_B;              // one operand's rows
  static constexpr int G_B = BY * BY * (int)sizeof(T);  // one G block
  static constexpr int G = 2 * REG_B, HALF = G + G_B;
  static constexpr int STAGE_B = 2 * HALF;
  static constexpr int NS = 4;                          // two workgroups per CU either way
  static constexpr int GW = G_B / 1024;                 // waves that copy one G block
  static_assert(2 * NS * STAGE_B <= 160 * 1024, "two workgroups per CU");
};

__device__ inline __amdgpu_buffer_rsrc_t rsrc(const void* base, int64_t nbytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)(uint32_t)nbytes, RSRC_W3);
}
// 16 bytes per lane from a buffer straight into LDS at lds + 16 * lane (no VGPR destination)
__device__ inline void bload_lds(__amdgpu_buffer_rsrc_t r, void* lds, unsigned voff, unsigned soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voff, soff, 0, 0);
}

// Waits until at most n of this wave's vector-memory operations are outstanding (n is
// wave-uniform) and its LDS operations are complete, then joins the workgroup barrier.  Written
// as one block so that neither the wait nor the barrier picks up the compiler's conservative
// vmcnt(0).
template <int N>
__device__ inline void wait_bar() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
// Wait for stage I + 1 with `later` further stages (0 <= later < 3) of Q or Q + 1 copies each
// (extra: this wave also copies a G chunk) still allowed in flight, then the barrier.
template <int Q>
__device__ inline void wait_pipe(int later, bool extra) {
  if (later >= 2) {
    if (extra) wait_bar<2 * (Q + 1)>(); else wait_bar<2 * Q>();
  } else if (later == 1) {
    if (extra) wait_bar<Q + 1>(); else wait_bar<Q>();
  } else {
    wait_bar<0>();
  }
}

// Accumulators of a wave and the work of one grid point.
template <typename T>
struct Patch;

// The FP64 patch, one X ahead: u_r = E^Y_r fz + F^Y_r ez of the next X for the lane's four Y, E^Y and F^Y
// broadcast from lane B + r of the lane's row of 16 (DPP), between the products of the present X,
// acc_r += G^YZ t_r and accm_r += G^ZY t_r, so that nothing waits for the instruction before it.  Only
// v_fmac_f64 takes a 64-bit DPP source, so u starts from a moved zero; the four moves also keep the DPP reads
// the required two wait states behind any write of their source (inline assembly is invisible to the
// hazard pass).
#define H_ZERO \
  "v_mov_b64 %[u0], 0\n\t"  \
  "v_mov_b64 %[u1], 0\n\t"  \
  "v_mov_b64 %[u2], 0\n\t"  \
  "v_mov_b64 %[u3], 0\n\t"
#define H_BRACKET(y, z)                                              \
  "v_fmac_f64_dpp %[u0], %[" y "], %[" z "] row_newbcast:%[b0]\n\t" \
  "v_fmac_f64_dpp %[u1], %[" y "], %[" z "] row_newbcast:%[b1]\n\t" \
  "v_fmac_f64_dpp %[u2], %[" y "], %[" z "] row_newbcast:%[b2]\n\t" \
  "v_fmac_f64_dpp %[u3], %[" y "], %[" z "] row_newbcast:%[b3]\n\t"
#define H_USE(a, g)                   \
  "v_fmac_f64 %[" a "0], %[" g "0], %[t0]\n\t" \
  "v_fmac_f64 %[" a "1], %[" g "1], %[t1]\n\t" \
  "v_fmac_f64 %[" a "2], %[" g "2], %[t2]\n\t" \
  "v_fmac_f64 %[" a "3], %[" g "3], %[t3]\n\t"
template <int B>
__device__ inline void h_bracket(double (&u)[4], double ey, double fy, double ez, double fz) {
  asm volatile(H_ZERO H_BRACKET("ey", "fz") H_BRACKET("fy", "ez")
               : [u0] "=&v"(u[0]), [u1] "=&v"(u[1]), [u2] "=&v"(u[2]), [u3] "=&v"(u[3])
               : [ey] "v"(ey), [fy] "v"(fy), [ez] "v"(ez), [fz] "v"(fz), [b0] "n"(B), [b1] "n"(B + 1),
                 [b2] "n"(B + 2), [b3] "n"(B + 3));
}
__device__ inline void h_use(double (&acc)[4], double (&accm)[4], const double (&t)[4], const double (&g)[4],
                             const double (&gm)[4]) {
  asm volatile(H_USE("a", "g") H_USE("m", "h")
               : [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3]), [m0] "+v"(accm[0]),
                 [m1] "+v"(accm[1]), [m2] "+v"(accm[2]), [m3] "+v"(accm[3])
               : [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]), [g0] "v"(g[0]), [g1] "v"(g[1]),
                 [g2] "v"(g[2]), [g3] "v"(g[3]), [h0] "v"(gm[0]), [h1] "v"(gm[1]), [h2] "v"(gm[2]), [h3] "v"(gm[3]));
}
template <int B>
__device__ inline void h_step(double (&u)[4], double ey, double fy, double ez, double fz, double (&acc)[4],
                              double (&accm)[4], const double (&t)[4], const double (&g)[4], const double (&gm)[4]) {
  asm volatile(H_ZERO H_BRACKET("ey", "fz") H_USE("a", "g") H_BRACKET("fy", "ez") H_USE("m", "h")
               : [u0] "=&v"(u[0]), [u1] "=&v"(u[1]), [u2] "=&v"(u[2]), [u3] "=&v"(u[3]), [a0] "+v"(acc[0]),
                 [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3]), [m0] "+v"(accm[0]), [m1] "+v"(accm[1]),
                 [m2] "+v"(accm[2]), [m3] "+v"(accm[3])
               : [ey] "v"(ey), [fy] "v"(fy), [ez] "v"(ez), [fz] "v"(fz), [t0] "v"(t[0]), [t1] "v"(t[1]),
                 [t2] "v"(t[2]), [t3] "v"(t[3]), [g0] "v"(g[0]), [g1] "v"(g[1]), [g2] "v"(g[2]), [g3] "v"(g[3]),
                 [h0] "v"(gm[0]), [h1] "v"(gm[1]), [h2] "v"(gm[2]), [h3] "v"(gm[3]), [b0] "n"(B), [b1] "n"(B + 1),
                 [b2] "n"(B + 2), [b3] "n"(B + 3));
}
#undef H_ZERO
#undef H_BRACKET
#undef H_USE

template <>
struct Patch<double> {
  double acc[8][4], accm[8][4];  // [x][r]: X = 8 w + x of the slice
  __device__ static int x_of(int w) { return 8 * w; }
  // LDS byte offsets within a stage: the lane's broadcast source (lane m of a row of 16 holds Y r = m % 4 at X
  // m / 4 of each four), its Z row's granules, the G blocks
  unsigned ay[2], az[4], g, gt;
  __device__ void offsets(int lane, int w) {
    const int m = lane & 15, q = lane >> 4, y = 4 * q + (m & 3);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      ay[h] = (unsigned)(y * 256 + ((4 * w + 2 * h + (m >> 3)) ^ y) * 16 + ((m >> 2) & 1) * 8);
#pragma unroll
    for (int i = 0; i < 4; ++i) az[i] = (unsigned)(Geo<double>::HALF + m * 256 + ((4 * w + i) ^ m) * 16);
    g = (unsigned)(Geo<double>::G + q * 512 + m * 8);                          // [Y][Z]
    gt = (unsigned)(Geo<double>::HALF + Geo<double>::G + q * 256 + m * 16);    // see gt_source
  }
  // Source granule (16 bytes, of the row-major 16 x 16 block) of LDS granule s of each G block; G^ZY lands
  // as [Y / 2 % 2][Y / 4][Z] so that a lane's two pairs of Y are 16 lanes' consecutive granules.
  __device__ static int g_source(int s) { return s; }
  __device__ static int gt_source(int s) { return (s % 16) * 8 + 2 * (s / 16 % 4) + s / 64; }
  __device__ void point(const char* st) {
    constexpr int REG = Geo<double>::REG_B;
    double ey[2], fy[2], gv[4], gm[4];
    d2 fz[4], ez[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      ey[h] = *(const double*)(st + ay[h]);
      fy[h] = *(const double*)(st + ay[h] + REG);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) gv[r] = *(const double*)(st + g + 128 * r);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const d2 v = *(const d2*)(st + gt + 1024 * h);
      gm[2 * h] = v.x;
      gm[2 * h + 1] = v.y;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fz[i] = *(const d2*)(st + az[i]);
      ez[i] = *(const d2*)(st + az[i] + REG);
    }
    __builtin_amdgcn_sched_barrier(0);
    double t[2][4];
    h_bracket<0>(t[0], ey[0], fy[0], ez[0].x, fz[0].x);
    h_step<4>(t[1], ey[0], fy[0], ez[0].y, fz[0].y, acc[0], accm[0], t[0], gv, gm);
    h_step<8>(t[0], ey[0], fy[0], ez[1].x, fz[1].x, acc[1], accm[1], t[1], gv, gm);
    h_step<12>(t[1], ey[0], fy[0], ez[1].y, fz[1].y, acc[2], accm[2], t[0], gv, gm);
    h_step<0>(t[0], ey[1], fy[1], ez[2].x, fz[2].x, acc[3], accm[3], t[1], gv, gm);
    h_step<4>(t[1], ey[1], fy[1], ez[2].y, fz[2].y, acc[4], accm[4], t[0], gv, gm);
    h_step<8>(t[0], ey[1], fy[1], ez[3].x, fz[3].x, acc[5], accm[5], t[1], gv, gm);
    h_step<12>(t[1], ey[1], fy[1], ez[3].y, fz[3].y, acc[6], accm[6], t[0], gv, gm);
    h_use(acc[7], accm[7], t[1], gv, gm);
  }
  __device__ d2 pair(bool m, int h, int r) const {  // X = x_of(w) + 2 h, + 1
    return m ? d2{accm[2 * h][r], accm[2 * h + 1][r]} : d2{acc[2 * h][r], acc[2 * h + 1][r]};
  }
  __device__ void set_pair(bool m, int h, int r, d2 v) {
    if (m) { accm[2 * h][r] = v.x; accm[2 * h + 1][r] = v.y; }
    else { acc[2 * h][r] = v.x; acc[2 * h + 1][r] = v.y; }
  }
  __device__ void clear() {
#pragma unroll
    for (int x = 0; x < 8; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[x][r] = accm[x][r] = 0.0;
  }
  static constexpr int NPAIR = 4;
};

template <>
struct Patch<float> {
  float acc[4][4][4], accm[4][4][4];  // [j][b][r]: X = 16 w + 4 b + j (b: the instruction's block)
  __device__ static int x_of(int w) { return 16 * w; }
  unsigned a, g, gt;
  __device__ void offsets(int lane, int w) {
    const int row = lane & 15, k = lane >> 4;  // k: the instruction's block of four X
    a = (unsigned)(row * 256 + ((4 * w + k) ^ row) * 16);
    g = (unsigned)(Geo<float>::G + lane * 4);                                   // [r][Y / 4][Z]: see g_source
    gt = (unsigned)(Geo<float>::HALF + Geo<float>::G + row * 64 + k * 16);      // [Z][Y]: four Y
  }
  __device__ static int g_source(int s) { return (4 * (s / 4 % 4) + s / 16) * 4 + s % 4; }
  __device__ static int gt_source(int s) { return s; }
  __device__ void point(const char* st) {
    using C = Geo<float>;
    const f4 ey = *(const f4*)(st + a), fy = *(const f4*)(st + a + C::REG_B);
    const f4 fz = *(const f4*)(st + a + C::HALF), ez = *(const f4*)(st + a + C::HALF + C::REG_B);
    const f4 gm = *(const f4*)(st + gt);
    float gv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) gv[r] = *(const float*)(st + g + 256 * r);
    const f16 z = {0.0f};
    f16 t[2];
    auto bracket = [&](int j) {
      float e = ey[j];
      asm volatile("" : "+v"(e));
      const f16 u = __builtin_amdgcn_mfma_f32_16x16x1f32(e, fz[j], z, 0, 0, 0);
      return __builtin_amdgcn_mfma_f32_16x16x1f32(fy[j], ez[j], u, 0, 0, 0);
    };
    __builtin_amdgcn_sched_barrier(0);
    t[0] = bracket(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j < 3) {
        t[(j + 1) & 1] = bracket(j + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[j][b][r] = __builtin_fmaf(gv[r], t[j & 1][4 * b + r], acc[j][b][r]);
          accm[j][b][r] = __builtin_fmaf(gm[r], t[j & 1][4 * b + r], accm[j][b][r]);
        }
#pragma unroll
      for (int b = 0; b < 4; ++b)
        asm volatile("" : "+v"(acc[j][b][0]), "+v"(acc[j][b][1]), "+v"(acc[j][b][2]), "+v"(acc[j][b][3]),
                          "+v"(accm[j][b][0]), "+v"(accm[j][b][1]), "+v"(accm[j][b][2]), "+v"(accm[j][b][3]));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __device__ d2 pair(bool m, int h, int r) const {
    const int b = h / 2, j = 2 * (h & 1);
    return m ? d2{(double)accm[j][b][r], (double)accm[j + 1][b][r]} : d2{(double)acc[j][b][r], (double)acc[j + 1][b][r]};
  }
  __device__ void clear() {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[j][b][r] = accm[j][b][r] = 0.0f;
  }
  static constexpr int NPAIR = 8;
};

template <typename T>
__global__ __launch_bounds__(256, 2) void h_kernel(int Pp, int Xb, int64_t ldi, int64_t nIall, const T* __restrict__ E,
                                                   const T* __restrict__ F, const T* __restrict__ G,
                                                   double* __restrict__ H, const uint32_t* __restrict__ tiles,
                                                   int flags) {
  using C = Geo<T>;
  __shared__ __attribute__((aligned(16))) char lds[C::NS * C::STAGE_B];
  const uint32_t tile = tiles[blockIdx.x];
  if (tile & EMPTY) return;  // whole workgroup, before any barrier
  const bool rev = flags & 1;    // walk the grid points backwards
  const bool fresh = flags & 2;  // first chunk: H starts from zero instead of being read
  const int Yb = tile & 511, Zb = (tile >> 9) & 511, zs = (tile >> 18) & 3, xt = (tile >> 20) & 1023;
  const bool mirror = Yb != Zb;
  const int y0 = Yb * BY, z0 = Zb * BY;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __builtin_assume(w >= 0 && w < 4);

  // A diagonal block has no mirror: its G^ZY slots stay zero (the copies never write them).
  for (int b = 0; b < C::NS; ++b) {
    char* sb = lds + b * C::STAGE_B;
    if (!mirror)
      for (int i = threadIdx.x; i < BY * BY; i += 256) ((T*)(sb + C::HALF + C::G))[i] = (T)0;
  }

  Patch<T> p;
  p.offsets(lane, w);
  // this slice's grid points and its H (gridDim.y slices)
  const int64_t I0 = nIall * blockIdx.y / gridDim.y, nI = nIall * (blockIdx.y + 1) / gridDim.y - I0;
  H += (int64_t)blockIdx.y * Pp * Pp * Xb;
  // lane's element (Y, Z, X) of H and of its mirror
  const int Z = z0 + (lane & 15), X0 = xt * XT + zs * C::XW + Patch<T>::x_of(w);
  auto at = [&](bool m, int r) {
    const int64_t Y = y0 + 4 * (lane >> 4) + r;
    return H + (m ? (int64_t)Z * Pp + Y : Y * Pp + Z) * Xb + X0;
  };
  bool loaded = false;
  if constexpr (C::F64) {
    if (!fresh) {
      loaded = true;
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int h = 0; h < Patch<T>::NPAIR; ++h)
            p.set_pair(m, h, r, m == 0 || mirror ? *(const d2*)(at(m, r) + 2 * h) : d2{0.0, 0.0});
    }
  }
  if (!loaded) {
    p.clear();
  }

  // Copies of one stage: wave w takes rows 4 w .. 4 w + 3 of each of the four operands (1 KB each), and a
  // 1 KB chunk of a G block: waves 0 .. GW - 1 of G^YZ, the next GW (off the diagonal) of G^ZY.
  const int crow = 4 * w + (lane >> 4);
  const unsigned voff_r = (unsigned)crow * (XT * (int)sizeof(T)) + (unsigned)((lane & 15) ^ crow) * 16u;
  const bool g_yz = w < C::GW, g_zy = !g_yz && w < 2 * C::GW && mirror;
  const bool extra = g_yz || g_zy;
  const int gs = (g_yz ? w : w - C::GW) * 64 + lane;
  const unsigned nb16 = (unsigned)Pp / 16u;
  const unsigned voff_g = (unsigned)(g_yz ? Patch<T>::g_source(gs) : Patch<T>::gt_source(gs)) * 16u;
  const unsigned so_g = (g_zy ? (unsigned)Zb * nb16 + (unsigned)Yb : (unsigned)Yb * nb16 + (unsigned)Zb) * (unsigned)C::G_B;
  const unsigned lds_g = (unsigned)(g_yz ? C::G + w * 1024 : C::HALF + C::G + (w - C::GW) * 1024);
  const unsigned so_y = (unsigned)y0 * (XT * (int)sizeof(T)) + (unsigned)zs * C::ROW_B;
  const unsigned so_z = (unsigned)z0 * (XT * (int)sizeof(T)) + (unsigned)zs * C::ROW_B;
  const int64_t PX = (int64_t)Pp * XT;  // elements of E, F per (X tile, I)
  const int64_t PP = (int64_t)Pp * Pp;  // elements of G per I
  // Sources of the next stage to copy: a generation walks the grid points forwards or (rev)
  // backwards, so each stage moves the three pointers by one grid point.
  const int64_t first = I0 + ((rev && nI > 0) ? nI - 1 : 0);
  const T* e_at = E + ((int64_t)xt * ldi + first) * PX;
  const T* f_at = F + ((int64_t)xt * ldi + first) * PX;
  const T* g_at = G + first * PP;
  const int64_t dPX = rev ? -PX : PX, dPP = rev ? -PP : PP;
  auto stage_in = [&](int buf) {
    const __amdgpu_buffer_rsrc_t re = rsrc(e_at, PX * (int)sizeof(T));
    const __amdgpu_buffer_rsrc_t rf = rsrc(f_at, PX * (int)sizeof(T));
    char* sb = lds + buf * C::STAGE_B + w * 1024;
    bload_lds(re, sb, voff_r, so_y);
    bload_lds(rf, sb + C::REG_B, voff_r, so_y);
    bload_lds(rf, sb + C::HALF, voff_r, so_z);
    bload_lds(re, sb + C::HALF + C::REG_B, voff_r, so_z);
    if (extra) bload_lds(rsrc(g_at, PP * (int)sizeof(T)), lds + buf * C::STAGE_B + lds_g, voff_g, so_g);
    e_at += dPX;
    f_at += dPX;
    g_at += dPP;
  };

  constexpr int NS = C::NS, D = NS - 1;  // stages in flight ahead of the one being consumed
  static_assert(D <= 3, "wait_pipe allows at most two stages in flight behind the next one");
  auto next = [](int b) { return b + 1 == NS ? 0 : b + 1; };
  int64_t issued = 0;
  int sbuf = 0;  // buffer of the next stage to copy: (buf + D) % NS once the pipe is full
  for (; issued < D && issued < nI; ++issued) {
    stage_in(sbuf);
    sbuf = next(sbuf);
  }
  wait_pipe<4>((int)(issued > 0 ? issued - 1 : 0), extra);  // stage 0 has landed everywhere
  auto consume = [&](int buf) {
    __builtin_amdgcn_sched_barrier(0);
    p.point(lds + buf * C::STAGE_B);
    __builtin_amdgcn_sched_barrier(0);
  };
  // The two workgroups of a CU (ids 256 apart, one round of the device's CUs) take the higher wave priority in
  // turn, two grid points each.  Left at equal priority the older one always wins: it ran a 300-point tile in
  // 193 us and the other, alone at the end with one wave per SIMD, in 287 us; in turn both take 255 us.
  const int odd_round = ((blockIdx.x + gridDim.x * blockIdx.y) >> 8) & 1;
  // Steady state: every grid point also issues the stage D ahead, and the stage after the next
  // one (D - 1 of them) may stay in flight.  NS points a turn, so that buffers are constants.
  const int64_t steady = nI - D;
  int64_t I = 0;
  for (; I + NS <= steady; I += NS)
#pragma unroll
    for (int b = 0; b < NS; ++b) {
      if (((b >> 1) ^ odd_round) & 1) __builtin_amdgcn_s_setprio(2);
      else __builtin_amdgcn_s_setprio(1);
      stage_in((b + D) % NS);
      consume(b);
      wait_pipe<4>(D - 1, extra);
    }
  // The rest: fewer than NS points that still copy, then those of the stages in flight.
  int buf = 0;
  for (; I < nI; ++I) {
    if (I < steady) {
      stage_in(sbuf);
      sbuf = next(sbuf);
    }
    consume(buf);
    const int64_t later = I < steady ? D - 1 : nI - I - 2;
    wait_pipe<4>((int)(later > 0 ? later : 0), extra);
    buf = next(buf);
  }

#pragma unroll
  for (int m = 0; m < 2; ++m) {
    if (m == 1 && !mirror) break;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < Patch<T>::NPAIR; ++h) {
        d2* q = (d2*)(at(m, r) + 2 * h);
        const d2 v = p.pair(m, h, r);
        if constexpr (C::F64) *q = v;             // already continues H
        else *q = fresh ? v : *q + v;
      }
  }
}

// Position of cell (y, z) along the Hilbert curve that fills an n x n grid (n a power of two).
int64_t hilbert_index(int64_t n, int64_t y, int64_t z) {
  int64_t d = 0;
  for (int64_t s = n / 2; s > 0; s /= 2) {
    const int64_t ry = (y & s) ? 1 : 0, rz = (z & s) ? 1 : 0;
    d += s * s * ((3 * ry) ^ rz);
    if (rz == 0) {  // rotate the quadrant so the curve enters and leaves it at the right corners
      if (ry == 1) {
        y = n - 1 - y;
        z = n - 1 - z;
      }
      std::swap(y, z);
    }
  }
  return d;
}

template <int NZS>
std::vector<uint32_t> tiles_for(int64_t Pp, int64_t Xb, int64_t slots) {
  const int64_t nB = Pp / BY, nX = Xb / XT;
  // Block pairs (Yb <= Zb) in Hilbert-curve order: any run of consecutive pairs covers a compact
  // patch of the (Y, Z) triangle, so the runs that share an XCD's L2 touch few distinct operand
  // rows and G blocks (about 20% fewer bytes per grid point than row-major groups of 4 x 8 blocks,
  // whose runs straddle two groups once the diagonal groups put them out of step).
  int64_t n = 1;
  while (n < nB) n *= 2;
  std::vector<std::pair<int64_t, uint32_t>> pairs;
  pairs.reserve((size_t)(nB * (nB + 1) / 2));
  for (int64_t yb = 0; yb < nB; ++yb)
    for (int64_t zb = yb; zb < nB; ++zb) pairs.push_back({hilbert_index(n, yb, zb), (uint32_t)(yb | (zb << 9))});
  std::sort(pairs.begin(), pairs.end());
  std::vector<uint32_t> lin;
  lin.reserve(pairs.size() * NZS * (size_t)nX);
  for (int64_t xt = 0; xt < nX; ++xt)
    for (const auto& p : pairs)
      for (int64_t s = 0; s < NZS; ++s) lin.push_back(p.second | (uint32_t)(s << 18) | (uint32_t)(xt << 20));
  const int64_t runs = ((int64_t)lin.size() + slots - 1) / slots;
  std::vector<uint32_t> out((size_t)(((runs + 7) / 8) * 8 * slots), EMPTY);
  for (size_t e = 0; e < lin.size(); ++e) {
    const int64_t c = (int64_t)e / slots, k = (int64_t)e % slots;
    out[(size_t)((c / 8) * 8 * slots + k * 8 + c % 8)] = lin[e];
  }
  return out;
}

template <typename T>
hipError_t launch(int64_t Pp, int64_t Xb, int64_t ldi, int64_t nI, const T* E, const T* F, const T* G, double* H,
                  const uint32_t* tiles, int64_t ntiles, int64_t slots, int slices, bool fresh, hipStream_t s) {
  if (Pp % BY != 0 || Pp <= 0 || Pp > 8192 || Xb % XT != 0 || Xb > (Pp + XT - 1) / XT * XT || Xb <= 0 || ntiles <= 0 || ntiles > 2147483647LL ||
      nI < 0 || ldi < nI || slots < 1 || ntiles % (8 * slots) != 0 || slices < 1 || slices > H_SLICES)
    return hipErrorInvalidValue;
  // One launch per generation of 8 slots tiles (every workgroup resident at once): the runs of
  // a generation start together, so the workgroups sharing operand rows through an L2 stay
  // within one tile's lifetime of each other.
  const int64_t gen = 8 * slots;
  for (int64_t t0 = 0; t0 < ntiles; t0 += gen) {
    hipLaunchKernelGGL(h_kernel<T>, dim3((unsigned)gen, (unsigned)slices), dim3(256), 0, s, (int)Pp, (int)Xb, ldi, nI, E, F, G, H,
                       tiles + t0, (int)((t0 / gen) & 1) | (fresh ? 2 : 0));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Resident workgroups per XCD (8 XCDs; workgroup b runs on XCD b % 8): CUs per XCD times the
// workgroups that fit on one CU.
template <typename T>
int64_t slots_per_xcd() {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, h_kernel<T>, 256, 0) != hipSuccess)
    return 0;
  return std::max<int64_t>(1, (int64_t)(cus / 8) * std::max(per_cu, 1));
}

int64_t h_run(int64_t Pp, int64_t Xb, int64_t slots, int nzs) {
  const int64_t nB = Pp / BY, tiles = nB * (nB + 1) / 2 * nzs * (Xb / XT);
  return std::min(slots, std::max<int64_t>(1, (tiles + 7) / 8));
}

}  // namespace

int64_t h_slots_per_xcd() { return slots_per_xcd<double>(); }

int64_t h_run_length(int64_t Pp, int64_t Xb, int64_t slots) { return h_run(Pp, Xb, slots, Geo<double>::NZS); }
int64_t h32_run_length(int64_t Pp, int64_t Xb, int64_t slots) { return h_run(Pp, Xb, slots, Geo<float>::NZS); }

// Slices of the grid points, each with its own H, that fill the device's 8 slots tiles where the ranks have
// too few (the caller adds the slices up): one workgroup's walk over the points is a serial chain.  At least 16
// points each.  With even runs (h_run_length), a solve at P = 120 (144 tiles, 300 points): 8.7 -> 7.9 ms, a residual
// at P = 50 (20 tiles, 110 points): 0.755 -> 0.717.
int h_slices(int64_t Pp, int64_t Xb, int64_t nI, int64_t slots) {
  const int64_t nB = Pp / BY, tiles = nB * (nB + 1) / 2 * Geo<double>::NZS * (Xb / XT);
  return (int)std::max<int64_t>(1, std::min<int64_t>({8 * slots / tiles, nI / 16, H_SLICES}));
}

// Tile table: every (X tile, Y block Yb, Z block Zb >= Yb, slice of X) once, in runs of `slots`
// tiles that share an X tile and a Hilbert-curve patch of block pairs; run c sits at workgroup ids
// b = 8 slots (c / 8) + 8 k + (c % 8), k < slots, so that it runs on one XCD.  Unused entries are
// EMPTY.
std::vector<uint32_t> h_tiles(int64_t Pp, int64_t Xb, int64_t slots) { return tiles_for<Geo<double>::NZS>(Pp, Xb, slots); }

hipError_t h_accumulate(int64_t Pp, int64_t Xb, int64_t ldi, int64_t nI, const double* E, const double* F,
                        const double* G, double* H, const uint32_t* tiles, int64_t ntiles, int64_t slots, int slices,
                        bool fresh, hipStream_t s) {
  return launch<double>(Pp, Xb, ldi, nI, E, F, G, H, tiles, ntiles, slots, slices, fresh, s);
}

int64_t h32_slots_per_xcd() { return slots_per_xcd<float>(); }

std::vector<uint32_t> h32_tiles(int64_t Pp, int64_t Xb, int64_t slots) { return tiles_for<Geo<float>::NZS>(Pp, Xb, slots); }

hipError_t h_accumulate_f32(int64_t Pp, int64_t Xb, int64_t ldi, int64_t nI, const float* E, const float* F,
                            const float* G, double* H, const uint32_t* tiles, int64_t ntiles, int64_t slots,
                            bool fresh, hipStream_t s) {
  return launch<float>(Pp, Xb, ldi, nI, E, F, G, H, tiles, ntiles, slots, 1, fresh, s);
}

}  // namespace thc
