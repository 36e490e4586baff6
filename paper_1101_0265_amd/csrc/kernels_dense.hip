// Dense kernels of libsnf for gfx950 (MI355X, CDNA4).
//
//  * f_0              -- X_0 = f_0(F) (Algorithm 1 or 2 initial map) into a zero-padded
//                        n_pad x n_pad buffer, symmetric by construction (upper triangle of F
//                        read, LDS-transposed for the lower half), plus per-block partial sums
//                        of tr X_0 and ||X_0||_F^2 and the low-precision operand copy.
//  * product kernels  -- P = A.B for symmetric A, B on MFMA (f64 16x16x4, f32 16x16x4,
//                        bf16 16x16x32 with f32 accumulation), LDS double-buffered 128x128
//                        output tiles, only the upper triangle of tiles (P is symmetric) with
//                        the mirror written by the same workgroup; fused epilogue
//                        Y = c2 P + c1 X + c0 I and FP64 partial sums of ||P - X||_F^2,
//                        tr Y, ||Y||_F^2 per tile.
//                        The FP64 variant with a second epilogue output serves the first
//                        product of a P_{i,j} iteration.
//  * direct kernels   -- FP64 solves up to the order where a tile of at most 96x96 per compute
//                        unit covers the upper triangle: operands straight from L2 to
//                        registers, k split over the four waves of a workgroup, the schedule at
//                        the head of the next step's kernel; at the smallest orders the whole
//                        solve in one workgroup, iterates in LDS.
//  * schedule_kernel  -- one workgroup: fixed-order reduction of the per-tile partials and the
//                        scalar state machine (branch, alpha, beta, beta-bar, stopping).
//  * start / finish   -- a solve's tables with its f_0; D and the final state out.
//  * copy kernels     -- padded <-> caller layout.
//  * grouped kernels  -- the serving loop's step over many requests in one launch.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <type_traits>

#include "schedule_math.h"
#include "snf_internal.h"
#include "wave_sum.h"

namespace snf {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef float flt4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 16-byte load through a global-address-space pointer, so the compiler emits global_load
// (counted by vmcnt only) instead of flat_load, whose completion is also tracked by lgkmcnt
// and would make every LDS-read wait of the main loop wait for the operand prefetch too.
template <typename T>
__device__ __forceinline__ u32x4 gload16(const T* p) {
  return *(const __attribute__((address_space(1))) u32x4*)(p);
}

__device__ __forceinline__ unsigned short f32_to_bf16_rne(float f) {
  // round-to-nearest-even truncation of an IEEE binary32 to bfloat16 (NaN kept quiet)
  unsigned int u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

// ---------------------------------------------------------------------------------------
// Wave / block reductions in a fixed order (deterministic).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum three values over the block (up to 8 waves), in wave order; result valid in thread 0.
__device__ __forceinline__ void block_sum3(double& a, double& b, double& c, double* lds24) {
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    lds24[w * 3 + 0] = a;
    lds24[w * 3 + 1] = b;
    lds24[w * 3 + 2] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = blockDim.x >> 6;
    double sa = lds24[0], sb = lds24[1], sc = lds24[2];
    for (int i = 1; i < nw; ++i) {
      sa += lds24[3 * i + 0];
      sb += lds24[3 * i + 1];
      sc += lds24[3 * i + 2];
    }
    a = sa;
    b = sb;
    c = sc;
  }
}

// ---------------------------------------------------------------------------------------
// f0: X_0 = f_0(F)
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void f0_body(const double* __restrict__ F, int64_t n, int64_t ld,
                                        int64_t np, const SnfHeader& h, double* __restrict__ X,
                                        void* __restrict__ LP, int lowp_kind,
                                        double* __restrict__ partials) {
  __shared__ double tile[32][33];
  __shared__ double red[24];
  const int alg1 = (h.scheme == SNF_MCWEENY || h.scheme == SNF_SNF_FIXMU || h.pmm_m || h.pij_i);
  const double lmin = h.lambda_min, lmax = h.lambda_max, mu = h.mu, gamma = h.gamma;
  const double xs = h.xstar;
  const int64_t nt = np / 32;
  const int64_t ntiles = nt * nt;
  double t1 = 0.0, t2 = 0.0;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int64_t bi = t / nt, bj = t % nt;
    const int64_t si = bi < bj ? bi : bj, sj = bi < bj ? bj : bi;  // source tile (upper)
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int64_t gr = si * 32 + r, gc = sj * 32 + tx;
      tile[r][tx] = (gr < n && gc < n) ? F[gr * ld + gc] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int64_t gr = bi * 32 + r, gc = bj * 32 + tx;
      const double v = (gr <= gc) ? tile[r][tx] : tile[tx][r];
      double x = 0.0;
      if (gr < n && gc < n) {
        const bool d = (gr == gc);
        if (alg1) {
          x = ((d ? mu : 0.0) - v) / gamma + (d ? xs : 0.0);
        } else {
          x = ((d ? lmax : 0.0) - v) / (lmax - lmin);
        }
        if (d) t1 += x;
        t2 += x * x;
      }
      X[gr * np + gc] = x;
      if (lowp_kind == kPrecF32) {
        ((float*)LP)[gr * np + gc] = (float)x;
      } else if (lowp_kind == kPrecBF16) {
        ((unsigned short*)LP)[gr * np + gc] = f32_to_bf16_rne((float)x);
      }
    }
  }
  double e0 = 0.0;
  block_sum3(e0, t1, t2, red);
  if (threadIdx.x == 0) {
    partials[blockIdx.x * 4 + 0] = 0.0;
    partials[blockIdx.x * 4 + 1] = t1;
    partials[blockIdx.x * 4 + 2] = t2;
    partials[blockIdx.x * 4 + 3] = 0.0;
  }
}

__global__ __launch_bounds__(256) void f0_kernel(const double* __restrict__ F, int64_t n,
                                                 int64_t ld, int64_t np,
                                                 const SnfState* __restrict__ st,
                                                 const Buffers* __restrict__ bufs,
                                                 int lowp_kind, double* __restrict__ partials) {
  f0_body(F, n, ld, np, *st, bufs->x[st->cur], bufs->lp[st->cur], lowp_kind, partials);
}

void launch_f0(const double* F, int64_t n, int64_t ld, int64_t np, SnfState* st,
               const Buffers* bufs_dev, int lowp_kind, double* partials, hipStream_t s) {
  hipLaunchKernelGGL(f0_kernel, dim3(kF0Blocks), dim3(256), 0, s, F, n, ld, np, st, bufs_dev,
                     lowp_kind, partials);
}

// ---------------------------------------------------------------------------------------
// Tile enumeration: upper triangle of 128x128 tiles (bi <= bj) or the full grid, with the
// workgroup id remapped so that each XCD (workgroups are dealt round-robin to the 8 XCDs)
// works on a contiguous stretch of the tile list, which shares operand panels in its L2.
// ---------------------------------------------------------------------------------------
int num_product_tiles(int64_t np, int sym) {
  const int64_t nt = np / kTile;
  return (int)(sym ? nt * (nt + 1) / 2 : nt * nt);
}

__device__ __forceinline__ int xcd_remap(int w, int total) {
  const int xcd = w & 7, slot = w >> 3;
  const int base = total >> 3, rem = total & 7;
  return xcd * base + (xcd < rem ? xcd : rem) + slot;
}

// Order of the upper-triangle tiles: the triangle is cut into blocks of kOrderG x kOrderG
// tiles; the off-diagonal blocks come first (row-major over the blocks, row-major inside a
// block), then the diagonal blocks (their upper triangles, row-major).  A full off-diagonal
// block is 64 tiles, what one XCD runs at once (32 CUs x 2 workgroups), and needs 16 operand
// panels (tile (i, j) reads row panels i and j, by symmetry).  Summed over the XCDs and
// their waves of 64, the row-major order of the whole triangle touches 1.4x as many panels
// at n = 4096 and 2.7x at n = 8192.
constexpr int kOrderG = 8;

__device__ __forceinline__ void tile_coords(int t, int nt, int sym, int& bi, int& bj) {
  if (!sym) {
    bi = t / nt;
    bj = t % nt;
    return;
  }
  const int G = kOrderG;
  const int nb = (nt + G - 1) / G;
  // off-diagonal blocks: block row P holds G * (nt - (P + 1) G) tiles (only the last block
  // row and column can be partial, and the last block row has no off-diagonal block)
  int rem = t;
  for (int P = 0; P + 1 < nb; ++P) {
    const int right = nt - (P + 1) * G;
    const int cnt = G * right;
    if (rem < cnt) {
      const int q = rem / (G * G);               // full blocks to the left in this row
      const int Q = P + 1 + q;
      const int hq = min(G, nt - Q * G);
      const int rr = rem - q * G * G;
      bi = P * G + rr / hq;
      bj = Q * G + rr % hq;
      return;
    }
    rem -= cnt;
  }
  // diagonal blocks: block P of h = min(G, nt - P G) tiles a side holds h (h + 1) / 2
  for (int P = 0; P < nb; ++P) {
    const int h = min(G, nt - P * G);
    const int cnt = h * (h + 1) / 2;
    if (rem < cnt || P + 1 == nb) {
      int r = 0;
      while (rem >= h - r) {
        rem -= h - r;
        ++r;
      }
      bi = P * G + r;
      bj = P * G + r + rem;
      return;
    }
    rem -= cnt;
  }
}

// ---------------------------------------------------------------------------------------
// MFMA wrappers, the shared epilogue, slices
// ---------------------------------------------------------------------------------------
template <typename T> struct Mfma;
template <> struct Mfma<double> {
  typedef dbl4 acc_t;
  static constexpr int kBK = 16;   // k-depth per stage (128 B per LDS row)
  static constexpr int kPad = 16;  // row stride 144 doubles = 1152 B
  __device__ static __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma<float> {
  typedef flt4 acc_t;
  static constexpr int kBK = 32;
  static constexpr int kPad = 16;  // row stride 144 floats = 576 B
  __device__ static __forceinline__ acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Shared epilogue over the 64x64 wave tile held as acc[4][4] (MFMA 16x16 blocks).
// Accumulator layout of lane l, register v: column l % 16 and row
//   4 (l / 16) + v   for the f32 and bf16 MFMAs (ROWS_INTERLEAVED = false),
//   (l / 16) + 4 v   for the f64 MFMA          (ROWS_INTERLEAVED = true).
struct EpiArgs {
  const double* Xt;  // linear term X (FP64)
  double* Y;         // output (FP64)
  void* LPY;         // low-precision copy of the output, or unused
  double* Y2;        // second output d2 P + d1 X + d0 I (FP64), or null
  int lowp_kind;     // kPrecF32 / kPrecBF16 / -1
  int want_e;
  double c2, c1, c0;
  double d2, d1, d0;
};

__device__ __forceinline__ EpiArgs epi_args(const SnfHeader* st, const Buffers* bufs) {
  EpiArgs e;
  e.Xt = bufs->x[st->ix];
  e.Y = bufs->x[st->io];
  e.LPY = bufs->lp[st->io];
  e.Y2 = st->dual ? bufs->x[st->io2] : nullptr;
  e.d2 = st->d2;
  e.d1 = st->d1;
  e.d0 = st->d0;
  e.lowp_kind = st->write_lowp ? (st->mode == SNF_P_BF16_REF64 ? kPrecBF16 : kPrecF32) : -1;
  e.want_e = st->want_e;
  e.c2 = st->c2;
  e.c1 = st->c1;
  e.c0 = st->c0;
  return e;
}

// Epilogue of one product entry p at global (r, c), x = X[r][c] (loaded by the caller, ahead
// of the stores, so that the loads of many entries are in flight together: the compiler may not
// move a load of X above a store to Y, which it cannot tell apart): Y = c2 p + c1 X +
// c0 [r == c], the FP64 sums, the mirror write.  In symmetric mode a diagonal tile keeps its
// upper half and mirrors it, so the result is exactly symmetric; every off-diagonal entry then
// stands for two.  With DUAL the second output Y2 is written too (compiled only into the
// kernel variants that need it, so the others keep their register budget).
template <bool DUAL = false>
__device__ __forceinline__ void epi_elem(double p, double x, int64_t r, int64_t c, int sym,
                                         int diag, int64_t n, int64_t np, const EpiArgs& ea,
                                         double& e2, double& t1, double& t2) {
  if (diag && sym && r > c) return;
  const bool mirror = sym && r != c;
  const double w = mirror ? 2.0 : 1.0;
  if (ea.want_e) {
    const double d = p - x;
    e2 += w * (d * d);
  }
  double y = ea.c2 * p + ea.c1 * x + (r == c ? ea.c0 : 0.0);
  if (r >= n || c >= n) y = 0.0;
  if (r == c) t1 += y;
  t2 += w * (y * y);
  ea.Y[r * np + c] = y;
  if (mirror) ea.Y[c * np + r] = y;
  if (DUAL && ea.Y2) {
    double y2 = ea.d2 * p + ea.d1 * x + (r == c ? ea.d0 : 0.0);
    if (r >= n || c >= n) y2 = 0.0;
    ea.Y2[r * np + c] = y2;
    if (mirror) ea.Y2[c * np + r] = y2;
  }
  if (ea.lowp_kind == kPrecF32) {
    const float yf = (float)y;
    ((float*)ea.LPY)[r * np + c] = yf;
    if (mirror) ((float*)ea.LPY)[c * np + r] = yf;
  } else if (ea.lowp_kind == kPrecBF16) {
    const unsigned short yb = f32_to_bf16_rne((float)y);
    ((unsigned short*)ea.LPY)[r * np + c] = yb;
    if (mirror) ((unsigned short*)ea.LPY)[c * np + r] = yb;
  }
}

// Row of accumulator register v of lane l inside its 16x16 MFMA block:
//   4 (l / 16) + v   for the f32 and bf16 MFMAs (ROWS_INTERLEAVED = false),
//   (l / 16) + 4 v   for the f64 MFMA          (ROWS_INTERLEAVED = true);
// the column is l % 16 for all three.
template <bool ROWS_INTERLEAVED>
__device__ __forceinline__ int acc_row(int lane, int v) {
  return ROWS_INTERLEAVED ? (lane >> 4) + 4 * v : 4 * (lane >> 4) + v;
}

// Off-diagonal tile of a symmetric product in the f32 / bf16 accumulator layout: the lane's
// four values are rows r0 .. r0 + 3 of column c, so their mirror entries Y[c][r0 .. r0 + 3] are
// contiguous and go out as two 16-byte stores (and one 16- or 8-byte store of the
// low-precision copy) instead of four scattered 8-byte ones.  Same values as epi_elem.
template <typename Acc4>
__device__ __forceinline__ void epi_quad_mirrored(const Acc4& acc4, const double (&x4)[4],
                                                  int64_t r0, int64_t c, int64_t n, int64_t np,
                                                  const EpiArgs& ea, double& e2, double& t2) {
  double y[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t r = r0 + v;
    const double p = (double)acc4[v];
    const double x = x4[v];
    if (ea.want_e) {
      const double d = p - x;
      e2 += 2.0 * (d * d);
    }
    double yv = ea.c2 * p + ea.c1 * x;      // r != c in an off-diagonal tile
    if (r >= n || c >= n) yv = 0.0;
    t2 += 2.0 * (yv * yv);
    ea.Y[r * np + c] = yv;
    y[v] = yv;
  }
  double* ym = ea.Y + c * np + r0;
  *(double2*)(ym) = double2{y[0], y[1]};
  *(double2*)(ym + 2) = double2{y[2], y[3]};
  if (ea.lowp_kind == kPrecF32) {
    float* lp = (float*)ea.LPY;
    float f[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      f[v] = (float)y[v];
      lp[(r0 + v) * np + c] = f[v];
    }
    *(float4*)(lp + c * np + r0) = float4{f[0], f[1], f[2], f[3]};
  } else if (ea.lowp_kind == kPrecBF16) {
    unsigned short* lp = (unsigned short*)ea.LPY;
    unsigned short b[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      b[v] = f32_to_bf16_rne((float)y[v]);
      lp[(r0 + v) * np + c] = b[v];
    }
    *(uint2*)(lp + c * np + r0) = uint2{(unsigned)b[0] | ((unsigned)b[1] << 16),
                                        (unsigned)b[2] | ((unsigned)b[3] << 16)};
  }
}

// X[r][c] of the four entries of MFMA block (m, q) held by this lane.
template <bool ROWS_INTERLEAVED>
__device__ __forceinline__ void load_x_block(double (&x4)[4], int m, int q, int gi0, int gj0,
                                             int64_t np, const EpiArgs& ea) {
  const int lane = threadIdx.x & 63;
  const int64_t c = gj0 + q * 16 + (lane & 15);
#pragma unroll
  for (int v = 0; v < 4; ++v)
    x4[v] = ea.Xt[(gi0 + m * 16 + acc_row<ROWS_INTERLEAVED>(lane, v)) * np + c];
}

// One 16x16 MFMA block (m, q) of the wave tile: acc4 holds its four values of this lane, x4
// the matching entries of X.
template <bool ROWS_INTERLEAVED, bool DUAL, typename Acc4>
__device__ __forceinline__ void epilogue_block(const Acc4& acc4, const double (&x4)[4], int m,
                                               int q, int gi0, int gj0, int sym, int diag,
                                               int64_t n, int64_t np, const EpiArgs& ea,
                                               double& e2, double& t1, double& t2) {
  const int lane = threadIdx.x & 63;
  const int64_t c = gj0 + q * 16 + (lane & 15);
  if (!ROWS_INTERLEAVED && !DUAL && sym && !diag) {
    epi_quad_mirrored(acc4, x4, gi0 + m * 16 + acc_row<false>(lane, 0), c, n, np, ea, e2, t2);
    return;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t r = gi0 + m * 16 + acc_row<ROWS_INTERLEAVED>(lane, v);
    epi_elem<DUAL>((double)acc4[v], x4[v], r, c, sym, diag, n, np, ea, e2, t1, t2);
  }
}

// The wave tile's epilogue.  X values are loaded in batches ahead of the stores: BATCH -1
// loads each value just before its entry's stores, 0 the four values of one MFMA block before
// that block's stores, 1 those of a row of blocks before the row's stores, 2 also the next
// row's before the current row's stores (more registers each: the FP64 kernels, at 4 waves per
// SIMD, have room only for -1).
template <bool ROWS_INTERLEAVED, bool DUAL, int BATCH = 0, int MT, int QT, typename AccT>
__device__ __forceinline__ void epilogue(const AccT (&acc)[MT][QT], int gi0, int gj0, int sym,
                                         int diag, int64_t n, int64_t np, const EpiArgs& ea,
                                         double& e2, double& t1, double& t2) {
  if constexpr (BATCH < 0) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        const int64_t c = gj0 + q * 16 + (lane & 15);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t r = gi0 + m * 16 + acc_row<ROWS_INTERLEAVED>(lane, v);
          if (diag && sym && r > c) continue;   // (the entry's mirror is written instead)
          epi_elem<DUAL>((double)acc[m][q][v], ea.Xt[r * np + c], r, c, sym, diag, n, np, ea,
                         e2, t1, t2);
        }
      }
  } else if constexpr (BATCH == 0) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        double x4[4];
        load_x_block<ROWS_INTERLEAVED>(x4, m, q, gi0, gj0, np, ea);
        epilogue_block<ROWS_INTERLEAVED, DUAL>(acc[m][q], x4, m, q, gi0, gj0, sym, diag, n, np,
                                               ea, e2, t1, t2);
      }
  } else {
    constexpr int NB = BATCH == 2 ? 2 : 1;
    double xs[NB][QT][4];
    if (BATCH == 2) {
#pragma unroll
      for (int q = 0; q < QT; ++q)
        load_x_block<ROWS_INTERLEAVED>(xs[0][q], 0, q, gi0, gj0, np, ea);
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int nm = BATCH == 2 ? m + 1 : m;
      if (nm < MT) {
#pragma unroll
        for (int q = 0; q < QT; ++q)
          load_x_block<ROWS_INTERLEAVED>(xs[nm % NB][q], nm, q, gi0, gj0, np, ea);
      }
#pragma unroll
      for (int q = 0; q < QT; ++q)
        epilogue_block<ROWS_INTERLEAVED, DUAL>(acc[m][q], xs[m % NB][q], m, q, gi0, gj0, sym,
                                               diag, n, np, ea, e2, t1, t2);
    }
  }
}

__device__ __forceinline__ void write_partials(double e2, double t1, double t2,
                                               double* partials, int tile) {
  __shared__ double red[24];
  block_sum3(e2, t1, t2, red);
  if (threadIdx.x == 0) {
    partials[tile * 4 + 0] = e2;
    partials[tile * 4 + 1] = t1;
    partials[tile * 4 + 2] = t2;
    partials[tile * 4 + 3] = 0.0;
  }
}

// Work decomposition of one product launch.  Workgroups [0, dp_tiles) compute whole tiles
// (id remapped per XCD); the remaining workgroups compute one of split_s k-slices of the
// tail tiles [dp_tiles, dp_tiles + tail_tiles) and store their raw accumulators; the
// fix-up kernel adds the slices of a tile in a fixed order and runs the epilogue.
struct WorkItem {
  int tile;
  int piece;     // -1 for a whole tile, else the slice's index into the split buffer
  int kt_begin, kt_end;
};

__device__ __forceinline__ WorkItem work_item(const ProductGrid& g, int KT) {
  WorkItem it;
  const int w = blockIdx.x;
  if (w < g.dp_tiles) {
    it.tile = xcd_remap(w, g.dp_tiles);
    it.piece = -1;
    it.kt_begin = 0;
    it.kt_end = KT;
  } else {
    const int q = w - g.dp_tiles;
    const int p = q % g.split_s;
    it.tile = g.dp_tiles + q / g.split_s;
    it.piece = q;
    it.kt_begin = (int)((int64_t)p * KT / g.split_s);
    it.kt_end = (int)((int64_t)(p + 1) * KT / g.split_s);
  }
  return it;
}

// Raw accumulators of a k-slice in tile order: split[piece][r][c], r, c < 128, whatever the
// thread layout of the kernel that produced them, in the accumulators' type (SliceT).
template <typename SliceT, bool ROWS_INTERLEAVED, int MT, int QT, typename AccT>
__device__ __forceinline__ void store_slice(const AccT (&acc)[MT][QT], int wr0, int wc0,
                                            double* split, int piece) {
  const int lane = threadIdx.x & 63;
  SliceT* base = (SliceT*)split + (size_t)piece * kTile * kTile;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int q = 0; q < QT; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = wr0 + m * 16 + acc_row<ROWS_INTERLEAVED>(lane, v);
        const int c = wc0 + q * 16 + (lane & 15);
        base[r * kTile + c] = acc[m][q][v];
      }
}

// ---------------------------------------------------------------------------------------
// Product kernel, f64 / f32 MFMA 16x16x4.
//   LDS tiles hold 'k-rows' of both operands: sA[k][i] = A[k0+k][i0+i] and
//   sB[k][j] = B[k0+k][j0+j]; A[i][k] = A[k][i] because A is symmetric, so both panels are
//   read with contiguous, coalesced rows.  MFMA operand of lane l: row/col (l % 16), k (l / 16).
// ---------------------------------------------------------------------------------------
// Thread layout: NT threads = (NT/64) waves in WR x WC, each wave a (TILE/WR) x (TILE/WC)
// piece of the tile made of MT x QT MFMA 16x16 blocks.
template <typename T, int TILE> struct Layout;
template <> struct Layout<double, kTile> {   // 8 waves of 64x32: 64 accumulator registers per
  static constexpr int NT = 512, WC = 4;     // lane, so 4 waves fit on each SIMD
};
template <> struct Layout<float, kTile> {    // 8 waves of 32x64: 32 accumulator registers per
  static constexpr int NT = 512, WC = 2;     // lane, 4 waves per SIMD
};
template <> struct Layout<float, kFineTile> {   // 4 waves of 32x32
  static constexpr int NT = 256, WC = 2;
};

template <typename T, int PREC, bool DUAL = false, int TILE = kTile>
__device__ __forceinline__ void product_body(const SnfState* __restrict__ st,
                                             const Buffers* __restrict__ bufs,
                                             const ProductGrid& g, const WorkItem& wi) {
  typedef Mfma<T> M;
  constexpr int NT = Layout<T, TILE>::NT, WC = Layout<T, TILE>::WC, WR = NT / 64 / WC;
  constexpr int TR = TILE / WR, TC = TILE / WC, MT = TR / 16, QT = TC / 16;
  constexpr int BK = M::kBK, LDS_W = TILE + M::kPad;
  constexpr int VE = 16 / sizeof(T);          // elements per 16-byte vector
  constexpr int VPR = TILE / VE;             // vectors per LDS row
  constexpr int RPP = NT / VPR;               // rows per load pass
  constexpr int PASSES = BK / RPP;
  __shared__ __attribute__((aligned(16))) T sA[2][BK][LDS_W];
  __shared__ __attribute__((aligned(16))) T sB[2][BK][LDS_W];

  const int64_t np = g.np;
  const T* A = (PREC == kPrecF64) ? (const T*)bufs->x[st->ia] : (const T*)bufs->lp[st->ia];
  const T* B = (PREC == kPrecF64) ? (const T*)bufs->x[st->ib] : (const T*)bufs->lp[st->ib];

  int bi, bj;
  tile_coords(wi.tile, (int)(np / TILE), g.sym, bi, bj);
  const int64_t i0 = (int64_t)bi * TILE, j0 = (int64_t)bj * TILE;

  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wr = wid / WC, wc = wid % WC;
  const int lrow = tid / VPR, lvec = tid % VPR;

  typename M::acc_t acc[MT][QT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int q = 0; q < QT; ++q) acc[m][q] = typename M::acc_t{0, 0, 0, 0};

  u32x4 ra0[PASSES], rb0[PASSES], ra1[PASSES], rb1[PASSES];
  auto gload = [&](u32x4 (&ra)[PASSES], u32x4 (&rb)[PASSES], int64_t k0) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int64_t k = k0 + p * RPP + lrow;
      ra[p] = gload16(A + k * np + i0 + lvec * VE);
      rb[p] = gload16(B + k * np + j0 + lvec * VE);
    }
  };
  auto lstore = [&](const u32x4 (&ra)[PASSES], const u32x4 (&rb)[PASSES], int buf) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      *(u32x4*)(&sA[buf][p * RPP + lrow][lvec * VE]) = ra[p];
      *(u32x4*)(&sB[buf][p * RPP + lrow][lvec * VE]) = rb[p];
    }
  };
  const int fr = lane & 15, fk = lane >> 4;
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      T a[MT], b[QT];
#pragma unroll
      for (int m = 0; m < MT; ++m) a[m] = sA[buf][kk + fk][wr * TR + m * 16 + fr];
#pragma unroll
      for (int q = 0; q < QT; ++q) b[q] = sB[buf][kk + fk][wc * TC + q * 16 + fr];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int q = 0; q < QT; ++q) acc[m][q] = M::mma(a[m], b[q], acc[m][q]);
    }
  };
  // FP32: operands two stages ahead in two register sets, the loads issued on every path
  // (past the end the last stage again, never stored) so that the wait before the LDS stores
  // leaves the newer set in flight.  FP64: one stage ahead (a stage's 32 MFMAs per wave take
  // long enough to cover the loads, and the FP64 kernel has no registers to spare).
  const int kb = wi.kt_begin, ke = wi.kt_end;
  gload(ra0, rb0, (int64_t)kb * BK);
  lstore(ra0, rb0, 0);
  if constexpr (PREC == kPrecF32) {
    gload(ra1, rb1, (int64_t)min(kb + 1, ke - 1) * BK);
    __syncthreads();
    int kt = kb;
    while (true) {
      {
        const int buf = (kt - kb) & 1;
        gload(ra0, rb0, (int64_t)min(kt + 2, ke - 1) * BK);
        compute(buf);
        if (kt + 1 < ke) lstore(ra1, rb1, buf ^ 1);
        __syncthreads();
        if (++kt >= ke) break;
      }
      {
        const int buf = (kt - kb) & 1;
        gload(ra1, rb1, (int64_t)min(kt + 2, ke - 1) * BK);
        compute(buf);
        if (kt + 1 < ke) lstore(ra0, rb0, buf ^ 1);
        __syncthreads();
        if (++kt >= ke) break;
      }
    }
  } else {
    __syncthreads();
    for (int kt = kb; kt < ke; ++kt) {
      const int buf = (kt - kb) & 1;
      const bool more = kt + 1 < ke;
      if (more) gload(ra0, rb0, (int64_t)(kt + 1) * BK);
      compute(buf);
      if (more) lstore(ra0, rb0, buf ^ 1);
      __syncthreads();
    }
  }

  if (wi.piece >= 0) {
    store_slice<T, PREC == kPrecF64>(acc, wr * TR, wc * TC, g.split_buf, wi.piece);
    return;
  }
  const EpiArgs ea = epi_args(st, bufs);
  double e2 = 0.0, t1 = 0.0, t2 = 0.0;
  epilogue<PREC == kPrecF64, DUAL, PREC == kPrecF64 ? -1 : 0>(acc, (int)(i0 + wr * TR),
                                                             (int)(j0 + wc * TC), g.sym,
                                   bi == bj, g.n, np, ea, e2, t1, t2);
  write_partials(e2, t1, t2, g.partials, wi.tile);
}

// ---------------------------------------------------------------------------------------
// Product kernel, bf16 MFMA 16x16x32 with f32 accumulation.
//   Here the LDS tiles are 'row panels' with k contiguous: sA[i][k] = A[i0+i][k0+k] and
//   sB[j][k] = B[j0+j][k0+k] (B[k][j] = B[j][k] by symmetry), because a lane's MFMA operand
//   is 8 consecutive k values of one row / column: lane l holds row (l % 16),
//   k = 8 (l / 16) .. 8 (l / 16) + 7.  Rows are 128 bytes (eight 16-byte chunks) without
//   padding; chunk c of row r is stored at position c ^ ((r >> 1) & 7), so that both the
//   stores (two rows of eight chunks per 16 lanes) and the operand reads (16 rows, one chunk
//   each) hit every bank once.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void product_bf16_body(const SnfState* __restrict__ st,
                                                  const Buffers* __restrict__ bufs,
                                                  const ProductGrid& g, const WorkItem& wi) {
  constexpr int BK = 64;                 // bf16 per LDS row per stage = 128 B
  constexpr int LDS_W = BK;              // row stride 128 B, chunks swizzled
  constexpr int VPR = BK / 8;            // 16-byte vectors per row = 8
  constexpr int RPP = kThreads / VPR;    // 32 rows per pass
  constexpr int PASSES = kTile / RPP;    // 4
  __shared__ __attribute__((aligned(16))) unsigned short sA[2][kTile][LDS_W];
  __shared__ __attribute__((aligned(16))) unsigned short sB[2][kTile][LDS_W];

  const int64_t np = g.np;
  const unsigned short* A = (const unsigned short*)bufs->lp[st->ia];
  const unsigned short* B = (const unsigned short*)bufs->lp[st->ib];

  int bi, bj;
  tile_coords(wi.tile, (int)(np / kTile), g.sym, bi, bj);
  const int64_t i0 = (int64_t)bi * kTile, j0 = (int64_t)bj * kTile;

  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wr = wid >> 1, wc = wid & 1;
  const int lrow = tid / VPR, lvec = tid % VPR;

  flt4 acc[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[m][q] = flt4{0.f, 0.f, 0.f, 0.f};

  u32x4 ra0[PASSES], rb0[PASSES], ra1[PASSES], rb1[PASSES];
  auto gload = [&](u32x4 (&ra)[PASSES], u32x4 (&rb)[PASSES], int64_t k0) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int64_t r = p * RPP + lrow;
      ra[p] = gload16(A + (i0 + r) * np + k0 + lvec * 8);
      rb[p] = gload16(B + (j0 + r) * np + k0 + lvec * 8);
    }
  };
  auto lstore = [&](const u32x4 (&ra)[PASSES], const u32x4 (&rb)[PASSES], int buf) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int rr = p * RPP + lrow, pc = (lvec ^ ((rr >> 1) & 7)) * 8;
      *(u32x4*)(&sA[buf][rr][pc]) = ra[p];
      *(u32x4*)(&sB[buf][rr][pc]) = rb[p];
    }
  };
  const int fr = lane & 15, fk = (lane >> 4) * 8;
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 32) {
      bf16x8 a[4], b[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int rr = wr * 64 + m * 16 + fr;
        a[m] = *(const bf16x8*)(&sA[buf][rr][(((kk + fk) >> 3) ^ ((rr >> 1) & 7)) * 8]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int rr = wc * 64 + q * 16 + fr;
        b[q] = *(const bf16x8*)(&sB[buf][rr][(((kk + fk) >> 3) ^ ((rr >> 1) & 7)) * 8]);
      }
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc[m][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b[q], acc[m][q], 0, 0, 0);
    }
  };

  // Operands two stages ahead in two register sets: stage kt computes from LDS buffer
  // (kt - kb) & 1, stores stage kt + 1 (loaded during the previous stage) into the other
  // buffer and loads stage kt + 2.  The loads are issued on every path (past the end the
  // last stage again, never stored): with a conditional load the compiler's wait before the
  // LDS stores would also cover the newer set and the second stage of lead would be lost.
  const int kb = wi.kt_begin, ke = wi.kt_end;
  gload(ra0, rb0, (int64_t)kb * BK);
  lstore(ra0, rb0, 0);
  gload(ra1, rb1, (int64_t)min(kb + 1, ke - 1) * BK);
  __syncthreads();
  int kt = kb;
  while (true) {
    {
      const int buf = (kt - kb) & 1;
      gload(ra0, rb0, (int64_t)min(kt + 2, ke - 1) * BK);
      compute(buf);
      if (kt + 1 < ke) lstore(ra1, rb1, buf ^ 1);
      __syncthreads();
      if (++kt >= ke) break;
    }
    {
      const int buf = (kt - kb) & 1;
      gload(ra1, rb1, (int64_t)min(kt + 2, ke - 1) * BK);
      compute(buf);
      if (kt + 1 < ke) lstore(ra0, rb0, buf ^ 1);
      __syncthreads();
      if (++kt >= ke) break;
    }
  }

  if (wi.piece >= 0) {
    store_slice<float, false>(acc, wr * 64, wc * 64, g.split_buf, wi.piece);
    return;
  }
  const EpiArgs ea = epi_args(st, bufs);
  double e2 = 0.0, t1 = 0.0, t2 = 0.0;
  epilogue<false, false, 2>(acc, (int)(i0 + wr * 64), (int)(j0 + wc * 64), g.sym, bi == bj,
                            g.n,
                         np, ea, e2, t1, t2);
  write_partials(e2, t1, t2, g.partials, wi.tile);
}

__global__ __launch_bounds__(512, 2) void product_f64_kernel(const SnfState* __restrict__ st,
                                                             const Buffers* __restrict__ bufs,
                                                             ProductGrid g) {
  if (st->stop || st->prec != kPrecF64 || st->dual) return;
  product_body<double, kPrecF64>(st, bufs, g, work_item(g, (int)(g.np / Mfma<double>::kBK)));
}

// The FP64 product whose epilogue also writes the second output (the first product of a
// P_{i,j} iteration); the host launches it beside product_f64_kernel for those schemes and
// exactly one of the two runs.
__global__ __launch_bounds__(512, 2) void product_f64_dual_kernel(const SnfState* __restrict__ st,
                                                                  const Buffers* __restrict__ bufs,
                                                                  ProductGrid g) {
  if (st->stop || st->prec != kPrecF64 || !st->dual) return;
  product_body<double, kPrecF64, true>(st, bufs, g,
                                       work_item(g, (int)(g.np / Mfma<double>::kBK)));
}

__global__ __launch_bounds__(512, 2) void product_f32_kernel(const SnfState* __restrict__ st,
                                                             const Buffers* __restrict__ bufs,
                                                             ProductGrid g) {
  if (st->stop || st->prec != kPrecF32) return;
  product_body<float, kPrecF32>(st, bufs, g, work_item(g, (int)(g.np / Mfma<float>::kBK)));
}

// Both of them, for launches of at most a workgroup per compute unit, where the LDS of both is no
// loss: a step of an FP32-start solve then has no launch that only finds out that the product is
// the other kernel's (19 products: n = 130 0.48 ms with the empty launches, 0.44 without; 300 0.54,
// 0.495; 700 0.78, 0.72; 1000 0.925, 0.875; 1900 2.42, 2.36).
__global__ __launch_bounds__(512, 2) void product_f64_f32_kernel(const SnfState* __restrict__ st,
                                                                 const Buffers* __restrict__ bufs,
                                                                 ProductGrid g) {
  if (st->stop) return;
  if (st->prec == kPrecF64)
    product_body<double, kPrecF64>(st, bufs, g, work_item(g, (int)(g.np / Mfma<double>::kBK)));
  else
    product_body<float, kPrecF32>(st, bufs, g, work_item(g, (int)(g.np / Mfma<float>::kBK)));
}

__global__ __launch_bounds__(256, 2) void product_bf16_kernel(const SnfState* __restrict__ st,
                                                              const Buffers* __restrict__ bufs,
                                                              ProductGrid g) {
  if (st->stop || st->prec != kPrecBF16) return;
  product_bf16_body(st, bufs, g, work_item(g, (int)(g.np / 64)));
}

// Fix-up of the split tail tiles: workgroup (t, b) handles rows 8b .. 8b + 7 of tail tile t
// (256 threads, 4 consecutive columns each); it adds the k-slices in slice order in FP64 (the
// loads of four slices in flight at a time), runs the epilogue of those entries and stores its
// sums in its own partials slot.  Bound by its read of the slices, which the FP32 and BF16
// products leave in FP32 as they accumulate it (stored in FP64, an FP32-start solve of 19 products
// took 0.59 ms at n = 300, 0.875 at 700, 1.00 at 1000 and 3.08 at 2000; this 0.525, 0.79, 0.93 and
// 3.00).  Eight slices in flight, and the linear term's loads ahead of them: no faster.
constexpr int kMaxSplit = 16;
template <typename SliceT>
__device__ __forceinline__ void add_slices(const double* split, size_t at, int count,
                                           double (&sum)[4]) {
  typedef SliceT vec __attribute__((ext_vector_type(4)));
  const vec* base = (const vec*)((const SliceT*)split + at);
  for (int p0 = 0; p0 < count; p0 += 4) {
    vec part[4];
#pragma unroll
    for (int pp = 0; pp < 4; ++pp)
      part[pp] = p0 + pp < count ? base[(size_t)(p0 + pp) * (kTile * kTile / 4)] : vec(0);
#pragma unroll
    for (int pp = 0; pp < 4; ++pp)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (p0 + pp < count) sum[v] += (double)part[pp][v];
  }
}

__global__ __launch_bounds__(256) void split_fixup_kernel(const SnfState* __restrict__ st,
                                                          const Buffers* __restrict__ bufs,
                                                          ProductGrid g) {
  if (st->stop) return;
  const int t = blockIdx.x >> 4, b = blockIdx.x & 15;
  const int tile = g.dp_tiles + t;
  int bi, bj;
  tile_coords(tile, (int)(g.np / kTile), g.sym, bi, bj);
  const int r = 8 * b + (threadIdx.x >> 5), c0 = (threadIdx.x & 31) * 4;
  const size_t at = (size_t)t * g.split_s * kTile * kTile + r * kTile + c0;
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
  if (st->prec == kPrecF64)
    add_slices<double>(g.split_buf, at, g.split_s, sum);
  else
    add_slices<float>(g.split_buf, at, g.split_s, sum);
  const EpiArgs ea = epi_args(st, bufs);
  double e2 = 0.0, t1 = 0.0, t2 = 0.0;
  const int64_t gr = (int64_t)bi * kTile + r;
  double xs[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) xs[v] = ea.Xt[gr * g.np + (int64_t)bj * kTile + c0 + v];
#pragma unroll
  for (int v = 0; v < 4; ++v)
    epi_elem<true>(sum[v], xs[v], gr, (int64_t)bj * kTile + c0 + v, g.sym, bi == bj, g.n, g.np,
                   ea, e2, t1, t2);
  write_partials(e2, t1, t2, g.partials, g.dp_tiles + blockIdx.x);
}

ProductGrid make_product_grid(int64_t np, int64_t n, int sym, int num_cus, double* partials,
                              double* split_buf, int split_cap, int stage_depth) {
  ProductGrid g;
  g.np = np;
  g.n = n;
  g.sym = sym;
  g.partials = partials;
  g.split_buf = split_buf;
  const int tiles = num_product_tiles(np, sym);
  g.dp_tiles = tiles;
  g.tail_tiles = 0;
  g.split_s = 1;
  g.partial_count = tiles;
  if (num_cus <= 0 || !split_buf) return g;
  const int rem = tiles % num_cus;
  // every slice needs at least one k-stage of the deepest stage that may run (f64 16,
  // f32 32, bf16 64 values of k per stage)
  const int kt_min = (int)(np / stage_depth);
  if (rem == 0) return g;
  int s;
  if (rem <= num_cus / 2) {
    s = num_cus / rem;            // a short tail: one slice per compute unit
  } else if (tiles == rem) {
    // a single wave of more than half as many tiles as compute units: whole tiles would
    // run one workgroup per compute unit; three or more slices per tile fill both
    // workgroup slots of every unit (n = 2048: 136 tiles, 3 slices each).  A lone workgroup
    // already gets about half the unit's rate, so two slices per tile gain nothing.
    s = 2 * num_cus / rem;
    if (s < 3) return g;
  } else {
    return g;                     // a long tail behind full waves: whole tiles
  }
  if (s > kt_min) s = kt_min;
  if (s > kMaxSplit) s = kMaxSplit;
  if (s < 2 || rem * s > split_cap) return g;
  g.dp_tiles = tiles - rem;
  g.tail_tiles = rem;
  g.split_s = s;
  g.partial_count = g.dp_tiles + 16 * rem;   // one slot per fix-up workgroup
  return g;
}

void launch_product(int prec, SnfState* st, const Buffers* bufs_dev, const ProductGrid& g,
                    hipStream_t s) {
  const int grid = g.dp_tiles + g.tail_tiles * g.split_s;
  if (prec == kPrecF64) {
    hipLaunchKernelGGL(product_f64_kernel, dim3(grid), dim3(Layout<double, kTile>::NT), 0, s, st,
                       bufs_dev, g);
  } else if (prec == kPrecF32) {
    hipLaunchKernelGGL(product_f32_kernel, dim3(grid), dim3(Layout<float, kTile>::NT), 0, s, st,
                       bufs_dev, g);
  } else {
    hipLaunchKernelGGL(product_bf16_kernel, dim3(grid), dim3(kThreads), 0, s, st, bufs_dev, g);
  }
}

bool launch_product_f64_f32(SnfState* st, const Buffers* bufs_dev, const ProductGrid& g,
                            int num_cus, hipStream_t s) {
  static_assert(Layout<double, kTile>::NT == 512 && Layout<float, kTile>::NT == 512,
                "one launch shape");
  const int grid = g.dp_tiles + g.tail_tiles * g.split_s;
  if (grid > num_cus) return false;
  hipLaunchKernelGGL(product_f64_f32_kernel, dim3(grid), dim3(512), 0, s, st, bufs_dev, g);
  return true;
}

void launch_product_dual(SnfState* st, const Buffers* bufs_dev, const ProductGrid& g,
                         hipStream_t s) {
  const int grid = g.dp_tiles + g.tail_tiles * g.split_s;
  hipLaunchKernelGGL(product_f64_dual_kernel, dim3(grid), dim3(Layout<double, kTile>::NT), 0, s, st,
                     bufs_dev, g);
}

void launch_split_fixup(SnfState* st, const Buffers* bufs_dev, const ProductGrid& g,
                        hipStream_t s) {
  if (g.tail_tiles == 0) return;
  hipLaunchKernelGGL(split_fixup_kernel, dim3(g.tail_tiles * 16), dim3(kThreads), 0, s, st,
                     bufs_dev, g);
}
// ---------------------------------------------------------------------------------------
// Schedule: reduce the partials in a fixed order, then advance the scalar state.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void decide(SnfScalars* s, const SnfConfig* c, const SnfTables* t,
                                       double root) {
#pragma clang fp contract(off)
  // precision phase (only for the mixed-precision modes)
  if (c->mode != SNF_P_FP64) {
    if (s->phase == kPhaseHigh && (s->betabar - s->beta) >= c->gap_switch) s->phase = kPhaseLow;
    if (s->phase == kPhaseLow && c->mode != SNF_P_FP32) {
      const double bound = s->beta > 1.0 - s->betabar ? s->beta : 1.0 - s->betabar;
      if (bound <= c->lowp_floor) s->phase = kPhaseRefine;
    }
  }
  s->prec = (s->phase == kPhaseLow) ? (c->mode == SNF_P_BF16_REF64 ? kPrecBF16 : kPrecF32)
                                    : kPrecF64;
  s->write_lowp = (c->mode != SNF_P_FP64 && s->phase != kPhaseRefine) ? 1 : 0;

  int scheme = c->scheme;
  if (s->phase == kPhaseRefine) scheme = c->has_nocc ? SNF_SP2_TRACE : SNF_MCWEENY;

  double a = 0.0;
  int br;
  if (scheme_is_pij(scheme)) {
    br = SNF_BRANCH_PIJ;
    a = (scheme == SNF_SNF_FIXMU_PIJ) ? root : 1.0;
  } else if (scheme == SNF_SP2_TRACE) {
    br = sched::trace_square(s->t1, s->t2, (double)c->n_occ) ? SNF_BRANCH_SQUARE
                                                             : SNF_BRANCH_FOLD;
  } else if (scheme == SNF_TC2_BETA || scheme == SNF_SNF_VARMU) {
    const bool sq = sched::alg2_square(s->beta, s->betabar);
    br = sq ? SNF_BRANCH_SQUARE : SNF_BRANCH_FOLD;
    if (scheme == SNF_SNF_VARMU)
      a = sq ? sched::alg2_square_alpha(s->beta) : sched::alg2_fold_alpha(s->betabar);
  } else if (scheme_pmm_m(scheme)) {
    br = s->pmm_m == 3 ? SNF_BRANCH_P33 : SNF_BRANCH_P55;
    a = (scheme == SNF_SNF_FIXMU3 || scheme == SNF_SNF_FIXMU5) ? root : 1.0;
  } else {
    br = SNF_BRANCH_P11;
    a = (scheme == SNF_SNF_FIXMU) ? sched::alg1_alpha(s->beta) : 1.0;
  }
  s->branch = br;
  s->alpha = a;
  // (results in locals, stored once: stores at the end of several branches would be merged into
  // one through a computed address, and the state could not stay in registers)
  double kc2, kc1, kc0, kd2 = s->d2, kd1 = s->d1, kd0 = s->d0;
  if (br == SNF_BRANCH_PIJ) {
    // W = V^2, V = a (X - x* I): W = a^2 P - 2 a^2 x* X + a^2 x*^2 I; and beside it the top
    // Horner level T = q_2h W + q_(2h-1) V + q_(2h-2) I in the same epilogue
    const double xs = s->xstar, a2 = a * a;
    const int h = (s->pij_i + s->pij_j) / 2;
    const double qt = t->pq[2 * h], qo = t->pq[2 * h - 1], qc = t->pq[2 * h - 2];
    kc2 = a2;
    kc1 = -2.0 * a2 * xs;
    kc0 = a2 * xs * xs;
    kd2 = qt * a2;
    kd1 = qo * a - 2.0 * qt * a2 * xs;
    kd0 = qt * a2 * xs * xs - qo * a * xs + qc;
  } else if (br == SNF_BRANCH_P33 || br == SNF_BRANCH_P55) {
    // W = (a (X - I/2))^2 = a^2 P - a^2 X + (a^2 / 4) I
    const double a2 = a * a;
    kc2 = a2;
    kc1 = -a2;
    kc0 = 0.25 * a2;
  } else if (br == SNF_BRANCH_SQUARE) {          // ((1+a) X - a I)^2 = (1+a)^2 P - 2a(1+a) X + a^2 I
    kc2 = (1.0 + a) * (1.0 + a);
    kc1 = -2.0 * a * (1.0 + a);
    kc0 = a * a;
  } else if (br == SNF_BRANCH_FOLD) {     // 2(1+a) X - (1+a)^2 P
    kc2 = -((1.0 + a) * (1.0 + a));
    kc1 = 2.0 * (1.0 + a);
    kc0 = 0.0;
  } else {                                // S2 = Xs^2 = a^2 P + 2 a c X + c^2 I, c = (1-a)/2
    const double sh = 0.5 * (1.0 - a);
    kc2 = a * a;
    kc1 = 2.0 * a * sh;
    kc0 = sh * sh;
  }
  s->c2 = kc2;
  s->c1 = kc1;
  s->c0 = kc0;
  s->d2 = kd2;
  s->d1 = kd1;
  s->d0 = kd0;
  s->kind = kKindSquare;
  s->want_e = 1;
  s->ia = s->ib = s->ix = s->cur;
  const int cur = s->cur, w = (cur + 1) & 3, ta = (cur + 2) & 3;
  int io = (br == SNF_BRANCH_P11) ? 2 : 1 - cur, left = s->horner_left, bw = s->bw, bt = s->bt;
  int io2 = s->io2, dual = 0;
  if (br == SNF_BRANCH_P33 || br == SNF_BRANCH_P55) {
    bw = io = w;
    left = s->pmm_m - 1;
  } else if (br == SNF_BRANCH_PIJ) {
    bw = io = w;
    dual = 1;
    io2 = bt = ta;
    left = (s->pij_i + s->pij_j) / 2 - 1;
  }
  s->io = io;
  s->io2 = io2;
  s->bw = bw;
  s->bt = bt;
  s->dual = dual;
  s->horner_left = left;
}

__device__ __forceinline__ void advance_beta(SnfScalars* s, const SnfTables* t, int br, double a) {
#pragma clang fp contract(off)
  if (br == SNF_BRANCH_SQUARE) {
    s->beta = sched::alg2_square_map(s->beta, a);
    s->betabar = sched::alg2_square_map(s->betabar, a);
  } else if (br == SNF_BRANCH_FOLD) {
    s->beta = sched::alg2_fold_map(s->beta, a);
    s->betabar = sched::alg2_fold_map(s->betabar, a);
  } else if (br == SNF_BRANCH_P11) {
    s->beta = sched::alg1_beta_next(s->beta, a);
    s->betabar = 1.0 - s->beta;
  } else if (br == SNF_BRANCH_PIJ) {
    const double xs = s->xstar;
    const double an = sched::pij_side_next_tab(s->pij_i, s->pij_j, t->pbin[0], xs, s->beta, a);
    const double bn =
        sched::pij_side_next_tab(s->pij_j, s->pij_i, t->pbin[1], 1.0 - xs, s->abar, a);
    s->beta = an;
    s->abar = bn;
    s->betabar = 1.0 - bn;
  } else {
    s->beta = sched::pij_eval_tab(s->pmm_m, s->pmm_m, t->pbin[0], a * (s->beta - 0.5) + 0.5);
    s->betabar = 1.0 - s->beta;
  }
}

// The bisection of sched::pmm_alpha_tab and sched::pij_alpha_side_tab by a wave, bit for bit: its
// halves each solve one side; in a round the 31 lanes of a half evaluate every midpoint that the
// next five halvings may meet (lane l: node l of a binary heap, its right child the upper half),
// and the walk down the answers takes the halvings.  Bound by the chain of 53 halvings, which in
// one thread took 0.5 us each and twice as many for P_{i,j}: scaled P_{3,1}, 28 products, n = 64
// 0.555 ms, this 0.28; 256 0.79, 0.50; 2100 5.00, 4.74; P_{3,3}, 25 products, n = 256 0.51, 0.40.
template <typename Diff>
__device__ __forceinline__ double wave_bisect(bool open, double hi, const Diff& diff) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63, node = (lane & 31) ? lane & 31 : 1;
  const int depth = 31 - __clz(node);
  double lo = 1.0;
  bool end = !open;
  for (int round = 0; round < 440 && __ballot(!end) != 0; ++round) {
    double a = lo, b = hi, mid = 0.5 * (a + b);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k < depth) {
        if ((node >> (depth - 1 - k)) & 1) a = mid; else b = mid;
        mid = 0.5 * (a + b);
      }
    const unsigned ends = (unsigned)(__ballot(mid <= a || mid >= b) >> (lane & 32));
    const unsigned ups = (unsigned)(__ballot(diff(mid) < 0.0) >> (lane & 32));
    int at = 1;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      end = end || ((ends >> at) & 1);
      if (!end) {
        const int up = (ups >> at) & 1;
        const double m = 0.5 * (lo + hi);
        if (up) lo = m; else hi = m;
        at = 2 * at + up;
      }
    }
  }
  return lo;
}

// Alpha of the iteration that the schedule on header h (in LDS) is about to set up, where it is
// the root of an Eq. 3 (else 0): the scaled P_{m,m} and P_{i,j} schemes, at the start (init) and
// behind an iteration's last product.  Every lane of one wave calls it and gets the result.
__device__ __forceinline__ double schedule_root(const SnfHeader& h, int init) {
#pragma clang fp contract(off)
  const int m = h.scheme == SNF_SNF_FIXMU3 || h.scheme == SNF_SNF_FIXMU5 ? h.pmm_m : 0;
  if (!m && h.scheme != SNF_SNF_FIXMU_PIJ) return 0.0;
  if (!init && h.kind != kKindFinal) return 0.0;
  SnfScalars s = h;
  if (!init) advance_beta(&s, &h, s.branch, s.alpha);
  if (m) {
    const double* bin = h.pbin[0];
    const double beta = s.beta;
    return wave_bisect(beta > 0.0 && beta < 0.5, 1.0 / (1.0 - 2.0 * beta), [&](double mid) {
#pragma clang fp contract(off)
      return sched::pij_eval_tab(m, m, bin, 0.5 * (1.0 - mid)) -
             sched::pij_eval_tab(m, m, bin, mid * (beta - 0.5) + 0.5);
    });
  }
  const bool hi_side = (threadIdx.x & 32) != 0;
  const int i = hi_side ? s.pij_j : s.pij_i, j = hi_side ? s.pij_i : s.pij_j;
  const double* bin = h.pbin[hi_side ? 1 : 0];
  const double xs = hi_side ? 1.0 - s.xstar : s.xstar, a = hi_side ? s.abar : s.beta;
  const double root = wave_bisect(a > 0.0 && a < xs, xs / (xs - a), [&](double mid) {
#pragma clang fp contract(off)
    return sched::pij_eval_tab(i, j, bin, xs * (1.0 - mid)) -
           sched::pij_eval_tab(i, j, bin, xs - mid * (xs - a));
  });
  const double lo = __shfl(root, 0), hi = __shfl(root, 32);
  return lo < hi ? lo : hi;
}

// Set up the next product of a P_{m,m} iteration once the previous one finished:
// P(1/2 + v) = 1/2 + v r(v^2), v = a (X - I/2), W = v^2.  After W: T = r_m W^2 + r_{m-1} W
// + r_{m-2} I from W.W; then T <- W.T + r_k I down to k = 0; then X_new = 1/2 I + v T.
__device__ __forceinline__ void pmm_next(SnfScalars* s, const SnfTables* t) {
#pragma clang fp contract(off)
  const int m = s->pmm_m;
  const double* r = t->pr;
  const int ta = (s->cur + 2) & 3, tb = (s->cur + 3) & 3;
  s->want_e = 0;
  if (s->kind == kKindSquare) {             // W done: first Horner level from W.W
    s->kind = kKindHorner;
    s->ia = s->ib = s->ix = s->bw;
    s->io = s->bt = ta;
    s->c2 = r[m];
    s->c1 = r[m - 1];
    s->c0 = r[m - 2];
    return;
  }
  if (s->kind == kKindHorner && s->horner_left > 0) {   // T <- W.T + r_k I
    const int k = s->horner_left - 1;
    s->ia = s->bw;
    s->ib = s->ix = s->bt;
    s->io = (s->bt == ta) ? tb : ta;
    s->bt = s->io;
    s->c2 = 1.0;
    s->c1 = 0.0;
    s->c0 = r[k];
    return;
  }
  // T = r(W) done: X_new = a X.T - (a / 2) T + I / 2, written over W
  s->kind = kKindFinal;
  s->ia = s->cur;
  s->ib = s->ix = s->bt;
  s->io = s->bw;
  s->c2 = s->alpha;
  s->c1 = -0.5 * s->alpha;
  s->c0 = 0.5;
}

// Set up the next product of a P_{i,j} iteration: P(x* + v) = x* + v Q(v), v = a (X - x* I),
// W = v^2, Q(v) = sum_k (q_2k + q_(2k+1) v) W^k.  The first product gave W and the top level
// T; then T <- T.W + q_(2k+1) V + q_2k I for k = h - 2 .. 0; then X_new = x* I + V T.
__device__ __forceinline__ void pij_next(SnfScalars* s, const SnfTables* t) {
#pragma clang fp contract(off)
  const double a = s->alpha, xs = s->xstar;
  const int ta = (s->cur + 2) & 3, tb = (s->cur + 3) & 3;
  s->want_e = 0;
  s->dual = 0;
  if (s->horner_left > 0) {
    const int k = s->horner_left - 1;
    s->kind = kKindHorner;
    s->ia = s->bt;
    s->ib = s->bw;
    s->ix = s->cur;
    s->io = (s->bt == ta) ? tb : ta;
    s->bt = s->io;
    s->c2 = 1.0;
    s->c1 = t->pq[2 * k + 1] * a;
    s->c0 = t->pq[2 * k] - t->pq[2 * k + 1] * a * xs;
    return;
  }
  // X_new = a X.T - a x* T + x* I, written over W
  s->kind = kKindFinal;
  s->ia = s->cur;
  s->ib = s->ix = s->bt;
  s->io = s->bw;
  s->c2 = a;
  s->c1 = -(a * xs);
  s->c0 = xs;
}

__device__ __forceinline__ void finish(SnfScalars* s, const SnfConfig* c, int status) {
  if ((status == SNF_OK || status == SNF_OK_FLOOR) && c->has_nocc) {
    const double err = s->t1 - (double)c->n_occ;
    if (fabs(err) >= 0.5) status = SNF_EMIXED;
  }
  s->status = status;
  s->stop = 1;
}

// The scalar state machine, run by one thread on a copy of the state's header in LDS (s).  It
// and what it calls are inlined: as calls they took the header through flat addresses and a
// stack in scratch memory (a one-workgroup solve of order 64: 186 us, inlined 158).
// the per-iteration log record goes straight to memory (log; not written when null).
__device__ __forceinline__ void schedule_scalars(SnfScalars* __restrict__ s,
                                                 const SnfConfig* __restrict__ c,
                                                 const SnfTables* __restrict__ t,
                                                 snf_log_rec* __restrict__ log, double e2,
                                                 double t1, double t2, int init, double root) {
  if (init) {
    s->t1 = t1;
    s->t2 = t2;
    decide(s, c, t, root);
    return;
  }
  s->products += 1;
  const int f64 = s->prec == kPrecF64 ? 1 : 0;
  s->products_f64 += f64;
  s->products_lowp += 1 - f64;
  if (s->kind == kKindSquare) {
    const double e = sqrt(e2);
    s->e_last = e;
    const int it = s->iter;
    snf_log_rec* rec = log ? &log[it < SNF_LOG_MAX ? it : SNF_LOG_MAX - 1] : nullptr;
    if (rec) {
      rec->i = it;
      rec->branch = s->branch;
      rec->precision = s->prec;
      rec->reserved = s->phase;
      rec->alpha = s->alpha;
      rec->beta = s->beta;
      rec->betabar = s->betabar;
      rec->e = e;
      rec->t1 = s->t1;
      rec->t2 = s->t2;
    }
    s->nlog = it + 1;
    s->e_hist[2] = s->e_hist[1];
    s->e_hist[1] = s->e_hist[0];
    s->e_hist[0] = e;
    if (!isfinite(e)) { if (rec) rec->branch = -1; finish(s, c, SNF_ENONFINITE); return; }
    if (e <= c->tol) { if (rec) rec->branch = -1; finish(s, c, SNF_OK); return; }
    if (s->phase == kPhaseLow && c->mode == SNF_P_FP32 && it >= 2) {
      // floor of the FP32-only mode: stop once the predicted error is below the floor
      // parameter and the measured idempotency stopped shrinking
      const double bound = s->beta > 1.0 - s->betabar ? s->beta : 1.0 - s->betabar;
      if (bound <= c->lowp_floor && e > 0.5 * s->e_hist[2]) {
        if (rec) rec->branch = -1;
        finish(s, c, SNF_OK_FLOOR);
        return;
      }
    }
    if (it >= c->max_iter) { if (rec) rec->branch = -1; finish(s, c, SNF_ENOCONV); return; }
    if (s->pmm_m) {
      pmm_next(s, t);
      return;
    }
    if (s->pij_i) {
      pij_next(s, t);
      return;
    }
    if (s->branch == SNF_BRANCH_P11) {
      // second product of Algorithm 1: R = S2.X; X_new = (3 - 2c) S2 - 2 a R
      const double a = s->alpha, sh = 0.5 * (1.0 - a);
      s->kind = kKindCube;
      s->want_e = 0;
      s->c2 = -2.0 * a;
      s->c1 = 3.0 - 2.0 * sh;
      s->c0 = 0.0;
      s->ia = 2;            // S2
      s->ib = s->cur;       // X
      s->ix = 2;
      s->io = 1 - s->cur;
      return;
    }
    advance_beta(s, t, s->branch, s->alpha);
    s->iter = it + 1;
    s->cur = s->io;
    s->t1 = t1;
    s->t2 = t2;
    decide(s, c, t, root);
  } else if (s->kind == kKindHorner) {
    s->horner_left -= 1;
    if (s->pij_i) pij_next(s, t); else pmm_next(s, t);
  } else {                                  // kKindCube or kKindFinal: X_new is complete
    advance_beta(s, t, s->branch, s->alpha);
    s->iter += 1;
    s->cur = s->io;
    s->t1 = t1;
    s->t2 = t2;
    decide(s, c, t, root);
  }
}

// The same on a header in LDS: its scalars go to registers and back, as the state machine would
// otherwise wait for a chain of single LDS reads.
__device__ __forceinline__ void schedule_step(SnfHeader* __restrict__ hs,
                                              snf_log_rec* __restrict__ log, double e2, double t1,
                                              double t2, int init, double root) {
  SnfScalars sc = *hs;
  const SnfConfig cf = *hs;
  schedule_scalars(&sc, &cf, hs, log, e2, t1, t2, init, root);
  *static_cast<SnfScalars*>(hs) = sc;
}

// Reduce the partial sums in a fixed order, then advance the scalar state.  The state's
// header (everything before the log) is staged in LDS by all threads, advanced there by
// thread 0 and written back by all threads: one pass of coalesced accesses instead of a
// chain of dependent single-thread loads and stores to device memory.
__device__ __forceinline__ void schedule_body(SnfState* __restrict__ sg,
                                              const double* __restrict__ partials, int count,
                                              int init, SnfHeader* __restrict__ host,
                                              int32_t* __restrict__ progress = nullptr,
                                              int done = 0) {
  __shared__ double red[24];
  __shared__ __attribute__((aligned(16))) SnfHeader hs;
  static_assert(sizeof(SnfHeader) % 4 == 0, "copied by words");
  constexpr int words = (int)(sizeof(SnfHeader) / 4);
  unsigned* hb = (unsigned*)&hs;
  unsigned* gb = (unsigned*)(SnfHeader*)sg;
  for (int i = threadIdx.x; i < words; i += kReduceThreads) hb[i] = gb[i];
  double e2 = 0.0, t1 = 0.0, t2 = 0.0;
  for (int i = threadIdx.x; i < count; i += kReduceThreads) {
    e2 += partials[i * 4 + 0];
    t1 += partials[i * 4 + 1];
    t2 += partials[i * 4 + 2];
  }
  // one thread tells the host, ahead of the schedule: the store's way to host memory (1.5 us at
  // the end of the kernel) passes beside it
  const bool teller = progress && threadIdx.x == kReduceThreads - 64;
  if (teller) __hip_atomic_store(progress, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  block_sum3(e2, t1, t2, red);             // its barrier also publishes the header copy
  if (threadIdx.x < 64) {
    const double root = schedule_root(hs, init);
    if (threadIdx.x == 0) schedule_step(&hs, sg->log, e2, t1, t2, init, root);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < words; i += kReduceThreads) {
    gb[i] = hb[i];
    if (host) ((unsigned*)host)[i] = hb[i];
  }
  if (teller && hs.stop)
    __hip_atomic_store(progress, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------------------
// Direct step: FP64 solves whose upper triangle is covered by at most one TxT tile per compute
// unit (T = 32 .. 96).  A 128x128 engine has too few tiles there: it cut them into k-slices,
// added the slices in a second kernel and advanced the state in a third, and at n = 1000 the
// three took 27 + 13 + 5 us a product of 17 us of matrix-core work.  Here
//  * the k range is split over the four waves of a workgroup, each with the whole tile in its
//    accumulators, so nothing is shared until the end: no LDS staging and no barrier in the main
//    loop, operands go from L2 straight to registers, PD k-steps ahead;
//  * the four partial tiles are added in LDS in wave order, a band of 32 rows at a time;
//  * the schedule of step s runs at the head of step s + 1, in every workgroup for itself, beside
//    the product: the host knows which buffers a step reads.
// The bound is the matrix cores (FP64: 64 cycles an instruction and SIMD) plus, per step, about
// 6 us of launch boundary, cold operand loads and epilogue.
// A scale-and-fold solve of 19 products (wall time), this against the engine's three kernels (n
// > 896), 32x32 tiles and a schedule kernel (256 < n <= 896), those in one cooperative launch
// with grid barriers (n <= 256): n = 256 0.27 / 0.43 ms, 400 0.32 / 0.58, 704 0.45 / 0.88, 1056
// 0.77 / 1.26, 1408 1.25 / 1.92, 1760 2.03 / 3.07, 2112 3.19 / 4.46.  A step at n = 256 takes 8 us: 1.7
// until the operands are there (the schedule, 2.5 us from its sums on, beside the 3 us of
// products), 2 the epilogue, 2 to the next launch's first instruction.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double* pick_buf(const Buffers& b, int i) {
  double* p = b.x[0];
  if (i == 1) p = b.x[1];
  if (i == 2) p = b.x[2];
  if (i == 3) p = b.x[3];
  return p;
}

// Operand registers of PD k-steps for a tile side of TB 16-blocks.  Lane (fr, fk) = (l % 16,
// l / 16) loads row k + fk of the operand (A[i][k] = A[k][i] by symmetry): columns 2 fr, 2 fr + 1
// of each 32 (16-byte loads; block 2 p holds the even columns of pair p, block 2 p + 1 the odd
// ones) and, for odd TB, column fr of the last 16.
template <int TB, int PD>
struct DirectOperand {
  static constexpr int P = TB / 2, O = TB & 1;
  u32x4 pair[PD][P > 0 ? P : 1];
  double last[PD];
  __device__ __forceinline__ void load(const double* rowptr, int slot) {
    const int fr = threadIdx.x & 15;
#pragma unroll
    for (int p = 0; p < P; ++p) pair[slot][p] = gload16(rowptr + 32 * p + 2 * fr);
    if constexpr (O)
      last[slot] = *(const __attribute__((address_space(1))) double*)(rowptr + 32 * P + fr);
  }
  __device__ __forceinline__ double get(int slot, int m) const {
    if (O && m == TB - 1) return last[slot];
    const u32x4 v = pair[slot][m >> 1];
    const unsigned lo = (m & 1) ? v[2] : v[0], hi = (m & 1) ? v[3] : v[1];
    return __hiloint2double((int)hi, (int)lo);
  }
};

// Combination, sums and stores of one tile: bands of 32 rows (one pair of block rows; the last 16
// rows for odd TB): add the four partial tiles in wave order, combine, store the rows, then the
// mirror from LDS so that its stores are contiguous too.  load_x(p) fetches band p of the linear
// term into xs (band 0 is there already).
struct DirectOut {
  double* Y;
  double* Y2;              // second output, or null
  void* lp;                // low-precision copy of Y (LOWP), of kind lowp_kind (-1: none)
  int lowp_kind, n;
  int64_t ld;
  double c2, c1, c0, d2, d1, d0;
};

__device__ __forceinline__ void direct_lowp(const DirectOut& o, int64_t at, double y) {
  if (o.lowp_kind == kPrecF32) ((float*)o.lp)[at] = (float)y;
  else if (o.lowp_kind == kPrecBF16) ((unsigned short*)o.lp)[at] = f32_to_bf16_rne((float)y);
}

template <int TB, int NC, bool LOWP, int PR, int NE, typename LoadX>
__device__ __forceinline__ void direct_bands(const dbl4 (&acc)[TB][TB / NC],
                                             double (&part)[4][PR][16 * TB + 2], double2 (&xs)[NE],
                                             LoadX load_x, const DirectOut& o, int64_t i0,
                                             int64_t j0, bool worker, double& e2, double& t1,
                                             double& t2) {
  constexpr int T = 16 * TB, QB = TB / NC, NT = kDirectThreads * NC, W2 = T / 2;
  constexpr int P = TB / 2, O = TB & 1, QP = QB / 2, QO = QB & 1;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 15, fk = lane >> 4, kq = wid & 3, cg = wid >> 2;
  const bool diag = i0 == j0;
#pragma unroll
  for (int p = 0; p < P + O; ++p) {
    const int rows = p < P ? 32 : 16;
    if (worker) {
#pragma unroll
      for (int mm = 0; mm < (p < P ? 2 : 1); ++mm) {
        const int m = 2 * p + mm;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int t = fk + 4 * v, r = p < P ? 2 * t + mm : t;
#pragma unroll
          for (int q = 0; q < QP; ++q)
            *(double2*)(&part[kq][r][cg * 16 * QB + 32 * q + 2 * fr]) =
                double2{acc[m][2 * q][v], acc[m][2 * q + 1][v]};
          if (QO) part[kq][r][cg * 16 * QB + 32 * QP + fr] = acc[m][QB - 1][v];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int idx = e * NT + tid, r = idx / W2, c = 2 * (idx % W2);
      if (!worker || r >= rows) continue;
      const int gr = (int)i0 + 32 * p + r, gc = (int)j0 + c;
      double y[2], y2[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double pr = ((part[0][r][c + h] + part[1][r][c + h]) + part[2][r][c + h]) +
                          part[3][r][c + h];
        const double x = h ? xs[e].y : xs[e].x;
        const bool on = gr == gc + h, in = gr < o.n && gc + h < o.n;
        y[h] = in ? o.c2 * pr + o.c1 * x + (on ? o.c0 : 0.0) : 0.0;
        y2[h] = in ? o.d2 * pr + o.d1 * x + (on ? o.d0 : 0.0) : 0.0;
        if (!diag || gr <= gc + h) {       // (a diagonal tile keeps its upper half)
          const double w = on ? 1.0 : 2.0, d = pr - x;
          e2 += w * (d * d);
          t2 += w * (y[h] * y[h]);
          if (on) t1 += y[h];
          if (diag) {
            o.Y[(int64_t)gr * o.ld + gc + h] = y[h];
            if (o.Y2) o.Y2[(int64_t)gr * o.ld + gc + h] = y2[h];
            if (LOWP) direct_lowp(o, (int64_t)gr * o.ld + gc + h, y[h]);
          }
        }
      }
      if (!diag) {
        *(double2*)(o.Y + (int64_t)gr * o.ld + gc) = double2{y[0], y[1]};
        if (o.Y2) *(double2*)(o.Y2 + (int64_t)gr * o.ld + gc) = double2{y2[0], y2[1]};
        if (LOWP) {
          direct_lowp(o, (int64_t)gr * o.ld + gc, y[0]);
          direct_lowp(o, (int64_t)gr * o.ld + gc + 1, y[1]);
        }
      }
      *(double2*)(&part[0][r][c]) = double2{y[0], y[1]};   // (this thread's own entries)
      if (o.Y2) *(double2*)(&part[1][r][c]) = double2{y2[0], y2[1]};
    }
    if (p + 1 < P + O) load_x(p + 1);   // (a band ahead)
    __syncthreads();
    for (int idx = worker ? tid : rows * T; idx < rows * T; idx += NT) {
      const int r = idx % rows, c = idx / rows;
      const int gr = (int)i0 + 32 * p + r, gc = (int)j0 + c;
      if (diag && gr >= gc) continue;
      o.Y[(int64_t)gc * o.ld + gr] = part[0][r][c];
      if (o.Y2) o.Y2[(int64_t)gc * o.ld + gr] = part[1][r][c];
      if (LOWP) direct_lowp(o, (int64_t)gc * o.ld + gr, part[0][r][c]);
    }
    if (p + 1 < P + O) __syncthreads();
  }
}

// NC: column groups of the tile; four waves (the k quarters) for each, so that a wave holds
// TB x TB / NC blocks.  SW: one more wave, which runs the schedule beside the product (where the
// registers allow it; else wave 0 does, ahead of its share).  The product needs the schedule's
// result only in its epilogue, as the operands are known beforehand; a flag in LDS stops the
// waves early once the schedule has stopped the solve.
template <int TB, int NC, int PD, bool SW>
__global__ __launch_bounds__(kDirectThreads* NC + (SW ? 64 : 0)) void direct_step_kernel(
    DirectArgs g, int step, int pa, int pb, int px) {
  constexpr int T = 16 * TB, QB = TB / NC, NT = kDirectThreads * NC;
  static_assert(QB * NC == TB, "equal column groups");
  // The rounding of a sum grows with the terms that go to one running sum.  A quarter's terms go to
  // S of them in turn, or where the registers do not hold more accumulators to one in PH phases,
  // each then added to the phases before: at most n / 16 terms a sum (T = 32), n / 16 + 28 (48) and
  // n / 8 + 28 (64), as few as in the engine's up to 16 k-slices.  With one sum a quarter |D -
  // D_exact|_F was up to 1.6 times the engine's (scaled P_{1,3}, n = 512: 2.15e-13, engine 1.36e-13,
  // this 1.26e-13; Algorithm 1, n = 1000: 1.98e-13, 1.53e-13, 1.23e-13), at the same time within
  // 1%.  From T = 80 on the engine had two or three slices.
  constexpr int S = TB == 2 ? 4 : 1, PH = TB == 3 ? 4 : TB == 4 ? 2 : 1;
  static_assert(S == 1 || S == 4, "added by pairs");
  constexpr int P = TB / 2, LW = T + 2;
  constexpr int SWAVE = SW ? 4 * NC : 0;
  // the product starts ahead of the schedule; the largest tiles wait for it, as their product
  // takes 20 times as long and the look at the flag costs their loop more (n = 1760: 5%)
  constexpr bool EARLY = TB <= 4;
  __shared__ __attribute__((aligned(16))) SnfHeader hs;
  __shared__ double red[3 * 9];
  __shared__ int stopped;                  // set by the schedule, looked at between k-steps
  // (more than half of a compute unit's LDS: two workgroups on one unit would leave another idle)
  constexpr int PR = 4 * 32 * LW * 8 > (82 << 10) ? 32 : (82 << 10) / (4 * LW * 8) + 1;
  __shared__ __attribute__((aligned(16))) double part[4][PR][LW];
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool worker = !SW || wid != SWAVE;
  const int fr = lane & 15, fk = lane >> 4;
  const int kq = wid & 3, cg = wid >> 2;                // k quarter, column group
  const int64_t ld = g.ld;
  const int tiles = g.nt * (g.nt + 1) / 2;
  const int tile = xcd_remap(blockIdx.x, tiles);
  int bi, bj;
  tile_coords(tile, g.nt, 1, bi, bj);
  const int64_t i0 = (int64_t)bi * T, j0 = (int64_t)bj * T;

  const SnfHeader* hd = g.hdr + (step & 1);
  if (tid == 0) stopped = 0;
  if (hd->stop) {
    // a launch after the stop: hand the state on
    if (blockIdx.x == 0) {
      const unsigned* gh = (const unsigned*)hd;
      unsigned* gn = (unsigned*)(g.hdr + ((step + 1) & 1));
      for (int i = tid; i < (int)(sizeof(SnfHeader) / 4); i += blockDim.x) gn[i] = gh[i];
    }
    return;
  }
  __syncthreads();

  // the schedule of the step before (step 0: the first decision), by one wave
  constexpr int HW = (int)(sizeof(SnfHeader) / 4), HL = (HW + 63) / 64;
  static_assert(sizeof(SnfHeader) % 4 == 0, "copied by words");
  unsigned hw[HL];
  double e2 = 0.0, t1 = 0.0, t2 = 0.0;
  if (wid == SWAVE) {
    // header and sums ahead of any operand: loads return in order
    const unsigned* gh = (const unsigned*)hd;
#pragma unroll
    for (int i = 0; i < HL; ++i) hw[i] = i * 64 + lane < HW ? gh[i * 64 + lane] : 0u;
    const int count = step ? tiles : kDirectF0Blocks;
    const double* ps = g.partials + (size_t)((step + 1) & 1) * kDirectSlots * 4;
#pragma unroll
    for (int i = 0; i < kDirectThreads / 64; ++i) {
      const int q = i * 64 + lane;
      if (q < count) {
        e2 += ps[q * 4 + 0];
        t1 += ps[q * 4 + 1];
        t2 += ps[q * 4 + 2];
      }
    }
  }
  auto schedule = [&]() {
#pragma unroll
    for (int i = 0; i < HL; ++i)
      if (i * 64 + lane < HW) ((unsigned*)&hs)[i * 64 + lane] = hw[i];
    e2 = wave_sum_rows(e2);
    t1 = wave_sum_rows(t1);
    t2 = wave_sum_rows(t2);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // (FP64 instructions share the matrix cores' units with the other waves' products)
    __builtin_amdgcn_s_setprio(3);
    const double root = schedule_root(hs, step == 0);
    if (lane == 0) {
      schedule_step(&hs, blockIdx.x == 0 ? g.log : nullptr, e2, t1, t2, step == 0, root);
      // the product under way reads the buffers that the host named: another choice is an error
      if (!hs.stop && (hs.ia != pa || hs.ib != pb || hs.ix != px)) {
        hs.status = SNF_EDEVICE;
        hs.stop = 1;
      }
      if (hs.stop) *(volatile int*)&stopped = 1;
    }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (blockIdx.x == 0) {
      unsigned* gn = (unsigned*)(g.hdr + ((step + 1) & 1));
#pragma unroll
      for (int i = 0; i < HL; ++i)
        if (i * 64 + lane < HW) gn[i * 64 + lane] = ((const unsigned*)&hs)[i * 64 + lane];
      if (lane == 0 && g.progress)
        __hip_atomic_store(g.progress, hs.stop ? -1 : step + 1, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
  };

  // the wave's k-steps (4 values of k each); rows n .. ld - 1 of the buffers are zero
  const int KT = (int)((g.n + 3) / 4);
  const int kb = kq * KT / 4, ke = (kq + 1) * KT / 4;
  dbl4 acc[S][TB][QB];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int m = 0; m < TB; ++m)
#pragma unroll
        for (int q = 0; q < QB; ++q) acc[i][m][q] = dbl4{0.0, 0.0, 0.0, 0.0};
  };
  clear();
  DirectOperand<TB, PD> A;
  DirectOperand<QB, PD> B;
  auto load = [&](const double* Ap, const double* Bp, int ks, int slot) {
    const int64_t off = (int64_t)(4 * min(ks, max(ke - 1, kb)) + fk) * ld;
    A.load(Ap + off + i0, slot);
    B.load(Bp + off + j0 + cg * 16 * QB, slot);
  };
  auto compute = [&](int slot) {
#pragma unroll
    for (int m = 0; m < TB; ++m)
#pragma unroll
      for (int q = 0; q < QB; ++q)
        acc[slot % S][m][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(
            A.get(slot, m), B.get(slot, q), acc[slot % S][m][q], 0, 0, 0);
  };
  dbl4 tot[PH > 1 ? TB : 1][PH > 1 ? QB : 1];           // sums of the phases before this one
#pragma unroll
  for (int m = 0; m < (PH > 1 ? TB : 1); ++m)
#pragma unroll
    for (int q = 0; q < (PH > 1 ? QB : 1); ++q) tot[m][q] = dbl4{0.0, 0.0, 0.0, 0.0};
  // the linear term's values of a band of 32 rows; the first band's ahead of the product where
  // the registers allow it
  constexpr bool XA = TB <= 4;
  constexpr int W2 = T / 2, NE = 32 * W2 / NT;           // column pairs per row, per thread
  double2 xs[NE];
  auto load_x = [&](const double* X, int p) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int idx = e * NT + tid, r = idx / W2, c = 2 * (idx % W2);
      if (worker && r < (p < P ? 32 : 16))
        xs[e] = *(const double2*)(X + (i0 + 32 * p + r) * ld + j0 + c);
    }
  };
  if (worker) {
    const double *Ap = pick_buf(g.bufs, pa), *Bp = pick_buf(g.bufs, pb);
#pragma unroll
    for (int u = 0; u < PD; ++u) load(Ap, Bp, kb + u, u);
    if (XA) load_x(pick_buf(g.bufs, px), 0);
    __builtin_amdgcn_sched_barrier(0);
    if (!SW && wid == SWAVE) schedule();
    if constexpr (!EARLY) {
      __syncthreads();
      if (hs.stop) return;
    }
    int ks = kb;
    auto steps = [&](int end) {
      for (; ks + PD <= end; ks += PD) {
        if (EARLY && *(volatile int*)&stopped) break;
        // (past the end the last k-step again, never used: the number of loads in flight is the
        // same on every path, so a wait leaves the newer ones in flight)
#pragma unroll
        for (int u = 0; u < PD; ++u) {
          compute(u);
          load(Ap, Bp, ks + u + PD, u);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    if constexpr (PH > 1) {
      const int span = ((ke - kb + PH - 1) / PH + PD - 1) / PD * PD;
#pragma unroll 1
      for (int end = kb + span; end < ke; end += span) {
        steps(end);
#pragma unroll
        for (int m = 0; m < TB; ++m)
#pragma unroll
          for (int q = 0; q < QB; ++q) tot[m][q] += acc[0][m][q];
        clear();
      }
    }
    steps(ke);
#pragma unroll
    for (int u = 0; u < PD; ++u)
      if (ks + u < ke) compute(u);
  } else {
    schedule();
  }
  __syncthreads();
  if (hs.stop) return;

  // the wave's sums of its quarter
#pragma unroll
  for (int m = 0; m < TB; ++m)
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      if constexpr (S == 4)
        acc[0][m][q] = (acc[0][m][q] + acc[1][m][q]) + (acc[2][m][q] + acc[3][m][q]);
      if constexpr (PH > 1) acc[0][m][q] += tot[m][q];
    }

  // the tile's results
  const double* X = pick_buf(g.bufs, px);
  if (!XA) load_x(X, 0);
  DirectOut o;
  o.Y = pick_buf(g.bufs, __builtin_amdgcn_readfirstlane(hs.io));
  o.Y2 = __builtin_amdgcn_readfirstlane(hs.dual)
             ? pick_buf(g.bufs, __builtin_amdgcn_readfirstlane(hs.io2)) : nullptr;
  o.lp = nullptr;
  o.lowp_kind = -1;
  o.n = (int)g.n;
  o.ld = ld;
  o.c2 = hs.c2;
  o.c1 = hs.c1;
  o.c0 = hs.c0;
  o.d2 = hs.d2;
  o.d1 = hs.d1;
  o.d0 = hs.d0;
  e2 = t1 = t2 = 0.0;
  direct_bands<TB, NC, false>(acc[0], part, xs, [&](int p) { load_x(X, p); }, o, i0, j0, worker, e2,
                              t1, t2);
  e2 = wave_sum_rows(e2);
  t1 = wave_sum_rows(t1);
  t2 = wave_sum_rows(t2);
  if (lane == 0) {
    red[wid * 3 + 0] = e2;
    red[wid * 3 + 1] = t1;
    red[wid * 3 + 2] = t2;
  }
  __syncthreads();
  if (tid < 3) {                           // (waves in order)
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) sum += red[w * 3 + tid];
    g.partials[((size_t)(step & 1) * kDirectSlots + tile) * 4 + tid] = sum;
  }
}

// X_0 = f_0(F) on the whole ld x ld buffer (zero beyond n), upper triangle of F read, as
// f0_kernel; block partials into parity 1, where step 0 looks for them.
__global__ __launch_bounds__(256) void direct_f0_kernel(DirectArgs g, SnfHeader h,
                                                        const double* __restrict__ F, int64_t ldf) {
  __shared__ double tile[32][33];
  __shared__ double red[24];
  if (blockIdx.x == 0 && threadIdx.x == 0) g.hdr[0] = h;
  const int alg1 = h.scheme == SNF_MCWEENY || h.scheme == SNF_SNF_FIXMU || h.pmm_m || h.pij_i;
  const double lmin = h.lambda_min, lmax = h.lambda_max, mu = h.mu, gamma = h.gamma, xs = h.xstar;
  double* X = g.bufs.x[0];
  const int n = (int)g.n, ld = (int)g.ld, nt = (ld + 31) / 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  double t1 = 0.0, t2 = 0.0;
  for (int t = blockIdx.x; t < nt * nt; t += gridDim.x) {
    const int bi = t / nt, bj = t % nt, si = min(bi, bj), sj = max(bi, bj);
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int gr = si * 32 + r, gc = sj * 32 + tx;
      tile[r][tx] = (gr < n && gc < n) ? F[(int64_t)gr * ldf + gc] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int gr = bi * 32 + r, gc = bj * 32 + tx;
      if (gr >= ld || gc >= ld) continue;
      const double v = (gr <= gc) ? tile[r][tx] : tile[tx][r];
      double x = 0.0;
      if (gr < n && gc < n) {
        const bool d = gr == gc;
        x = alg1 ? ((d ? mu : 0.0) - v) / gamma + (d ? xs : 0.0)
                 : ((d ? lmax : 0.0) - v) / (lmax - lmin);
        if (d) t1 += x;
        t2 += x * x;
      }
      X[(int64_t)gr * ld + gc] = x;
    }
  }
  double e0 = 0.0;
  block_sum3(e0, t1, t2, red);
  if (threadIdx.x == 0) {
    double* po = g.partials + ((size_t)kDirectSlots + blockIdx.x) * 4;
    po[0] = 0.0;
    po[1] = t1;
    po[2] = t2;
  }
}

// D = X_cur and the final state out (host-visible memory: no copy engine and no extra launch).
__global__ __launch_bounds__(256) void direct_out_kernel(DirectArgs g, int slot,
                                                         double* __restrict__ D, int64_t ldd,
                                                         SnfState* __restrict__ out) {
  const SnfHeader* h = g.hdr + slot;
  const double* X = pick_buf(g.bufs, h->cur);
  const int n = (int)g.n;
  for (int r = blockIdx.x; r < n; r += gridDim.x)
    for (int c = threadIdx.x; c < n; c += 256) D[r * ldd + c] = X[(int64_t)r * g.ld + c];
  if (blockIdx.x == 0) {
    unsigned* o = (unsigned*)(SnfHeader*)out;
    for (int i = threadIdx.x; i < (int)(sizeof(SnfHeader) / 4); i += 256) o[i] = ((const unsigned*)h)[i];
    const int words = min(h->nlog, SNF_LOG_MAX) * (int)(sizeof(snf_log_rec) / 4);
    unsigned* ol = (unsigned*)out->log;
    for (int i = threadIdx.x; i < words; i += 256) ol[i] = ((const unsigned*)g.log)[i];
  }
}

void launch_direct_f0(const DirectArgs& a, const SnfHeader& h, const double* F, int64_t ldf,
                      hipStream_t s) {
  hipLaunchKernelGGL(direct_f0_kernel, dim3(kDirectF0Blocks), dim3(256), 0, s, a, h, F, ldf);
}

void launch_direct_step(int tile, const DirectArgs& a, int step, const int (&op)[3],
                        hipStream_t s) {
  const dim3 grid(a.nt * (a.nt + 1) / 2);
#define SNF_DIRECT(TB, NC, PD, SW)                                                          \
  hipLaunchKernelGGL((direct_step_kernel<TB, NC, PD, SW>), grid,                            \
                     dim3(kDirectThreads * NC + (SW ? 64 : 0)), 0, s, a, step, op[0],  \
                     op[1], op[2])
  switch (tile) {
    case 32: SNF_DIRECT(2, 1, 8, true); break;
    case 48: SNF_DIRECT(3, 1, 7, true); break;
    case 64: SNF_DIRECT(4, 2, 7, false); break;
    case 80: SNF_DIRECT(5, 1, 6, false); break;
    default: SNF_DIRECT(6, 2, 4, false); break;
  }
#undef SNF_DIRECT
}

void launch_direct_out(const DirectArgs& a, int slot, double* D, int64_t ldd, SnfState* out,
                       hipStream_t s) {
  hipLaunchKernelGGL(direct_out_kernel, dim3((unsigned)(a.n < 1024 ? a.n : 1024)), dim3(256), 0, s,
                     a, slot, D, ldd, out);
}

// The buffer sequence of decide(), pmm_next() and pij_next().
void StepOperands::next(int (&op)[3]) {
  const bool pij = scheme_is_pij(scheme), chain = scheme_pmm_m(scheme) || pij;
  const int bw = (cur + 1) & 3, ta = (cur + 2) & 3, tb = (cur + 3) & 3;
  auto set = [&](int a, int b, int x) {
    op[0] = a;
    op[1] = b;
    op[2] = x;
  };
  if (k == 0) {                            // X.X
    set(cur, cur, cur);
    bt = ta;
  } else if (!chain) {                     // S2.X
    set(2, cur, 2);
  } else if (k == per_it - 1) {            // X.T
    set(cur, bt, bt);
  } else if (pij) {                        // T <- T.W
    set(bt, bw, cur);
    bt = bt == ta ? tb : ta;
  } else if (k == 1) {                     // T from W.W
    set(bw, bw, bw);
  } else {                                 // T <- W.T
    set(bw, bt, bt);
    bt = bt == ta ? tb : ta;
  }
  if (++k == per_it) {
    k = 0;
    cur = chain ? bw : 1 - cur;
  }
}

// ---------------------------------------------------------------------------------------
// The smallest orders: the whole solve in one workgroup, the iterates in LDS (160 KB: two
// buffers up to order 80, four up to 64).  A step of such a solve is bound by
// latency, so nothing leaves the compute unit between steps: no launch, no grid barrier, no
// memory.  Eight waves share the 16x16 blocks of the upper triangle; a step's results stay in
// registers until the sums are known, so X needs no second buffer and is still whole when the
// stop test passes.  A step at n = 64 takes 4.5 us: 2.3 the products, 0.4 the sums, 1.4 the
// schedule, 0.4 the writes.  The 19 products of the solves above at n = 17 / 40 / 64 / 80: 0.10 /
// 0.11 / 0.13 / 0.16 ms, against 0.37 ms in a cooperative launch of 32x32 tiles.  Above order 80 the
// direct steps take over (at 96, with a third block for some waves, such a solve took 0.23 ms
// against their 0.22).
// ---------------------------------------------------------------------------------------
constexpr int kWgThreads = 512, kWgWaves = kWgThreads / 64;
constexpr int kWgMaxBlocks = 5;          // 16x16 blocks a side

static int wg_buffers(int scheme) {
  if (scheme_pmm_m(scheme) || scheme_is_pij(scheme)) return 4;
  return (scheme == SNF_MCWEENY || scheme == SNF_SNF_FIXMU) ? 2 : 1;
}

size_t solve_wg_bytes(int64_t n, int scheme) {
  if (n > 16 * kWgMaxBlocks) return 0;
  const int64_t np = (n + 15) / 16 * 16;
  const size_t bytes = (size_t)wg_buffers(scheme) * np * np * sizeof(double);
  return bytes <= (size_t)144 << 10 ? bytes : 0;
}

// NB buffers: 1: X in place; 2: X, S2 (index 2); 4: by index.
template <int NB>
__global__ __launch_bounds__(kWgThreads) void solve_wg_kernel(SnfHeader h,
                                                              const double* __restrict__ F,
                                                              int64_t ldf, double* __restrict__ D,
                                                              int64_t ldd, SnfState* __restrict__ out,
                                                              int max_steps) {
  constexpr int MB = 2;                    // blocks per wave at the largest order
  static_assert(kWgMaxBlocks * (kWgMaxBlocks + 1) / 2 <= MB * kWgWaves, "every block has a wave");
  extern __shared__ __attribute__((aligned(16))) double xbuf[];
  __shared__ __attribute__((aligned(16))) SnfHeader hs;
  __shared__ double red[3 * kWgWaves];
  const int n = (int)h.n, np = (n + 15) / 16 * 16;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int fr = lane & 15, fk = lane >> 4;
  // The columns of row r are permuted within each 16 by r mod 16 (a mirrored write of 16 rows of
  // one column then touches every bank once, as 16 columns of one row do), and odd rows swap 16
  // by 16 where rows are a multiple of 256 B apart (two rows of 16 values then cover the banks
  // once).  Unpermuted, the writes took 1.1 us a step at order 64 and 2.3 at 96.
  const int sw = np % 32 ? 0 : 16;
  auto at = [&](int r, int c) { return r * np + (c ^ ((r & 15) | ((r & 1) ? sw : 0))); };
  auto buf = [&](int i) {
    return xbuf + (size_t)(NB == 1 ? 0 : NB == 2 ? (i == 2 ? 1 : 0) : i) * np * np;
  };
  auto sum3 = [&](double& a, double& b, double& c) {     // valid in thread 0
    a = wave_sum_rows(a);
    b = wave_sum_rows(b);
    c = wave_sum_rows(c);
    if (lane == 0) {
      red[wid * 3 + 0] = a;
      red[wid * 3 + 1] = b;
      red[wid * 3 + 2] = c;
    }
    __syncthreads();
    if (tid == 0) {
      a = b = c = 0.0;
      for (int w = 0; w < kWgWaves; ++w) {
        a += red[w * 3 + 0];
        b += red[w * 3 + 1];
        c += red[w * 3 + 2];
      }
    }
  };
  double e2 = 0.0, t1 = 0.0, t2 = 0.0;
  {
    if (tid == 0) hs = h;
    const int alg1 = h.scheme == SNF_MCWEENY || h.scheme == SNF_SNF_FIXMU || h.pmm_m || h.pij_i;
    for (int idx = tid; idx < np * np; idx += kWgThreads) {
      const int r = idx / np, c = idx - r * np;
      if (r > c) continue;
      double x = 0.0;
      if (c < n) {
        const double v = F[r * ldf + c];
        const bool d = r == c;
        x = alg1 ? ((d ? h.mu : 0.0) - v) / h.gamma + (d ? h.xstar : 0.0)
                 : ((d ? h.lambda_max : 0.0) - v) / (h.lambda_max - h.lambda_min);
        if (d) t1 += x;
        t2 += (d ? 1.0 : 2.0) * (x * x);
      }
      xbuf[at(r, c)] = x;
      xbuf[at(c, r)] = x;
    }
    sum3(e2, t1, t2);
    if (tid < 64) {
      const double root = schedule_root(hs, 1);
      if (tid == 0) schedule_step(&hs, out->log, e2, t1, t2, 1, root);
    }
    __syncthreads();
  }
  const int nb = np / 16, cnt = nb * (nb + 1) / 2;
  int br[MB], bc[MB];                // the wave's blocks
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    int rem = wid + i * kWgWaves, r = 0;
    while (r < nb && rem >= nb - r) {
      rem -= nb - r;
      ++r;
    }
    br[i] = __builtin_amdgcn_readfirstlane(r);
    bc[i] = __builtin_amdgcn_readfirstlane(r + rem);
  }
  const int mine = __builtin_amdgcn_readfirstlane((cnt - wid + kWgWaves - 1) / kWgWaves);
  for (int step = 0; step < max_steps && !hs.stop; ++step) {
    const double *A = buf(hs.ia), *B = buf(hs.ib), *L = buf(hs.ix);
    double *Y = buf(hs.io), *Y2 = buf(hs.io2);
    const bool dual = NB == 4 && hs.dual;
    const double c2 = hs.c2, c1 = hs.c1, c0 = hs.c0, d2 = hs.d2, d1 = hs.d1, d0 = hs.d0;
    double y[MB][4], y2[MB][4];
    e2 = t1 = t2 = 0.0;
    // the wave's blocks side by side, four k-steps of operands at a time
    auto product = [&](auto countc) {
      constexpr int C = decltype(countc)::value;
      // Four sums a block, the k-steps in turn: their chains are no longer than the 16 or 32 terms
      // of the kernels that this one replaced.  With two sums |D - D_exact|_F grew by up to 1.16
      // times (varying-mu, n = 80: 1.14e-14 to 1.27e-14; scaled P_{3,1}, n = 64: 3.80e-14 to
      // 4.24e-14).
      dbl4 acc[C][4];
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[i][u] = dbl4{0.0, 0.0, 0.0, 0.0};
      for (int k = 0; k < np; k += 16) {
        double av[C][4], bv[C][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < C; ++i) {
            av[i][u] = A[at(k + 4 * u + fk, br[i] * 16 + fr)];
            bv[i][u] = B[at(k + 4 * u + fk, bc[i] * 16 + fr)];
          }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < C; ++i)
            acc[i][u] =
                __builtin_amdgcn_mfma_f64_16x16x4f64(av[i][u], bv[i][u], acc[i][u], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = br[i] * 16 + fk + 4 * v, c = bc[i] * 16 + fr;
          const double p = (acc[i][0][v] + acc[i][1][v]) + (acc[i][2][v] + acc[i][3][v]);
          const double x = L[at(r, c)];
          const bool on = r == c, in = r < n && c < n;
          y[i][v] = in ? c2 * p + c1 * x + (on ? c0 : 0.0) : 0.0;
          if (NB == 4) y2[i][v] = in ? d2 * p + d1 * x + (on ? d0 : 0.0) : 0.0;
          if (r <= c) {
            const double w = on ? 1.0 : 2.0, d = p - x;
            e2 += w * (d * d);
            t2 += w * (y[i][v] * y[i][v]);
            if (on) t1 += y[i][v];
          }
        }
    };
    if (mine == 2) product(std::integral_constant<int, 2>());
    else if (mine == 1) product(std::integral_constant<int, 1>());
    sum3(e2, t1, t2);                      // (its barrier: every read of the operands is done)
    if (tid < 64) {
      const double root = schedule_root(hs, 0);
      if (tid == 0) schedule_step(&hs, out->log, e2, t1, t2, 0, root);
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      if (NB != 1 && wid + i * kWgWaves < cnt) {         // (the result is in another buffer)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = br[i] * 16 + fk + 4 * v, c = bc[i] * 16 + fr;
          if (r > c) continue;
          Y[at(r, c)] = y[i][v];
          Y[at(c, r)] = y[i][v];
          if (dual) Y2[at(r, c)] = y2[i][v];
          if (dual) Y2[at(c, r)] = y2[i][v];
        }
      }
    }
    __syncthreads();
    if (NB == 1) {
      if (hs.stop) break;                  // X is the result
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (wid + i * kWgWaves < cnt) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int r = br[i] * 16 + fk + 4 * v, c = bc[i] * 16 + fr;
            if (r > c) continue;
            Y[at(r, c)] = y[i][v];
            Y[at(c, r)] = y[i][v];
          }
        }
      }
      __syncthreads();
    }
  }
  const double* X = buf(hs.cur);
  for (int r = wid; r < n; r += kWgWaves)
    for (int c = lane; c < n; c += 64) D[r * ldd + c] = X[at(r, c)];
  unsigned* o = (unsigned*)(SnfHeader*)out;
  for (int i = tid; i < (int)(sizeof(SnfHeader) / 4); i += kWgThreads) o[i] = ((const unsigned*)&hs)[i];
}

// (The launch's own status: an error that an earlier call left must not count as a refusal, as the
// caller would then run the direct steps beside the launched solve.)
template <int NB>
static int launch_wg(size_t bytes, SnfHeader h, const double* F, int64_t ldf, double* D,
                     int64_t ldd, SnfState* out, int max_steps, hipStream_t s) {
  if (bytes > ((size_t)64 << 10) &&
      hipFuncSetAttribute((const void*)solve_wg_kernel<NB>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
    return -1;
  void* args[] = {&h, &F, &ldf, &D, &ldd, &out, &max_steps};
  return hipLaunchKernel((const void*)solve_wg_kernel<NB>, dim3(1), dim3(kWgThreads), args, bytes,
                         s) == hipSuccess ? 0 : -1;
}

int launch_solve_wg(const SnfHeader& h, const double* F, int64_t ldf, double* D, int64_t ldd,
                    SnfState* out, int max_steps, hipStream_t s) {
  const size_t bytes = solve_wg_bytes(h.n, h.scheme);
  switch (wg_buffers(h.scheme)) {
    case 1: return launch_wg<1>(bytes, h, F, ldf, D, ldd, out, max_steps, s);
    case 2: return launch_wg<2>(bytes, h, F, ldf, D, ldd, out, max_steps, s);
    default: return launch_wg<4>(bytes, h, F, ldf, D, ldd, out, max_steps, s);
  }
}

__global__ __launch_bounds__(kReduceThreads) void schedule_kernel(SnfState* __restrict__ s,
                                                                  const double* __restrict__ partials,
                                                                  int count, int init,
                                                                  SnfHeader* __restrict__ host,
                                                                  int32_t* __restrict__ progress,
                                                                  int done) {
  if (s->stop) return;
  schedule_body(s, partials, count, init, host, progress, done);
}

void launch_schedule(SnfState* st, const double* partials, int count, int init, hipStream_t s,
                     SnfHeader* host, int32_t* progress, int done) {
  hipLaunchKernelGGL(schedule_kernel, dim3(1), dim3(kReduceThreads), 0, s, st, partials,
                     count, init, host, progress, done);
}

// ---------------------------------------------------------------------------------------
// Copies
// ---------------------------------------------------------------------------------------
static unsigned copy_blocks(int64_t rows) { return (unsigned)(rows < 2048 ? rows : 2048); }

// Two values at any 8-byte address of global memory, as one 16-byte access (which the target allows
// at 4-byte steps there).  Rows that are not 16-byte aligned took 8-byte accesses 32 bytes apart
// from lane to lane: a two-operand FP64 step of n = 8191 spent 890 us beside its product, one of
// 3001 169, this 702 and 139 (the copies before that, element by element, 767 and 150).
typedef double dbl2a8 __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ dbl2a8 gload2(const double* p) {
  return *(const __attribute__((address_space(1))) dbl2a8*)(p);
}

// dst[r][c] = src[r][c] for r, c < n: a row per workgroup and turn (no index division), four
// columns per thread, as two 16-byte accesses.
__device__ __forceinline__ void copy_rows(const double* __restrict__ src, int64_t lds_,
                                          double* __restrict__ dst, int64_t ldd, int64_t n) {
  for (int64_t r = blockIdx.x; r < n; r += gridDim.x) {
    const double* p = src + r * lds_;
    double* q = dst + r * ldd;
    for (int64_t c = 4 * (int64_t)threadIdx.x; c < n; c += 4 * (int64_t)blockDim.x) {
      if (c + 4 <= n) {
        const dbl2a8 v0 = gload2(p + c), v1 = gload2(p + c + 2);
        *(dbl2a8*)(q + c) = v0;
        *(dbl2a8*)(q + c + 2) = v1;
      } else {
        for (int64_t e = c; e < n && e < c + 4; ++e) q[e] = p[e];
      }
    }
  }
}

// The padded copy of a caller's matrix, zero beyond n, and its low-precision copy; dst may be
// null (the caller's matrix serves as it is), and so may lp.
__global__ __launch_bounds__(256) void pad_copy_kernel(const double* __restrict__ src, int64_t n,
                                                       int64_t ld, double* __restrict__ dst,
                                                       int64_t np, void* __restrict__ lp,
                                                       int lowp_kind) {
  for (int64_t r = blockIdx.x; r < np; r += gridDim.x) {
    const double* p = src + r * ld;
    for (int64_t c = 4 * (int64_t)threadIdx.x; c < np; c += 4 * (int64_t)blockDim.x) {
      double v[4] = {0.0, 0.0, 0.0, 0.0};
      if (r < n) {
        if (c + 4 <= n) {
          const dbl2a8 v0 = gload2(p + c), v1 = gload2(p + c + 2);
          v[0] = v0.x;
          v[1] = v0.y;
          v[2] = v1.x;
          v[3] = v1.y;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (c + e < n) v[e] = p[c + e];
        }
      }
      const int64_t o = r * np + c;
      if (dst) {
        *(double2*)(dst + o) = double2{v[0], v[1]};
        *(double2*)(dst + o + 2) = double2{v[2], v[3]};
      }
      if (lowp_kind == kPrecF32) {
        *(float4*)((float*)lp + o) = float4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
      } else if (lowp_kind == kPrecBF16) {
        unsigned b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) b[e] = f32_to_bf16_rne((float)v[e]);
        *(uint2*)((unsigned short*)lp + o) = uint2{b[0] | (b[1] << 16), b[2] | (b[3] << 16)};
      }
    }
  }
}

void launch_pad_copy(const double* src, int64_t n, int64_t ld, double* dst, int64_t np,
                     void* lp_dst, int lowp_kind, hipStream_t s) {
  hipLaunchKernelGGL(pad_copy_kernel, dim3(copy_blocks(np)), dim3(256), 0, s, src, n, ld, dst, np,
                     lp_dst, lowp_kind);
}

__global__ __launch_bounds__(256) void unpad_copy_kernel(const double* __restrict__ src, int64_t np,
                                                         int64_t n, double* __restrict__ dst,
                                                         int64_t ld) {
  copy_rows(src, np, dst, ld, n);
}

void launch_unpad_copy(const double* src, int64_t np, int64_t n, double* dst, int64_t ld,
                       hipStream_t s) {
  hipLaunchKernelGGL(unpad_copy_kernel, dim3(copy_blocks(n)), dim3(256), 0, s, src, np, n, dst, ld);
}

__global__ void sum_partials_kernel(const double* __restrict__ partials, int count,
                                    double* __restrict__ out3) {
  __shared__ double red[24];
  double a = 0.0, b = 0.0, c = 0.0;
  for (int i = threadIdx.x; i < count; i += kReduceThreads) {
    a += partials[i * 4 + 0];
    b += partials[i * 4 + 1];
    c += partials[i * 4 + 2];
  }
  block_sum3(a, b, c, red);
  if (threadIdx.x == 0) {
    out3[0] = a;
    out3[1] = b;
    out3[2] = c;
  }
}

void launch_sum_partials(const double* partials, int count, double* out3, hipStream_t s) {
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(kReduceThreads), 0, s, partials, count,
                     out3);
}

// ---------------------------------------------------------------------------------------
// Subspace correction (one Newton step on the occupied subspace that re-references F): the
// elementwise parts.  Every kernel walks 32 x 32 tiles of the padded order with a grid-stride
// loop; a tile's transposed partner is staged through LDS so that both reads are coalesced.
// Entries outside the true order n are written as 0, like every other padded buffer.
// ---------------------------------------------------------------------------------------
// V = W + W^T - 2 M (the coupling of G between the subspace of D~ and its complement, with
// W = G D~ and M = D~ G D~), X1 = V, Xbd = G - V (G's part that commutes with D~).
__global__ __launch_bounds__(256) void newton_split_kernel(const double* __restrict__ G,
                                                           const double* __restrict__ W,
                                                           const double* __restrict__ M,
                                                           int64_t n, int64_t np,
                                                           double* __restrict__ Xbd,
                                                           float* __restrict__ Xbd_lp,
                                                           double* __restrict__ X1,
                                                           float* __restrict__ X1_lp) {
  __shared__ double wt[32][33];
  const int64_t nt = np / 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int64_t t = blockIdx.x; t < nt * nt; t += gridDim.x) {
    const int64_t bi = t / nt, bj = t % nt;
    __syncthreads();
    for (int r = ty; r < 32; r += 8) wt[r][tx] = W[(bj * 32 + r) * np + bi * 32 + tx];
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int64_t gr = bi * 32 + r, gc = bj * 32 + tx;
      const int64_t idx = gr * np + gc;
      double v = (W[idx] + wt[tx][r]) - 2.0 * M[idx];
      double xb = G[idx] - v;
      if (gr >= n || gc >= n) v = xb = 0.0;
      X1[idx] = v;
      Xbd[idx] = xb;
      if (X1_lp) X1_lp[idx] = (float)v;
      if (Xbd_lp) Xbd_lp[idx] = (float)xb;
    }
  }
}

// X1_new = c2 (Z + Z^T) + c1 X1: the derivative of the step X <- c2 X^2 + c1 X + c0 I along
// X1, with Z = X X1 (so Z^T = X1 X for symmetric X and X1).  Exactly symmetric.
__global__ __launch_bounds__(256) void newton_sym_kernel(const double* __restrict__ Z,
                                                         const double* __restrict__ X1,
                                                         double c2, double c1, int64_t n,
                                                         int64_t np, double* __restrict__ out,
                                                         float* __restrict__ out_lp) {
  __shared__ double zt[32][33];
  const int64_t nt = np / 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int64_t t = blockIdx.x; t < nt * nt; t += gridDim.x) {
    const int64_t bi = t / nt, bj = t % nt;
    __syncthreads();
    for (int r = ty; r < 32; r += 8) zt[r][tx] = Z[(bj * 32 + r) * np + bi * 32 + tx];
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int64_t gr = bi * 32 + r, gc = bj * 32 + tx;
      const int64_t idx = gr * np + gc;
      double y = c2 * (Z[idx] + zt[tx][r]) + c1 * X1[idx];
      if (gr >= n || gc >= n) y = 0.0;
      out[idx] = y;
      if (out_lp) out_lp[idx] = (float)y;
    }
  }
}

// out = D~ + X1 (the first-order corrected projector) and per-block FP64 sums of its trace
// and squared Frobenius norm, in the partial-sum layout of f0_kernel (the refinement's
// schedule starts from them).
__global__ __launch_bounds__(256) void newton_add_kernel(const double* __restrict__ Dt,
                                                         const double* __restrict__ X1,
                                                         int64_t n, int64_t np,
                                                         double* __restrict__ out,
                                                         double* __restrict__ partials) {
  __shared__ double red[24];
  double t1 = 0.0, t2 = 0.0;
  const int64_t total = np * np;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = idx / np, c = idx % np;
    double y = Dt[idx] + X1[idx];
    if (r >= n || c >= n) y = 0.0;
    out[idx] = y;
    if (r == c) t1 += y;
    t2 += y * y;
  }
  double e0 = 0.0;
  block_sum3(e0, t1, t2, red);
  if (threadIdx.x == 0) {
    partials[blockIdx.x * 4 + 0] = 0.0;
    partials[blockIdx.x * 4 + 1] = t1;
    partials[blockIdx.x * 4 + 2] = t2;
    partials[blockIdx.x * 4 + 3] = 0.0;
  }
}

// Write the operand / output indices, precision and epilogue coefficients of the next product
// of a host-planned sequence into the state the product kernels read.
__global__ void newton_set_kernel(SnfState* __restrict__ st, const NewtonOp* __restrict__ ops,
                                  int k) {
  if (threadIdx.x != 0) return;
  const NewtonOp o = ops[k];
  st->ia = o.ia;
  st->ib = o.ib;
  st->ix = o.ix;
  st->io = o.io;
  st->prec = o.prec;
  st->write_lowp = o.write_lowp;
  st->c2 = o.c2;
  st->c1 = o.c1;
  st->c0 = o.c0;
  st->want_e = 0;
  st->dual = 0;
  st->stop = 0;
}

void launch_newton_split(const double* G, const double* W, const double* M, int64_t n,
                         int64_t np, double* Xbd, float* Xbd_lp, double* X1, float* X1_lp,
                         hipStream_t s) {
  hipLaunchKernelGGL(newton_split_kernel, dim3(kF0Blocks), dim3(256), 0, s, G, W, M, n, np, Xbd,
                     Xbd_lp, X1, X1_lp);
}

void launch_newton_sym(const double* Z, const double* X1, double c2, double c1, int64_t n,
                       int64_t np, double* out, float* out_lp, hipStream_t s) {
  hipLaunchKernelGGL(newton_sym_kernel, dim3(kF0Blocks), dim3(256), 0, s, Z, X1, c2, c1, n, np,
                     out, out_lp);
}

void launch_newton_add(const double* Dt, const double* X1, int64_t n, int64_t np, double* out,
                       double* partials, hipStream_t s) {
  hipLaunchKernelGGL(newton_add_kernel, dim3(kF0Blocks), dim3(256), 0, s, Dt, X1, n, np, out,
                     partials);
}

void launch_newton_set(SnfState* st, const NewtonOp* ops, int k, hipStream_t s) {
  hipLaunchKernelGGL(newton_set_kernel, dim3(1), dim3(64), 0, s, st, ops, k);
}

// ---------------------------------------------------------------------------------------
// Grouped launches over many independent purifications (the serving loop): workgroup b of
// a launch belongs to active request a with offs[a] <= b < offs[a+1] and computes whole
// tile b - offs[a] of that request's pending product, exactly as the single-request
// kernels do (same decomposition, same partial-sum slots), so a request's results do not
// depend on which other requests share the launch.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ int group_find(const int* __restrict__ offs, int nactive, int b) {
  int lo = 0, hi = nactive;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (offs[mid] <= b) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ int slot_tiles(const SlotDesc& sd, int prec) {
  const int nt = (int)(sd.np / (prec == kPrecF64   ? sd.tile[kPrecF64]
                                : prec == kPrecF32 ? sd.tile[kPrecF32]
                                                   : sd.tile[kPrecBF16]));
  return nt * (nt + 1) / 2;
}

__device__ __forceinline__ ProductGrid slot_grid(const SlotDesc& sd, int prec) {
  ProductGrid g;
  g.np = sd.np;
  g.n = sd.n;
  g.sym = 1;
  g.dp_tiles = slot_tiles(sd, prec);
  g.tail_tiles = 0;
  g.split_s = 1;
  g.partial_count = g.dp_tiles;
  g.partials = sd.partials;
  g.split_buf = nullptr;
  return g;
}

// Requests with 64x64 tiles.  A group of requests seldom fills the chip evenly: with 128x128
// tiles a step lasted as long as the longest tile of its largest request (FP64 at n = 2048: 440
// us on one compute unit, FP32 220), the rest waiting.  Bursts, 128x128 to 64x64: 48 requests of
// order 64 to 2048 with an FP32 start 19.6 to 18.0 ms, 20 SP2 up to 700 7.6 to 5.1, 40 in FP64 up
// to 2048 15.6 to 14.9; the matrix cores are busy 65% of such a step.  FP32: the same sum order per
// entry in a quarter of the tile, four waves of 32x32 (k-panels of 16 rather than 32, or two waves
// of 64x32: no faster).
__global__ __launch_bounds__((Layout<float, kFineTile>::NT), 2) void grouped_fine_f32_kernel(
    const SlotDesc* __restrict__ slots, const int* __restrict__ active,
    const int* __restrict__ offs, int nactive) {
  const int a = group_find(offs, nactive, blockIdx.x);
  const SlotDesc sd = slots[active[a]];
  if (sd.st->stop || sd.st->prec != kPrecF32) return;
  const ProductGrid g = slot_grid(sd, kPrecF32);
  WorkItem wi;
  wi.tile = xcd_remap(blockIdx.x - offs[a], g.dp_tiles);
  wi.piece = -1;
  wi.kt_begin = 0;
  wi.kt_end = (int)(sd.np / Mfma<float>::kBK);
  product_body<float, kPrecF32, false, kFineTile>(sd.st, sd.bufs, g, wi);
}

// FP64: the direct step's product (k quarters to the waves of two column groups), on the state
// that the schedule kernel left.
__global__ __launch_bounds__(2 * kDirectThreads) void grouped_fine_f64_kernel(
    const SlotDesc* __restrict__ slots, const int* __restrict__ active,
    const int* __restrict__ offs, int nactive) {
  constexpr int TB = kFineTile / 16, NC = 2, PD = 7, T = kFineTile, QB = TB / NC;
  constexpr int NT = kDirectThreads * NC, W2 = T / 2, NE = 32 * W2 / NT;
  const int a = group_find(offs, nactive, blockIdx.x);
  const SlotDesc sd = slots[active[a]];
  const SnfHeader* st = sd.st;
  if (st->stop || st->prec != kPrecF64) return;
  __shared__ double red[3 * 8];
  __shared__ __attribute__((aligned(16))) double part[4][32][T + 2];
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fk = lane >> 4, kq = wid & 3, cg = wid >> 2;
  const int64_t ld = sd.np;
  const int tile = xcd_remap(blockIdx.x - offs[a], slot_tiles(sd, kPrecF64));
  int bi, bj;
  tile_coords(tile, (int)(sd.np / T), 1, bi, bj);
  const int64_t i0 = (int64_t)bi * T, j0 = (int64_t)bj * T;
  const Buffers& bufs = *sd.bufs;
  const double *Ap = bufs.x[st->ia], *Bp = bufs.x[st->ib], *X = bufs.x[st->ix];
  double2 xs[NE];
  auto load_x = [&](int p) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int idx = e * NT + tid, r = idx / W2, c = 2 * (idx % W2);
      xs[e] = *(const double2*)(X + (i0 + 32 * p + r) * ld + j0 + c);
    }
  };
  const int KT = (int)((sd.n + 3) / 4), kb = kq * KT / 4, ke = (kq + 1) * KT / 4;
  dbl4 acc[TB][QB];
#pragma unroll
  for (int m = 0; m < TB; ++m)
#pragma unroll
    for (int q = 0; q < QB; ++q) acc[m][q] = dbl4{0.0, 0.0, 0.0, 0.0};
  DirectOperand<TB, PD> A;
  DirectOperand<QB, PD> B;
  auto load = [&](int ks, int slot) {
    const int64_t off = (int64_t)(4 * min(ks, max(ke - 1, kb)) + fk) * ld;
    A.load(Ap + off + i0, slot);
    B.load(Bp + off + j0 + cg * 16 * QB, slot);
  };
  auto compute = [&](int slot) {
#pragma unroll
    for (int m = 0; m < TB; ++m)
#pragma unroll
      for (int q = 0; q < QB; ++q)
        acc[m][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(A.get(slot, m), B.get(slot, q), acc[m][q],
                                                         0, 0, 0);
  };
#pragma unroll
  for (int u = 0; u < PD; ++u) load(kb + u, u);
  load_x(0);
  __builtin_amdgcn_sched_barrier(0);
  int ks = kb;
  for (; ks + PD <= ke; ks += PD) {
#pragma unroll
    for (int u = 0; u < PD; ++u) {
      compute(u);
      load(ks + u + PD, u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < PD; ++u)
    if (ks + u < ke) compute(u);
  DirectOut o;
  o.Y = bufs.x[st->io];
  o.Y2 = st->dual ? bufs.x[st->io2] : nullptr;
  o.lp = bufs.lp[st->io];
  o.lowp_kind = st->write_lowp ? (st->mode == SNF_P_BF16_REF64 ? kPrecBF16 : kPrecF32) : -1;
  o.n = (int)sd.n;
  o.ld = ld;
  o.c2 = st->c2;
  o.c1 = st->c1;
  o.c0 = st->c0;
  o.d2 = st->d2;
  o.d1 = st->d1;
  o.d0 = st->d0;
  double e2 = 0.0, t1 = 0.0, t2 = 0.0;
  direct_bands<TB, NC, true>(acc, part, xs, load_x, o, i0, j0, true, e2, t1, t2);
  e2 = wave_sum_rows(e2);
  t1 = wave_sum_rows(t1);
  t2 = wave_sum_rows(t2);
  if (lane == 0) {
    red[wid * 3 + 0] = e2;
    red[wid * 3 + 1] = t1;
    red[wid * 3 + 2] = t2;
  }
  __syncthreads();
  if (tid < 3) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) sum += red[w * 3 + tid];
    sd.partials[(size_t)tile * 4 + tid] = sum;
  }
}

// DUAL: the FP64 variant whose epilogue also writes the second output (the first product of
// a P_{i,j} iteration); each request's state selects exactly one of the two FP64 variants.
template <typename T, int PREC, bool DUAL = false>
__global__ __launch_bounds__((Layout<T, kTile>::NT), 2) void grouped_product_kernel(const SlotDesc* __restrict__ slots,
                                                                 const int* __restrict__ active,
                                                                 const int* __restrict__ offs,
                                                                 int nactive) {
  const int a = group_find(offs, nactive, blockIdx.x);
  const SlotDesc sd = slots[active[a]];
  if (sd.st->stop || sd.st->prec != PREC || (PREC == kPrecF64 && (sd.st->dual != 0) != DUAL))
    return;
  const ProductGrid g = slot_grid(sd, PREC);
  WorkItem wi;
  wi.tile = blockIdx.x - offs[a];
  wi.piece = -1;
  wi.kt_begin = 0;
  wi.kt_end = (int)(sd.np / Mfma<T>::kBK);
  product_body<T, PREC, DUAL>(sd.st, sd.bufs, g, wi);
}

__global__ __launch_bounds__(256, 2) void grouped_product_bf16_kernel(const SlotDesc* __restrict__ slots,
                                                                      const int* __restrict__ active,
                                                                      const int* __restrict__ offs,
                                                                      int nactive) {
  const int a = group_find(offs, nactive, blockIdx.x);
  const SlotDesc sd = slots[active[a]];
  if (sd.st->stop || sd.st->prec != kPrecBF16) return;
  const ProductGrid g = slot_grid(sd, kPrecBF16);
  WorkItem wi;
  wi.tile = blockIdx.x - offs[a];
  wi.piece = -1;
  wi.kt_begin = 0;
  wi.kt_end = (int)(sd.np / 64);
  product_bf16_body(sd.st, sd.bufs, g, wi);
}

__global__ __launch_bounds__(kReduceThreads) void grouped_schedule_kernel(const SlotDesc* __restrict__ slots,
                                                                          const int* __restrict__ active) {
  const SlotDesc sd = slots[active[blockIdx.x]];
  if (sd.st->stop) return;
  schedule_body(sd.st, sd.partials, slot_tiles(sd, sd.st->prec), 0, nullptr);
}

// Start of a solve: its tables from the kernel arguments and X_0 = f_0(F) straight from F.  The
// serving loop waits for a burst's admissions one after the other, so their count of launches and
// copies is what bounds it: with a copy for each of the three tables and for F, and a retirement
// that copied the whole state (the full log) after D, 48 requests of order 64 to 256 took 4.8 ms,
// with one launch each 2.8.  The grid has no more workgroups than X_0 has 32x32 tiles.
__global__ __launch_bounds__(256) void solve_start_kernel(SolveStart a, const double* __restrict__ F,
                                                          int64_t ld, int lowp_kind) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *static_cast<SnfHeader*>(a.desc.st) = a.header;
    *a.desc.bufs = a.bufs;
    if (a.slot) *a.slot = a.desc;
  }
  f0_body(F, a.desc.n, ld, a.desc.np, a.header, a.bufs.x[0], a.bufs.lp[0], lowp_kind,
          a.desc.partials);
}

void launch_solve_start(const SolveStart& a, const double* F, int64_t ld, int lowp_kind,
                        hipStream_t s, int32_t* progress) {
  const int64_t nt = a.desc.np / 32;
  const int blocks = (int)(nt * nt < kF0Blocks ? nt * nt : kF0Blocks);
  hipLaunchKernelGGL(solve_start_kernel, dim3(blocks), dim3(256), 0, s, a, F, ld, lowp_kind);
  launch_schedule(a.desc.st, a.desc.partials, blocks, 1, s, nullptr, progress, 0);
}

// End of a solve: D, and the final state into host-visible memory (the header and the log written).
__global__ __launch_bounds__(256) void solve_finish_kernel(const SnfState* __restrict__ st,
                                                           const Buffers* __restrict__ bufs,
                                                           int64_t n, int64_t np,
                                                           double* __restrict__ D, int64_t ld,
                                                           SnfState* __restrict__ out) {
  copy_rows(bufs->x[st->cur], np, D, ld, n);
  if (blockIdx.x != 0) return;
  const unsigned* h = (const unsigned*)static_cast<const SnfHeader*>(st);
  unsigned* o = (unsigned*)static_cast<SnfHeader*>(out);
  for (int i = threadIdx.x; i < (int)(sizeof(SnfHeader) / 4); i += 256) o[i] = h[i];
  const int words = min(st->nlog, SNF_LOG_MAX) * (int)(sizeof(snf_log_rec) / 4);
  for (int i = threadIdx.x; i < words; i += 256)
    ((unsigned*)out->log)[i] = ((const unsigned*)st->log)[i];
}

void launch_solve_finish(const SnfState* st, const Buffers* bufs_dev, int64_t n, int64_t np,
                         double* D, int64_t ld, SnfState* out, hipStream_t s) {
  hipLaunchKernelGGL(solve_finish_kernel, dim3(copy_blocks(n)), dim3(256), 0, s, st, bufs_dev, n, np,
                     D, ld, out);
}

__global__ void grouped_state_kernel(const SlotDesc* __restrict__ slots,
                                     const int* __restrict__ active, int nactive,
                                     int32_t* __restrict__ state_out) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a < nactive) {
    const SnfState* st = slots[active[a]].st;
    state_out[a] = st->stop ? 1 + st->cur : -1 - st->prec;
  }
}

void launch_grouped_step(const GroupedStep& g, hipStream_t s, hipStream_t s2, hipEvent_t fork,
                         hipEvent_t join) {
  if (g.nactive <= 0) return;
  // the low-precision launches go to s2 after everything on s so far, and s waits for them
  // before the schedule: the product grids (different requests) share the GPU
  const bool split = g.list[kGroupF32Fine].n + g.list[kGroupF32].n + g.list[kGroupBF16].n > 0 &&
                     s2 && fork && join && hipEventRecord(fork, s) == hipSuccess &&
                     hipStreamWaitEvent(s2, fork, 0) == hipSuccess;
  hipStream_t sl = split ? s2 : s;
#define SNF_GROUPED(KERNEL, THREADS, KIND, STREAM)                                               \
  if (g.list[KIND].n > 0)                                                                        \
  hipLaunchKernelGGL(KERNEL, dim3(g.list[KIND].total), dim3(THREADS), 0, STREAM, g.slots,        \
                     g.list[KIND].active, g.list[KIND].offs, g.list[KIND].n)
  SNF_GROUPED(grouped_fine_f32_kernel, (Layout<float, kFineTile>::NT), kGroupF32Fine, sl);
  SNF_GROUPED((grouped_product_kernel<float, kPrecF32>), (Layout<float, kTile>::NT), kGroupF32, sl);
  SNF_GROUPED(grouped_product_bf16_kernel, kThreads, kGroupBF16, sl);
  SNF_GROUPED(grouped_fine_f64_kernel, 2 * kDirectThreads, kGroupF64Fine, s);
  SNF_GROUPED((grouped_product_kernel<double, kPrecF64>), (Layout<double, kTile>::NT), kGroupF64, s);
  SNF_GROUPED((grouped_product_kernel<double, kPrecF64, true>), (Layout<double, kTile>::NT),
              kGroupDual, s);
#undef SNF_GROUPED
  if (split && (hipEventRecord(join, s2) != hipSuccess ||
                hipStreamWaitEvent(s, join, 0) != hipSuccess))
    (void)hipStreamSynchronize(s2);    // the schedule must not start before that product
  hipLaunchKernelGGL(grouped_schedule_kernel, dim3(g.nactive), dim3(kReduceThreads), 0, s, g.slots,
                     g.active);
  hipLaunchKernelGGL(grouped_state_kernel, dim3((g.nactive + 255) / 256), dim3(256), 0, s, g.slots,
                     g.active, g.nactive, g.state_out);
}

}  // namespace snf
