// Bounds of the spectrum and of the gap edges, the inputs both algorithms take (the bounds
// paragraph after Fig. 3: extremal eigenvalues or bounds thereof, and for the scaled
// varying-mu scheme a lower bound of the highest occupied and an upper bound of the lowest
// unoccupied eigenvalue, obtainable from methods for interior eigenvalues).
//
// Lanczos with full reorthogonalisation runs on the device: the symmetric matrix-vector
// product reads only the upper triangle of the matrix in 64x64 tiles (row part and
// transposed column part of each off-diagonal tile from one copy in registers; bound by one
// pass over half the matrix per product), the Gram-Schmidt passes are fixed-order reductions, so every
// run gives the same tridiagonal bit for bit.  The host diagonalises the small tridiagonal
// (implicit QR) and forms the bounds.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "../../include/snf.h"
#include "wave_sum.h"

namespace snf {
namespace {

constexpr int kT = 64;              // tile side of the matrix-vector product
constexpr int kMaxSteps = 512;
constexpr int kVecThreads = 256;
constexpr double kBreakdown = 1e-12;

#define BD_HIP(call)                                    \
  do {                                                  \
    hipError_t _e = (call);                             \
    if (_e != hipSuccess) {                             \
      (void)hipGetLastError();                          \
      return SNF_EDEVICE;                               \
    }                                                   \
  } while (0)

// ---- symmetric matrix-vector product from the upper triangle ---------------------------
// Up to two vectors share each read of the matrix: y_v = a_v (M x_v) + b_v x_v.
struct SymvArgs {
  const double* M;
  int64_t ld, n, np;
  int nv, strip;                // vectors; tiles per strip
  const double* x[2];
  double* y[2];
  double a[2], b[2];
  double* part;                 // [nt][nt][nv][kT] column parts, then [nt][nt][nv][kT] row parts
  // x_v is not normalised yet: its squared norm in nt partial sums, the normalised vector's
  // place, and the norm's (or null); null: x_v is used as it is
  const double* nrm2[2];
  double* vout[2];
  double* beta[2];
  // last product of a Lanczos step: h_k = V_k . y_v for k <= j, block partials [k][nt]
  const double* V[2];
  double* hp[2];
  int j;
};

// The norm from its nt partial sums, by every wave for itself (fixed order).
__device__ __forceinline__ double norm_of(const double* __restrict__ nrm2, int nt) {
  double s = 0.0;
  for (int i = threadIdx.x & 63; i < nt; i += 64) s += nrm2[i];
  return sqrt(wave_sum_rows(s));
}

// One workgroup per strip of up to g.strip upper tiles (I, J), (I, J + 1), ... of block row I:
// the row part sum_J M_IJ x_J (for block I) and each tile's column part M_IJ^T x_I (for block J).
// Every thread keeps 16 values of the tile in registers (4 rows x 4 columns, 16 apart) and uses
// each for both parts, the next tile's 16 loads in flight meanwhile; sums run over the 16 lanes
// of a row once per strip and over the 16 threads of a column once per tile.  16 us with one
// vector and 17 us with two at n = 4096 (68 MB: 4.3 and 4.0 TB/s).  x through LDS instead, or
// x_J loaded a tile ahead, cost the two-vector kernel registers (3 -> 2 waves per SIMD) or time
// (24 -> 26 us, with strips of four tiles).
template <int NV, bool ABS>
__global__ __launch_bounds__(256) void symv_tile_kernel(SymvArgs g, int nt) {
  const int I = blockIdx.y, J0 = I + (int)blockIdx.x * g.strip;
  if (J0 >= nt) return;
  const int J1 = min(J0 + g.strip, nt);
  __shared__ double cs[2][4][NV][kT];      // column sums of the four waves, by tile parity
  const int t = threadIdx.x, tx = t & 15, ty = t >> 4, wid = t >> 6;
  const int64_t r0 = (int64_t)I * kT;
  double m[4][4];
  auto load = [&](int J, double (&o)[4][4]) {
    const int64_t c0 = (int64_t)J * kT;
    const double* p = g.M + (r0 + ty) * g.ld + c0 + tx;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const bool in = r0 + ty + 16 * q < g.n && c0 + tx + 16 * c < g.n &&
                        (J != I || tx + 16 * c >= ty + 16 * q);
        const double e = in ? p[(int64_t)(16 * q) * g.ld + 16 * c] : 0.0;
        o[q][c] = ABS ? fabs(e) : e;
      }
  };
  load(J0, m);                             // (ahead of the norm, which waits for its own loads)
  double inv[NV], xi[NV][4], row[NV][4];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    inv[v] = 1.0;
    if (g.nrm2[v]) {
      const double nrm = norm_of(g.nrm2[v], nt);
      inv[v] = nrm > 0.0 ? 1.0 / nrm : 0.0;      // a zero norm leaves zeros: T is cut there
      if (I == 0 && J0 == 0 && t == 0 && g.beta[v]) *g.beta[v] = nrm;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      row[v][q] = 0.0;
      xi[v][q] = g.x[v][r0 + ty + 16 * q] * inv[v];
    }
    if (J0 == I && g.vout[v] && t < kT) g.vout[v][r0 + t] = g.x[v][r0 + t] * inv[v];
  }
  for (int J = J0; J < J1; ++J) {
    const int par = (J - J0) & 1;
    double nx[4][4];
    if (J + 1 < J1) load(J + 1, nx);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double xj[4], col[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        xj[c] = g.x[v][(int64_t)J * kT + tx + 16 * c] * inv[v];
        col[c] = 0.0;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          row[v][q] += m[q][c] * xj[c];
          // (a diagonal entry counts once)
          const double e = (J == I && tx + 16 * c == ty + 16 * q) ? 0.0 : m[q][c];
          col[c] += e * xi[v][q];
        }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        col[c] += __shfl_xor(col[c], 16, 64);
        col[c] += __shfl_xor(col[c], 32, 64);
        if ((t & 63) < 16) cs[par][wid][v][tx + 16 * c] = col[c];
      }
    }
    __syncthreads();                       // (the other parity's sums were read before this)
    if (t < NV * kT) {
      const int v = t / kT, c = t % kT;
      g.part[(((size_t)I * nt + J) * NV + v) * kT + c] =
          ((cs[par][0][v][c] + cs[par][1][v][c]) + cs[par][2][v][c]) + cs[par][3][v][c];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < 4; ++c) m[q][c] = nx[q][c];
  }
  double* rp = g.part + (size_t)nt * nt * NV * kT;
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double s = row[v][q];
      s += __shfl_xor(s, 1, 64);
      s += __shfl_xor(s, 2, 64);
      s += __shfl_xor(s, 4, 64);
      s += __shfl_xor(s, 8, 64);
      if (tx == 0) rp[(((size_t)I * nt + blockIdx.x) * NV + v) * kT + ty + 16 * q] = s;
    }
}

// y_v[i] = a_v (sum of the row parts of the strips of block row B and the column parts of tiles
// (I <= B, B)) + b_v x_v[i]; zero beyond n.  One workgroup per row block B and vector: 16 waves
// each take every 16th part, then the 16 partial sums of a row are added in wave order (fixed
// order, no atomics).  The last product of a Lanczos step goes on to the block's share of the
// first Gram-Schmidt pass's dot products, which saves a launch that would read y again.
__global__ __launch_bounds__(1024) void symv_reduce_kernel(SymvArgs g, int nt) {
  __shared__ double acc[16][kT];
  const int B = blockIdx.x, v = blockIdx.y;
  const int grp = threadIdx.x / kT, r = threadIdx.x % kT;
  const int ns = (nt - B + g.strip - 1) / g.strip;
  const double* rp = g.part + (size_t)nt * nt * g.nv * kT;
  double s = 0.0;
  for (int q = grp; q < ns + B + 1; q += 16) {
    if (q < ns) s += rp[(((size_t)B * nt + q) * g.nv + v) * kT + r];
    else s += g.part[(((size_t)(q - ns) * nt + B) * g.nv + v) * kT + r];
  }
  acc[grp][r] = s;
  __syncthreads();
  const int64_t i = (int64_t)B * kT + r;
  if (grp == 0) {
    double tot = 0.0;
    for (int k = 0; k < 16; ++k) tot += acc[k][r];
    // (the normalised x_v, where this product was handed the raw one)
    const double x = g.b[v] != 0.0 ? (g.vout[v] ? g.vout[v][i] : g.x[v][i]) : 0.0;
    const double y = i < g.n ? g.a[v] * tot + g.b[v] * x : 0.0;
    g.y[v][i] = y;
    acc[0][r] = y;
  }
  if (!g.hp[v]) return;
  __syncthreads();
  const double y = acc[0][r];
  for (int k = grp; k <= g.j; k += 16) {
    const double d = wave_sum_rows(g.V[v][(size_t)k * g.np + i] * y);
    if (r == 0) g.hp[v][(size_t)k * nt + B] = d;
  }
}

// d[i] = M[i][i] for i < n.
__global__ __launch_bounds__(256) void diag_kernel(const double* M, int64_t ld, int64_t n,
                                                   double* d) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) d[i] = M[i * ld + i];
}

// ---- Lanczos vector operations (chains along blockIdx.y) -------------------------------
struct Chains {
  double* V;       // [chain][kMax + 1][np]
  double* w;       // [chain][np]
  double* hp;      // [chain][2][(kMax + 1) nt] block partials of the dot products, by pass
  double* nrm2;    // [chain][nt] block partials of ||w||^2
  double* alpha;   // [chain][kMax]
  double* beta;    // [chain][kMax]
  int64_t np;
  int kmax;
  int nt;
};

// One Gram-Schmidt pass on the 64 rows of block B: h_k = V_k . w from the block partials, w <- w
// - sum_{k <= j} h_k V_k (the terms over 16 waves, added in wave order), then the block's
// partials of what the next kernel needs: the second pass's dot products (PASS 0) or ||w||^2
// (PASS 1).  Every block sums all partials of h itself, which costs less than a launch; h_j goes
// into alpha_j (set on pass 0, added on 1).
// Long runs on small matrices, where one workgroup has every sum to itself, are bound by the wave
// sums (500 steps at n = 10: 25.2 ms with shuffles, 15.7 by DPP).
template <int PASS>
__global__ __launch_bounds__(1024) void lz_update_kernel(Chains c, int j) {
  __shared__ double h[kMaxSteps];
  __shared__ double acc[16][kT];
  const int B = blockIdx.x, ch = blockIdx.y, nt = c.nt;
  const int grp = threadIdx.x / kT, r = threadIdx.x % kT;
  const double* hp = c.hp + ((size_t)ch * 2 + PASS) * (c.kmax + 1) * nt;
  const double* V = c.V + (size_t)ch * (c.kmax + 1) * c.np;
  const int64_t i = (int64_t)B * kT + r;
  for (int k = grp; k <= j; k += 16) {
    double s = 0.0;
    for (int b = r; b < nt; b += 64) s += hp[(size_t)k * nt + b];
    s = wave_sum_rows(s);
    if (r == 0) h[k] = s;
  }
  __syncthreads();
  if (B == 0 && threadIdx.x == 0) {
    double* al = c.alpha + (size_t)ch * c.kmax + j;
    *al = PASS == 0 ? h[j] : *al + h[j];
  }
  double s = 0.0;
  for (int k = grp; k <= j; k += 16) s += h[k] * V[(size_t)k * c.np + i];
  acc[grp][r] = s;
  __syncthreads();
  if (grp == 0) {
    double tot = 0.0;
    for (int k = 0; k < 16; ++k) tot += acc[k][r];
    const double w = c.w[(size_t)ch * c.np + i] - tot;
    c.w[(size_t)ch * c.np + i] = w;
    acc[0][r] = w;
    if (PASS == 1) {
      const double q = wave_sum_rows(w * w);
      if (r == 0) c.nrm2[(size_t)ch * nt + B] = q;
    }
  }
  if (PASS == 1) return;
  __syncthreads();
  const double w = acc[0][r];
  double* hn = c.hp + ((size_t)ch * 2 + 1) * (c.kmax + 1) * nt;
  for (int k = grp; k <= j; k += 16) {
    const double d = wave_sum_rows(V[(size_t)k * c.np + i] * w);
    if (r == 0) hn[(size_t)k * nt + B] = d;
  }
}

// The last step's beta (the others are written where the vector is normalised).
__global__ __launch_bounds__(64) void lz_beta_kernel(Chains c, int j) {
  const int ch = blockIdx.x;
  const double b = norm_of(c.nrm2 + (size_t)ch * c.nt, c.nt);
  if (threadIdx.x == 0) c.beta[(size_t)ch * c.kmax + j] = b;
}

// x = 1 on [0, n), 0 beyond.
__global__ __launch_bounds__(kVecThreads) void fill_ones_kernel(double* x, int64_t n,
                                                                int64_t np) {
  const int64_t i = (int64_t)blockIdx.x * kVecThreads + threadIdx.x;
  if (i < np) x[i] = i < n ? 1.0 : 0.0;
}

// w = s and its squared norm for every chain; s = start (n values, zero padded), or the fixed
// pseudo-random vector u_i in [-1, 1) from SplitMix64 of i (Steele, Lea, Flood 2014).
__device__ __forceinline__ double splitmix_uniform(uint64_t i) {
  uint64_t z = i + 0x9E3779B97F4A7C15ull * (i + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z = z ^ (z >> 31);
  return (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

__global__ __launch_bounds__(kT) void lz_start_kernel(Chains c, const double* start, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  const int ch = blockIdx.y;
  double v = 0.0;
  if (i < n) v = start ? start[i] : splitmix_uniform((uint64_t)i);
  c.w[(size_t)ch * c.np + i] = v;
  const double q = wave_sum_rows(v * v);
  if (threadIdx.x == 0) c.nrm2[(size_t)ch * c.nt + blockIdx.x] = q;
}

// ---- host side -------------------------------------------------------------------------

// Extremal eigenvalues and the last components of their eigenvectors of the symmetric
// tridiagonal (a, b) of order k, by implicit QR steps with Wilkinson's shift (Golub and Van
// Loan, Matrix Computations, section 8.3): T <- Q^T T Q until every off-diagonal element is
// negligible.  Of the eigenvectors only their last components are wanted, so of Q only the last
// row is carried along: 2-3 sweeps of at most k rotations per eigenvalue, 80 us at k = 40 where
// cyclic Jacobi rotations on the dense k x k matrix with all of Q took 0.7 ms.
static void tridiag_extremes(std::vector<double> a, std::vector<double> b, int k, double* tmin,
                             double* smin_last, double* tmax, double* smax_last) {
  std::vector<double> z(k, 0.0);           // last row of Q
  z[k - 1] = 1.0;
  int hi = k - 1;
  for (int sweep = 0; hi > 0 && sweep < 60 * k; ++sweep) {
    // b[i] couples i and i + 1; the unreduced block that ends at hi starts at lo
    auto negligible = [&](int i) { return fabs(b[i]) <= 1e-16 * (fabs(a[i]) + fabs(a[i + 1])); };
    if (negligible(hi - 1)) {
      --hi;
      continue;
    }
    int lo = hi - 1;
    while (lo > 0 && !negligible(lo - 1)) --lo;
    // shift: the eigenvalue of the trailing 2 x 2 block nearer to a[hi]
    const double d = 0.5 * (a[hi - 1] - a[hi]), bb = b[hi - 1];
    const double shift = a[hi] - bb * bb / (d + copysign(hypot(d, bb), d));
    double x = a[lo] - shift, y = b[lo];
    for (int i = lo; i < hi; ++i) {        // chase the bulge y down the band
      const double r = hypot(x, y);
      const double c = r > 0.0 ? x / r : 1.0, sn = r > 0.0 ? y / r : 0.0;
      if (i > lo) b[i - 1] = r;
      const double p = a[i], q = a[i + 1], o = b[i];
      a[i] = c * c * p + 2.0 * c * sn * o + sn * sn * q;
      a[i + 1] = sn * sn * p - 2.0 * c * sn * o + c * c * q;
      b[i] = c * sn * (q - p) + (c * c - sn * sn) * o;
      if (i + 1 < hi) {
        x = b[i];
        y = sn * b[i + 1];
        b[i + 1] *= c;
      }
      const double z0 = z[i], z1 = z[i + 1];
      z[i] = c * z0 + sn * z1;
      z[i + 1] = c * z1 - sn * z0;
    }
  }
  int imin = 0, imax = 0;
  for (int i = 1; i < k; ++i) {
    if (a[i] < a[imin]) imin = i;
    if (a[i] > a[imax]) imax = i;
  }
  *tmin = a[imin];
  *tmax = a[imax];
  *smin_last = fabs(z[imin]);
  *smax_last = fabs(z[imax]);
}

// (theta_min, r_min, theta_max, r_max) from the Lanczos coefficients: T cut at the first
// beta_j <= 1e-12 max |alpha_0..j| (then the residuals are zero).
static void ritz_from(const double* al, const double* be, int steps, double* out4) {
  int k = steps;
  bool broke = false;
  double amax = 0.0;
  for (int j = 0; j < steps; ++j) {
    amax = std::max(amax, fabs(al[j]));
    if (be[j] <= kBreakdown * amax) {
      k = j + 1;
      broke = true;
      break;
    }
  }
  std::vector<double> a(al, al + k), b(be, be + k);
  double tmin, smin, tmax, smax;
  tridiag_extremes(a, b, k, &tmin, &smin, &tmax, &smax);
  const double tail = broke ? 0.0 : b[k - 1];
  out4[0] = tmin;
  out4[1] = tail * smin;
  out4[2] = tmax;
  out4[3] = tail * smax;
}

struct BoundsWorkspace {
  int64_t np = 0;
  int kmax = 0, nv = 0;
  double *V = nullptr, *w = nullptr, *hp = nullptr, *alpha = nullptr, *beta = nullptr;
  double *y = nullptr, *z = nullptr, *part = nullptr, *nrm2 = nullptr;
  double* host = nullptr;       // pinned read-back
  size_t host_cap = 0;
  std::mutex mu;
};

static std::mutex g_bd_mu;
static BoundsWorkspace* g_bd[64];

static BoundsWorkspace* bounds_workspace() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> g(g_bd_mu);
  if (!g_bd[dev]) g_bd[dev] = new BoundsWorkspace();
  return g_bd[dev];
}

static void release(BoundsWorkspace* w) {
  double** ptrs[] = {&w->V, &w->w, &w->hp, &w->alpha, &w->beta, &w->y, &w->z, &w->part,
                     &w->nrm2};
  for (double** p : ptrs) {
    if (*p) (void)hipFree(*p);
    *p = nullptr;
  }
  w->np = 0;
  w->kmax = 0;
  w->nv = 0;
}

static int ensure(BoundsWorkspace* w, int64_t np, int kmax, int nv) {
  if (np > w->np || kmax > w->kmax || nv > w->nv) {
    release(w);
    const int nt = (int)(np / kT);
    const size_t sizes[] = {(size_t)nv * (kmax + 1) * np, (size_t)nv * np,
                            (size_t)nv * 2 * (kmax + 1) * nt, (size_t)nv * kmax,
                            (size_t)nv * kmax, (size_t)nv * np, (size_t)nv * np,
                            (size_t)nt * nt * nv * 2 * kT, (size_t)nv * nt};
    double** ptrs[] = {&w->V, &w->w, &w->hp, &w->alpha, &w->beta, &w->y, &w->z, &w->part,
                       &w->nrm2};
    for (int i = 0; i < 9; ++i)
      if (hipMalloc(ptrs[i], sizes[i] * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        release(w);
        return SNF_ENOMEM;
      }
    w->np = np;
    w->kmax = kmax;
    w->nv = nv;
  }
  const size_t need = (size_t)2 * nv * kmax + 2 * (size_t)np;
  if (need > w->host_cap) {
    if (w->host) (void)hipHostFree(w->host);
    w->host = nullptr;
    w->host_cap = 0;
    BD_HIP(hipHostMalloc(&w->host, need * sizeof(double), hipHostMallocDefault));
    w->host_cap = need;
  }
  return SNF_OK;
}

// Tiles per strip, by the tiles a side alone: the more, the longer a workgroup's reads run on
// while its partial row sums are few, until too few strips are left for the chip.  40-step
// gap_bounds (spectral_bounds follows the same order within 5%), ms with 1, 2, 3, 4, 5, 8 tiles a
// strip: n = 1000 1.50 1.69 1.88 2.07 2.25 2.83; 2048 2.15 1.94 2.10 2.17 2.34 2.90; 3072 2.95 2.36
// 2.59 2.79 2.70 3.20; 4096 3.93 3.29 2.88 3.06 3.30 3.41; 6000 6.44 5.29 5.50 5.15 5.59 5.12; 9000
// 13.3 11.2 10.9 10.9 11.0 11.3; 16384 42.1 34.3 31.0 31.8 31.0 31.0.
// The grid is an odd number of strips wide: workgroups go to the 8 XCDs in turn, and where the
// width divided by 8 a row's strip k ran on the same XCD in every row, of which the later ones have
// no strip k (four tiles a strip: n = 8000 11.9 ms, 8.99 with an odd width; 4096 3.80, 3.06).
static void launch_symv(SymvArgs& g, hipStream_t s, bool abs_mode = false) {
  const int nt = (int)(g.np / kT);
  g.strip = nt < 32 ? 1 : nt < 52 ? 2 : nt < 72 ? 3 : nt < 200 ? 4 : 5;
  const dim3 grid(((nt + g.strip - 1) / g.strip) | 1, nt);
  if (abs_mode) hipLaunchKernelGGL((symv_tile_kernel<1, true>), grid, dim3(256), 0, s, g, nt);
  else if (g.nv == 1) hipLaunchKernelGGL((symv_tile_kernel<1, false>), grid, dim3(256), 0, s, g, nt);
  else hipLaunchKernelGGL((symv_tile_kernel<2, false>), grid, dim3(256), 0, s, g, nt);
  hipLaunchKernelGGL(symv_reduce_kernel, dim3(nt, g.nv), dim3(1024), 0, s, g, nt);
}

static SymvArgs symv_args(const double* M, int64_t ld, int64_t n, int64_t np, int nv,
                          double* part) {
  SymvArgs g;
  memset(&g, 0, sizeof(g));
  g.M = M;
  g.ld = ld;
  g.n = n;
  g.np = np;
  g.nv = nv;
  g.part = part;
  return g;
}

// Lanczos on nv chains.  apply(j, first, last) must leave A v_j of every chain in c.w: its first
// product takes the unnormalised vector in c.w and leaves v_j in V (first), its last one
// computes the first pass's dot products (last).  Four launches a step besides the products
// between them.
template <typename Apply>
static int run_lanczos(BoundsWorkspace* w, int64_t n, int64_t np, int nv, int steps,
                       const double* start, Apply apply, hipStream_t s) {
  const int nt = (int)(np / kT);
  Chains c{w->V, w->w, w->hp, w->nrm2, w->alpha, w->beta, np, w->kmax, nt};
  const dim3 gb(nt, nv);
  hipLaunchKernelGGL(lz_start_kernel, gb, dim3(kT), 0, s, c, start, n);
  BD_HIP(hipGetLastError());
  for (int j = 0; j < steps; ++j) {
    auto first = [&](SymvArgs& g) {
      for (int v = 0; v < nv; ++v) {
        g.x[v] = c.w + (size_t)v * np;
        g.nrm2[v] = c.nrm2 + (size_t)v * nt;
        g.vout[v] = c.V + ((size_t)v * (c.kmax + 1) + j) * np;
        g.beta[v] = j > 0 ? c.beta + (size_t)v * c.kmax + j - 1 : nullptr;
      }
    };
    auto last = [&](SymvArgs& g) {
      for (int v = 0; v < nv; ++v) {
        g.y[v] = c.w + (size_t)v * np;
        g.V[v] = c.V + (size_t)v * (c.kmax + 1) * np;
        g.hp[v] = c.hp + (size_t)v * 2 * (c.kmax + 1) * nt;
      }
      g.j = j;
    };
    apply(first, last);
    hipLaunchKernelGGL(lz_update_kernel<0>, gb, dim3(1024), 0, s, c, j);
    hipLaunchKernelGGL(lz_update_kernel<1>, gb, dim3(1024), 0, s, c, j);
    BD_HIP(hipGetLastError());
  }
  hipLaunchKernelGGL(lz_beta_kernel, dim3(nv), dim3(64), 0, s, c, steps - 1);
  BD_HIP(hipGetLastError());
  return SNF_OK;
}

}  // namespace

void bounds_release_all_devices() {
  int prev = 0;
  const bool restore = hipGetDevice(&prev) == hipSuccess;
  for (int dev = 0; dev < 64; ++dev) {
    BoundsWorkspace* w = nullptr;
    {
      std::lock_guard<std::mutex> g(g_bd_mu);
      w = g_bd[dev];
    }
    if (!w || hipSetDevice(dev) != hipSuccess) continue;
    std::lock_guard<std::mutex> g(w->mu);
    (void)hipDeviceSynchronize();
    release(w);
    if (w->host) (void)hipHostFree(w->host);
    w->host = nullptr;
    w->host_cap = 0;
  }
  if (restore) (void)hipSetDevice(prev);
}

}  // namespace snf

using namespace snf;

extern "C" {

int snf_spectral_bounds(const double* F_dev, int64_t n, int64_t ld, int32_t steps,
                        const double* start_dev, double* out, void* stream) {
  if (!F_dev || !out || n <= 0 || ld < n || steps < 1 || steps > kMaxSteps) return SNF_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  BoundsWorkspace* w = bounds_workspace();
  if (!w) return SNF_EDEVICE;
  std::lock_guard<std::mutex> guard(w->mu);
  const int64_t np = (n + kT - 1) / kT * kT;
  int rc = ensure(w, np, std::max(steps, w->kmax), std::max(1, w->nv));
  if (rc) return rc;
  const int kmax = w->kmax;
  auto apply = [&](auto first, auto last) {
    SymvArgs g = symv_args(F_dev, ld, n, np, 1, w->part);
    first(g);
    last(g);
    g.a[0] = 1.0;
    g.b[0] = 0.0;
    launch_symv(g, s);
  };
  rc = run_lanczos(w, n, np, 1, steps, start_dev, apply, s);
  if (rc) return rc;
  // Gershgorin: r_i = sum_j |F_ij| from the same product with |F| and x = 1
  {
    hipLaunchKernelGGL(fill_ones_kernel, dim3((unsigned)((np + kVecThreads - 1) / kVecThreads)),
                       dim3(kVecThreads), 0, s, w->z, n, np);
    SymvArgs g = symv_args(F_dev, ld, n, np, 1, w->part);
    g.x[0] = w->z;
    g.y[0] = w->y;
    g.a[0] = 1.0;
    g.b[0] = 0.0;
    launch_symv(g, s, true);
    BD_HIP(hipGetLastError());
  }
  double* hab = w->host;
  double* hrow = w->host + 2 * (size_t)w->nv * kmax;
  BD_HIP(hipMemcpyAsync(hab, w->alpha, steps * sizeof(double), hipMemcpyDeviceToHost, s));
  BD_HIP(hipMemcpyAsync(hab + kmax, w->beta, steps * sizeof(double), hipMemcpyDeviceToHost, s));
  BD_HIP(hipMemcpyAsync(hrow, w->y, n * sizeof(double), hipMemcpyDeviceToHost, s));
  hipLaunchKernelGGL(diag_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, F_dev, ld,
                     n, w->z);
  BD_HIP(hipGetLastError());
  double* diag = hrow + np;
  BD_HIP(hipMemcpyAsync(diag, w->z, n * sizeof(double), hipMemcpyDeviceToHost, s));
  BD_HIP(hipStreamSynchronize(s));
  double r4[4];
  ritz_from(hab, hab + kmax, steps, r4);
  const double pad = 1e-13 * std::max(fabs(r4[0]), fabs(r4[2]));
  out[0] = r4[0] - r4[1] - pad;
  out[1] = r4[2] + r4[3] + pad;
  double glo = INFINITY, ghi = -INFINITY;
  for (int64_t i = 0; i < n; ++i) {
    const double rad = hrow[i] - fabs(diag[i]);
    glo = std::min(glo, diag[i] - rad);
    ghi = std::max(ghi, diag[i] + rad);
  }
  out[2] = glo;
  out[3] = ghi;
  return SNF_OK;
}

int snf_gap_bounds(const double* F_dev, const double* D_dev, int64_t n, int64_t ld,
                   double lambda_min, double lambda_max, int32_t steps,
                   const double* start_dev, double* out, void* stream) {
  if (!F_dev || !D_dev || !out || n <= 0 || ld < n || steps < 1 || steps > kMaxSteps ||
      !isfinite(lambda_min) || !isfinite(lambda_max) || !(lambda_min < lambda_max))
    return SNF_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  BoundsWorkspace* w = bounds_workspace();
  if (!w) return SNF_EDEVICE;
  std::lock_guard<std::mutex> guard(w->mu);
  const int64_t np = (n + kT - 1) / kT * kT;
  int rc = ensure(w, np, std::max(steps, w->kmax), 2);
  if (rc) return rc;
  const int kmax = w->kmax;
  // chain 0: D (F - lambda_min I) D;  chain 1: (I - D)(lambda_max I - F)(I - D)
  auto apply = [&](auto first, auto last) {
    SymvArgs g = symv_args(D_dev, ld, n, np, 2, w->part);
    first(g);
    g.y[0] = w->y;
    g.y[1] = w->y + np;
    g.a[0] = 1.0;  g.b[0] = 0.0;
    g.a[1] = -1.0; g.b[1] = 1.0;
    launch_symv(g, s);
    SymvArgs f = symv_args(F_dev, ld, n, np, 2, w->part);
    f.x[0] = w->y;
    f.x[1] = w->y + np;
    f.y[0] = w->z;
    f.y[1] = w->z + np;
    f.a[0] = 1.0;  f.b[0] = -lambda_min;
    f.a[1] = -1.0; f.b[1] = lambda_max;
    launch_symv(f, s);
    SymvArgs d = symv_args(D_dev, ld, n, np, 2, w->part);
    d.x[0] = w->z;
    d.x[1] = w->z + np;
    last(d);
    d.a[0] = 1.0;  d.b[0] = 0.0;
    d.a[1] = -1.0; d.b[1] = 1.0;
    launch_symv(d, s);
  };
  rc = run_lanczos(w, n, np, 2, steps, start_dev, apply, s);
  if (rc) return rc;
  double* hab = w->host;
  for (int ch = 0; ch < 2; ++ch) {
    BD_HIP(hipMemcpyAsync(hab + (size_t)ch * 2 * kmax, w->alpha + (size_t)ch * kmax,
                          steps * sizeof(double), hipMemcpyDeviceToHost, s));
    BD_HIP(hipMemcpyAsync(hab + (size_t)ch * 2 * kmax + kmax, w->beta + (size_t)ch * kmax,
                          steps * sizeof(double), hipMemcpyDeviceToHost, s));
  }
  BD_HIP(hipStreamSynchronize(s));
  double r0[4], r1[4];
  ritz_from(hab, hab + kmax, steps, r0);
  ritz_from(hab + 2 * (size_t)kmax, hab + 3 * (size_t)kmax, steps, r1);
  const double pad = 1e-13 * (lambda_max - lambda_min);
  out[0] = lambda_min + r0[2] - pad;
  out[1] = lambda_max - r1[2] + pad;
  return SNF_OK;
}

}  // extern "C"
