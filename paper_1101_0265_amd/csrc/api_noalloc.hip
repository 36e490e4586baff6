// snf_purify_dense_noalloc: the dense purification of snf_purify_dense for callers that cannot
// allocate (code under stream capture, tight serving loops, harnesses that forbid hipMalloc).
//
// Every byte of device memory beyond the caller's F and D comes from `scratch`, a file-scope
// device array of fixed size: the FP64 iterate buffers, the per-tile partial sums, the scalar
// state.  Its device address is taken once per device with
// hipGetSymbolAddress (the array's name in host code is a host-side stand-in, not a device
// address) and kept; every kernel argument and copy uses that address.  Host staging (the
// scalar state, the stop flag) lives in static host arrays, and the step loop reads the stop
// flag with a synchronous copy instead of pinned memory and events, so the call makes no
// allocation of any kind.  The kernels are those of snf_purify_dense (the direct steps and the
// one-workgroup solve), launched in the same order on the same decomposition, so the results
// are the same bit for bit.
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <string.h>

#include <mutex>

#include "schedule_math.h"
#include "snf_internal.h"

namespace snf {
namespace na {

constexpr int64_t kNaMaxNp = SNF_NOALLOC_MAX_N;         // largest padded order taken
constexpr int64_t kNaMaxLd = 912;                       // largest row stride: 19 tiles of 48
constexpr int kNaPartialSlots = 2 * kDirectSlots;
constexpr size_t kNaMatrix = (size_t)kNaMaxLd * kNaMaxLd;

// Layout of the scratch array (offsets in doubles, each a multiple of 32, i.e. 256 bytes).
constexpr size_t align32(size_t v) { return (v + 31) / 32 * 32; }
constexpr size_t kOffState = 0;
constexpr size_t kOffHdr = align32(kOffState + (sizeof(SnfState) + 7) / 8);
constexpr size_t kOffClock = align32(kOffHdr + (2 * sizeof(SnfHeader) + 7) / 8);
constexpr size_t kOffPartials = align32(kOffClock + 2);
constexpr size_t kOffX = align32(kOffPartials + (size_t)kNaPartialSlots * 4);
constexpr size_t kScratchDoubles = SNF_NOALLOC_SCRATCH_BYTES / 8;
static_assert(kOffX + 4 * kNaMatrix <= kScratchDoubles,
              "the layout must fit in SNF_NOALLOC_SCRATCH_BYTES");

}  // namespace na
}  // namespace snf

// The scratch memory of snf_purify_dense_noalloc; each device holds its own copy until the
// process ends.
static __device__ __align__(256) double scratch[snf::na::kScratchDoubles];

namespace snf {
namespace {
using namespace na;

std::mutex g_na_mu[64];
double* g_na_ptr[64];                 // device address of scratch, per device
SnfState g_na_state[64];              // host staging of the scalar state, per device
int32_t g_na_flag[64];

__global__ void na_clock_kernel(unsigned long long* out) {
  if (threadIdx.x == 0) *out = wall_clock64();
}

#define NA_HIP(call)                                       \
  do {                                                     \
    hipError_t _e = (call);                                \
    if (_e != hipSuccess) return record_hip_error(_e, #call); \
  } while (0)

int na_body(const double* F_dev, int64_t n, int64_t ld, const snf_params* params,
            snf_scheme scheme, double* D_dev, snf_result* out, snf_log_rec* log,
            int32_t log_cap, hipStream_t s, int dev) {
  double* base = g_na_ptr[dev];
  if (!base) {
    // first call on this device: the device address of this device's copy of the array
    void* p = nullptr;
    NA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return SNF_EDEVICE;
    base = (double*)p;
    g_na_ptr[dev] = base;
  }
  SnfState* st = (SnfState*)(base + kOffState);
  unsigned long long* clk = (unsigned long long*)(base + kOffClock);
  SnfState* sh = &g_na_state[dev];
  init_state(sh, n, params, scheme, SNF_P_FP64);
  const int per_it = products_per_iteration(scheme, params->poly_i, params->poly_j);
  const int max_steps = (params->max_iter + 1) * per_it + 1;
  int cus = 0;
  NA_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int tile = noalloc_tile(n, cus, kNaMaxLd);
  if (!tile || direct_stride(n, tile) > kNaMaxLd) return SNF_ESIZE;
  hipLaunchKernelGGL(na_clock_kernel, dim3(1), dim3(64), 0, s, clk);
  bool in_wg = solve_wg_bytes(n, scheme) > 0;
  if (in_wg && launch_solve_wg(*sh, F_dev, ld, D_dev, ld, st, max_steps, s) != 0) {
    (void)hipGetLastError();    // the device refused the launch (nothing ran): the direct steps
    in_wg = false;
  }
  if (!in_wg) {
    // The iterate buffers hold kNaMatrix values each; the kernels index rows with this call's
    // stride, and every entry they read is written before (f_0 writes all of X_0 including its
    // zero padding, every step all of its output), so nothing left by an earlier call needs
    // clearing.
    DirectArgs a;
    for (int i = 0; i < 4; ++i) {
      a.bufs.x[i] = base + kOffX + (size_t)i * kNaMatrix;
      a.bufs.lp[i] = nullptr;
    }
    a.hdr = (SnfHeader*)(base + kOffHdr);
    a.log = st->log;
    a.partials = base + kOffPartials;
    a.progress = nullptr;
    a.n = n;
    a.ld = direct_stride(n, tile);
    a.nt = (int)((n + tile - 1) / tile);
    launch_direct_f0(a, *sh, F_dev, ld, s);
    StepOperands ops(scheme, per_it);
    int enq = 0;
    bool stopped = false;
    while (!stopped && enq <= max_steps) {
      for (int k = 0; k < 8 && enq <= max_steps; ++k, ++enq) {
        int op[3];
        ops.next(op);
        launch_direct_step(tile, a, enq, op, s);
      }
      NA_HIP(hipGetLastError());
      // a synchronous read of the stop flag (no pinned staging, no events)
      NA_HIP(hipMemcpyAsync(&g_na_flag[dev], &a.hdr[enq & 1].stop, sizeof(int32_t),
                            hipMemcpyDeviceToHost, s));
      NA_HIP(hipStreamSynchronize(s));
      stopped = g_na_flag[dev] != 0;
    }
    launch_direct_out(a, enq & 1, D_dev, ld, st, s);
  }
  hipLaunchKernelGGL(na_clock_kernel, dim3(1), dim3(64), 0, s, clk + 1);
  NA_HIP(hipGetLastError());
  NA_HIP(hipMemcpyAsync(sh, st, sizeof(SnfState), hipMemcpyDeviceToHost, s));
  unsigned long long ticks[2] = {0, 0};
  NA_HIP(hipMemcpyAsync(ticks, clk, sizeof(ticks), hipMemcpyDeviceToHost, s));
  NA_HIP(hipStreamSynchronize(s));
  const int status = sh->stop ? sh->status : SNF_ENOCONV;
  fill_result(sh, out, log, log_cap);
  out->status = status;
  if (status == SNF_EDEVICE) return record_hip_error(hipErrorUnknown, "a step's operands");
  int khz = 0;
  if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) == hipSuccess && khz > 0)
    out->device_ms = (double)(ticks[1] - ticks[0]) / (double)khz;
  return status;
}

}  // namespace
}  // namespace snf

using namespace snf;

extern "C" {

int snf_purify_dense_noalloc(const double* F_dev, int64_t n, int64_t ld,
                             const snf_params* params, snf_scheme scheme,
                             snf_precision precision, double* D_dev, snf_result* out,
                             snf_log_rec* log, int32_t log_cap, void* stream) {
  if (!out) return SNF_EINVAL;
  memset(out, 0, sizeof(*out));
  int rc = validate(n, params, scheme, precision);
  if (rc == SNF_OK && (!F_dev || !D_dev || ld < n || (const void*)F_dev == (const void*)D_dev))
    rc = SNF_EINVAL;
  if (rc == SNF_OK && (precision != SNF_P_FP64 || scheme_is_pij(scheme))) rc = SNF_EINVAL;
  if (rc == SNF_OK && (n + kTile - 1) / kTile * kTile > kNaMaxNp) rc = SNF_ESIZE;
  if (rc != SNF_OK) {
    out->status = rc;
    return rc;
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    out->status = SNF_EDEVICE;
    return SNF_EDEVICE;
  }
  std::lock_guard<std::mutex> guard(g_na_mu[dev]);
  rc = na_body(F_dev, n, ld, params, scheme, D_dev, out, log, log_cap, (hipStream_t)stream,
               dev);
  out->status = rc;
  return rc;
}

}  // extern "C"
