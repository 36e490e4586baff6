// Tiles and row strides of the FP64 direct steps (kernels_dense.hip).  Host arithmetic only, so that
// it is checked without a GPU.
#pragma once

#include <stdint.h>

namespace snf {

constexpr int kDirectThreads = 256;   // threads of a step's column group
constexpr int kDirectSlots = 512;     // partial-sum slots per step parity (f_0's blocks, tiles)

// Work of one workgroup per step: a TxT output tile of the upper triangle, T the smallest of
// 32, 48, 64, 80, 96 whose tiles number at most one per compute unit; 0: no such T.
inline int direct_tile(int64_t n, int num_cus) {
  if (num_cus > kDirectThreads) num_cus = kDirectThreads;   // (a step sums a slot per thread)
  for (int t = 32; t <= 96; t += 16) {
    const int64_t nt = (n + t - 1) / t;
    if (nt * (nt + 1) / 2 <= num_cus) return t;
  }
  return 0;
}

// Row stride of the iterate buffers for that T (a multiple of 16, at least T ceil(n / T)).
inline int64_t direct_stride(int64_t n, int tile) {
  const int64_t w = (n + tile - 1) / tile * tile;
  // rows a multiple of 2 KB apart would put the rows of one load on the same channels
  return w % 256 ? w : w + 16;
}

// The longest rows that the direct steps may take for order n on any device, 0 beyond their range.
inline int64_t direct_max_stride(int64_t n) {
  int64_t ld = 0;
  for (int t = 32; t <= 96; t += 16) {
    const int64_t nt = (n + t - 1) / t;
    if (nt * (nt + 1) / 2 <= kDirectThreads && direct_stride(n, t) > ld) ld = direct_stride(n, t);
  }
  return ld;
}

// The tile of snf_purify_dense_noalloc, whose buffers hold rows of max_ld values and which has no
// other path: that of snf_purify_dense, or, where the device has too few compute units for one
// (a part of a partitioned GPU) or the rows do not fit, what 256 units would take.  A step needs no
// two of its workgroups at once, so the tiles beyond the units wait their turn.
inline int noalloc_tile(int64_t n, int num_cus, int64_t max_ld) {
  const int t = direct_tile(n, num_cus);
  return t && direct_stride(n, t) <= max_ld ? t : direct_tile(n, kDirectThreads);
}

}  // namespace snf
