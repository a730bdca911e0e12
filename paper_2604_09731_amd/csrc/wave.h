// Wavefront helpers shared by the kernels that plan for themselves.
#ifndef SMART_WAVE_H_
#define SMART_WAVE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace smart {

__device__ inline int64_t readlane64(int64_t v, int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)v >> 32), lane);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// A value every lane agrees on, moved to scalar registers.
__device__ inline int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Inclusive add scan over the 64 lanes with data-parallel-primitive moves (no LDS traffic):
// shifts by 1, 2, 4, 8 inside each row of 16 lanes, then lane 15 of rows 0 and 2 is added to
// rows 1 and 3, then lane 31 to the upper half.  Lanes without a source add zero.
template <int kCtrl, int kRowMask>
__device__ inline int64_t dpp_add(int64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, kCtrl, kRowMask, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)v >> 32), kCtrl, kRowMask, 0xf, false);
  return v + (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// One wavefront: exclusive scan of v and (uniform) the total.
__device__ inline int64_t wave_excl_scan(int64_t v, int lane, int64_t* total) {
  int64_t incl = v;
  incl = dpp_add<0x111, 0xf>(incl);  // row_shr:1
  incl = dpp_add<0x112, 0xf>(incl);  // row_shr:2
  incl = dpp_add<0x114, 0xf>(incl);  // row_shr:4
  incl = dpp_add<0x118, 0xf>(incl);  // row_shr:8
  incl = dpp_add<0x142, 0xa>(incl);  // row_bcast:15 into rows 1 and 3
  incl = dpp_add<0x143, 0xc>(incl);  // row_bcast:31 into rows 2 and 3
  *total = readlane64(incl, 63);
  return incl - v;
}

}  // namespace smart
#endif
