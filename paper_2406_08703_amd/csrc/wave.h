// Sums over a wave of 64 lanes.
#pragma once

#include <hip/hip_runtime.h>

namespace dlx {

// v moved by one DPP step (no source: 0)
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// Sum over the 64 lanes (all active), valid in lane 63; always in the same order.
__device__ __forceinline__ double wave_total(double v) {
  v = dpp_add<0x111>(v);   // row_shr:1
  v = dpp_add<0x112>(v);   // row_shr:2
  v = dpp_add<0x114>(v);   // row_shr:4
  v = dpp_add<0x118>(v);   // row_shr:8
  v = dpp_add<0x142>(v);   // row_bcast:15
  return dpp_add<0x143>(v);   // row_bcast:31
}

// Largest of the 64 lanes' values (all active, none negative), the same in every lane.
__device__ __forceinline__ int wave_max(int v) {
#define DLX_MAX_STEP(CTRL) v = max(v, __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true))
  DLX_MAX_STEP(0x111);   // row_shr:1
  DLX_MAX_STEP(0x112);   // row_shr:2
  DLX_MAX_STEP(0x114);   // row_shr:4
  DLX_MAX_STEP(0x118);   // row_shr:8
  DLX_MAX_STEP(0x142);   // row_bcast:15
  DLX_MAX_STEP(0x143);   // row_bcast:31
#undef DLX_MAX_STEP
  return __builtin_amdgcn_readlane(v, 63);
}

}  // namespace dlx
