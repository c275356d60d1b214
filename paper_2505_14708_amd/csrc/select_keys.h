// What the selections share on the device.
#pragma once
#include <hip/hip_runtime.h>

namespace da {

// scores as unsigned keys of the same order
__device__ inline unsigned order_key(float x) {
  unsigned u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;       // NaN ranks below everything
  if ((u & 0x7fffffffu) == 0u) u = 0u;                  // -0 == +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// number of set bits of `m` strictly below this lane
__device__ inline int lane_prefix(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
}

}  // namespace da
