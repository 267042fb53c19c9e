// lanes.h -- exchange between adjacent lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>

namespace mfc {

// Exchange between adjacent lanes of a wave (DPP wave_shr:1 / wave_shl:1):
// lane i receives lane i-1's value (kFromPrev) or lane i+1's (kFromNext); the
// lane at the end with no source receives 0.  Called with every lane active.
constexpr int kFromPrev = 0x138;
constexpr int kFromNext = 0x130;
template <int CTRL>
__device__ __forceinline__ double lane_shift(double x) {
  const long long bits = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(bits & 0xffffffffll), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

}  // namespace mfc
