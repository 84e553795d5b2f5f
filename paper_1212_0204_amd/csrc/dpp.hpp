// dpp.hpp -- moves of FP64 values between the lanes of a wavefront by the
// ALU's cross-lane controls (no LDS): shifts by one lane and the maximum.
#pragma once
#include <hip/hip_runtime.h>

namespace hofks {

// v of the lane that DPP control CTRL selects (rows in ROW_MASK; lanes
// without a source keep v)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, ROW_MASK, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, ROW_MASK, 0xF,
                                             false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_max(double v) {
  return fmax(v, dpp_move<CTRL, ROW_MASK>(v));
}

// v of lane - 1 (lane 0: zero) and of lane + 1 (lane 63: zero)
template <int CTRL>
__device__ __forceinline__ double dpp_shift(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_prev(double v) { return dpp_shift<0x138>(v); }
__device__ __forceinline__ double lane_next(double v) { return dpp_shift<0x130>(v); }

// v of lane l, in every lane (l the same for the whole wavefront)
__device__ __forceinline__ double lane_value(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// maximum over the wavefront, in every lane: row shifts by 1, 2, 4 and 8
// leave each row's maximum in its lane 15, the row broadcasts carry rows 0
// and 2 into rows 1 and 3 and then row 1 into rows 2 and 3, and lane 63 is
// read back (cross-lane moves of the ALU instead of LDS permutes)
__device__ __forceinline__ double wave_max_dpp(double v) {
  v = dpp_max<0x111, 0xF>(v);
  v = dpp_max<0x112, 0xF>(v);
  v = dpp_max<0x114, 0xF>(v);
  v = dpp_max<0x118, 0xF>(v);
  v = dpp_max<0x142, 0xA>(v);
  v = dpp_max<0x143, 0xC>(v);
  return lane_value(v, 63);
}

}  // namespace hofks
