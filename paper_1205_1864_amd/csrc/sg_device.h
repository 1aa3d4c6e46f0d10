// Device-side helpers shared by the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace sgk {

// Uniform read of a table the kernels never write: through the constant address
// space so that it becomes a scalar load instead of a vector load plus readfirstlane.
template <typename T>
__device__ __forceinline__ T ld_uniform(const T* p, long i) {
  typedef const __attribute__((address_space(4))) T* cptr;
  return ((cptr)(p))[i];
}

// Whole-wavefront lane shifts (DPP wave_shl / wave_shr by one lane): lane i
// receives the value of lane i + 1 (from_next) or i - 1 (from_prev); the lane
// at the end of the wave receives 0.
__device__ __forceinline__ int dpp_from_next(int v) {  // lane i receives lane i + 1
  return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xF, 0xF, true);
}
__device__ __forceinline__ int dpp_from_prev(int v) {  // lane i receives lane i - 1
  return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, true);
}
__device__ __forceinline__ double from_next(double v) {
  const int lo = dpp_from_next(__double2loint(v));
  const int hi = dpp_from_next(__double2hiint(v));
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double from_prev(double v) {
  const int lo = dpp_from_prev(__double2loint(v));
  const int hi = dpp_from_prev(__double2hiint(v));
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float from_next(float v) { return __int_as_float(dpp_from_next(__float_as_int(v))); }
__device__ __forceinline__ float from_prev(float v) { return __int_as_float(dpp_from_prev(__float_as_int(v))); }

// DPP move of a double within rows of 16 lanes (every source lane exists).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double lane_f64(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum over the 64 lanes of a wave, the same in every lane and in a fixed
// order: butterflies within rows of 16 lanes (neighbour in the quad, the
// other pair of the quad, the other quad of each 8, the other 8 of each 16;
// both partners add the same two values), then the four row sums in order.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x140>(v);  // row_mirror
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}

// Exchange of values between running blocks through memory that every compute
// unit sees coherently (agent-scope atomics): a value is its own flag, since the
// place it goes to holds kEmpty before and no value is published with those bits.
constexpr unsigned long long kEmpty = 0x7ff8dead7ff8deadull;  // a NaN
__device__ __forceinline__ void agent_store(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long agent_load(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long publishable(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return b == kEmpty ? 0x7ff8000000000000ull : b;
}

}  // namespace sgk
