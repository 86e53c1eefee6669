// 1 / x, 1 / sqrt(x) and sqrt(x) of positive numbers in the normal range (with
// room for their squares), to rounding: the hardware's estimates (24 bits)
// and Newton or Goldschmidt steps.  The library forms also cover subnormal
// and infinite arguments, and their longer chains are the critical path of
// the rotation and reflector parameters.
#pragma once
#include <hip/hip_runtime.h>

namespace tn {

__device__ __forceinline__ double fast_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double fast_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}
__device__ __forceinline__ double fast_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double s = x * y, hy = 0.5 * y;  // s -> sqrt(x), hy -> 1 / (2 sqrt(x))
  const double r = fma(-s, hy, 0.5);
  s = fma(s, r, s);
  hy = fma(hy, r, hy);
  return fma(fma(-s, s, x), hy, s);
}

}  // namespace tn
