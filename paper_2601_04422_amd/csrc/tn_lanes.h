// Movement of float64 values between the lanes of a wavefront.
#pragma once
#include <hip/hip_runtime.h>

namespace tn {

// Value of lane (l + N) mod 16 of the same row of 16 lanes: a register move
// with a DPP row rotation (to the right by 16 - N lanes), no LDS traffic.
template <int N>
__device__ __forceinline__ double row_next(double x) {
  static_assert(N > 0 && N < 16, "a rotation inside a row of 16 lanes");
  constexpr int ctrl = 0x120 + (16 - N);  // row_ror:(16 - N)
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), ctrl, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), ctrl, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
template <int N>
__device__ __forceinline__ double2 row_next(double2 x) {
  return make_double2(row_next<N>(x.x), row_next<N>(x.y));
}

}  // namespace tn
