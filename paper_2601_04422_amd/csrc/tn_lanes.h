// Movement of float64 values between the lanes of a wavefront.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

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

// Value of lane 15 - l of the row of 16 lanes, in registers.
__device__ __forceinline__ double row_mirror(double x) {
  return __hiloint2double(
      __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x140, 0xF, 0xF, true),
      __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x140, 0xF, 0xF, true));
}
__device__ __forceinline__ double2 row_mirror(double2 x) {
  return make_double2(row_mirror(x.x), row_mirror(x.y));
}

// Value of lane l ^ 16 (rows of 16 lanes exchanged in pairs), in registers.
__device__ __forceinline__ double swap_rows(double x) {
  const bool odd = threadIdx.x & 16;
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
  return __hiloint2double(odd ? hi[0] : hi[1], odd ? lo[0] : lo[1]);
}
__device__ __forceinline__ double2 swap_rows(double2 x) {
  return make_double2(swap_rows(x.x), swap_rows(x.y));
}

// Value of lane l ^ 4: row_shl:4 into the even quads of a row, row_shr:4 into
// the odd ones.
__device__ __forceinline__ double quad_swap(double x) {
  auto one = [](int v) {
    const int y = __builtin_amdgcn_update_dpp(0, v, 0x104, 0xF, 0x5, false);
    return __builtin_amdgcn_update_dpp(y, v, 0x114, 0xF, 0xA, false);
  };
  return __hiloint2double(one(__double2hiint(x)), one(__double2loint(x)));
}

// Sum over the 64 lanes, in every lane, with the additions of a halving
// reduction.
__device__ __forceinline__ double wave_total(double v) {
  auto dpp = [](double x, auto ctrl) {
    constexpr int c = decltype(ctrl)::value;
    return __hiloint2double(
        __builtin_amdgcn_update_dpp(0, __double2hiint(x), c, 0xF, 0xF, true),
        __builtin_amdgcn_update_dpp(0, __double2loint(x), c, 0xF, 0xF, true));
  };
  {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  }
  {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  }
  v += dpp(v, std::integral_constant<int, 0x128>());  // row_ror:8
  v += quad_swap(v);
  v += dpp(v, std::integral_constant<int, 0x4E>());   // quad_perm [2, 3, 0, 1]
  return v + dpp(v, std::integral_constant<int, 0xB1>());
}

// Sums over the 64 lanes of a wavefront of N values per lane (N = 16, 32, 64),
// transposed on the way: lane l ends with the sum of value l / (64 / N).  Each
// step halves the values a lane holds (it keeps one half and hands the other to
// its partner), so N values take about 3 N register operations and no LDS,
// where N separate sums take 6 N exchanges.  With TREE the additions are those
// of a halving reduction (lane l with l ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1), at one
// more move per value in the fourth step.
template <int N, bool TREE = false>
__device__ __forceinline__ double wave_sums(double (&v)[N]) {
  static_assert(N == 16 || N == 32 || N == 64, "one value for whole groups of lanes");
  const int lane = threadIdx.x & 63;
  auto swap32 = [](double &a, double &b) {  // upper half of a <-> lower half of b
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(hi[0], lo[0]);
    b = __hiloint2double(hi[1], lo[1]);
  };
  auto swap16 = [](double &a, double &b) {  // odd rows of a <-> even rows of b
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(hi[0], lo[0]);
    b = __hiloint2double(hi[1], lo[1]);
  };
  auto dpp = [](double x, auto ctrl) {
    constexpr int c = decltype(ctrl)::value;
    return __hiloint2double(
        __builtin_amdgcn_update_dpp(0, __double2hiint(x), c, 0xF, 0xF, true),
        __builtin_amdgcn_update_dpp(0, __double2loint(x), c, 0xF, 0xF, true));
  };
#pragma unroll
  for (int i = 0; i < N / 2; i++) {
    swap32(v[i], v[i + N / 2]);
    v[i] += v[i + N / 2];
  }
#pragma unroll
  for (int i = 0; i < N / 4; i++) {
    swap16(v[i], v[i + N / 4]);
    v[i] += v[i + N / 4];
  }
  // inside a row of 16: partners l ^ 8, then l ^ 7, l ^ 2, l ^ 1 (a mirror of
  // eight lanes also flips the lower bits, which the later steps sum over)
  auto step = [&](int half, bool upper, auto ctrl) {
    if (half == 0) {
      v[0] += dpp(v[0], ctrl);
      return;
    }
#pragma unroll
    for (int i = 0; i < N / 8; i++)
      if (i < half) {
        const double keep = upper ? v[i + half] : v[i], give = upper ? v[i] : v[i + half];
        v[i] = keep + dpp(give, ctrl);
      }
  };
  step(N / 8, lane & 8, std::integral_constant<int, 0x128>());   // row_ror:8
  if constexpr (TREE) {
    const bool up = lane & 4;
#pragma unroll
    for (int i = 0; i < (N / 16 ? N / 16 : 1); i++) {
      const double keep = up ? v[i + N / 16] : v[i], give = up ? v[i] : v[i + N / 16];
      v[i] = keep + quad_swap(give);
    }
  } else {
    step(N / 16, lane & 4, std::integral_constant<int, 0x141>());  // row_half_mirror
  }
  step(N / 32, lane & 2, std::integral_constant<int, 0x4E>());   // quad_perm [2, 3, 0, 1]
  step(N / 64, lane & 1, std::integral_constant<int, 0xB1>());   // quad_perm [1, 0, 3, 2]
  return v[0];
}

// Value of lane `src` (the same for every lane of the wavefront).
__device__ __forceinline__ double lane_value(double x, int src) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), src),
                          __builtin_amdgcn_readlane(__double2loint(x), src));
}

}  // namespace tn
