// Wave-level reductions shared by the latency-bound kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace rif {

// x moved within each row of 16 lanes; every lane of the controls used here has a
// source, so no lane needs an old value.
template <int kCtrl>
__device__ __forceinline__ double dpp_move(double x) {
  const long long u = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, kCtrl, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), kCtrl, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_value(double x, int l) {
  const long long u = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)u, l), hi = __builtin_amdgcn_readlane((int)(u >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// The values of rows 0 and 2 (kHalves: lanes 0 - 31) in a, of rows 1 and 3 (lanes
// 32 - 63) in b, each in both places of the pair.
template <bool kHalves>
__device__ __forceinline__ void pair_values(double x, double& a, double& b) {
  const long long u = __double_as_longlong(x);
  const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
  const auto l = kHalves ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                         : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h = kHalves ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                         : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  a = __longlong_as_double(((long long)h[0] << 32) | (unsigned)l[0]);
  b = __longlong_as_double(((long long)h[1] << 32) | (unsigned)l[1]);
}
// Sum over the 64 lanes (all active), the same bits in every lane and every
// call: within each row of 16 lanes by DPP moves (swap neighbours, swap pairs,
// mirror, rotate by 8), then (row 0 + row 1) + (row 2 + row 3) by lane swaps.
// A chain of six additions; with the row sums read into scalars and added there an
// orbital step at n_bf 348 took 1587 us instead of 1573.
__device__ __forceinline__ double wave_sum_dpp(double x) {
  x += dpp_move<0xB1>(x);    // quad_perm [1,0,3,2]
  x += dpp_move<0x4E>(x);    // quad_perm [2,3,0,1]
  x += dpp_move<0x140>(x);   // row_mirror: quads 0 and 3, 1 and 2
  x += dpp_move<0x128>(x);   // row_ror:8
  double a, b;
  pair_values<false>(x, a, b);
  x = a + b;
  pair_values<true>(x, a, b);
  return a + b;
}

// Max over the 64 lanes (all active) of doubles (NaN lanes ignored, as fmax
// does) and min of ints, every lane getting the result; both are
// order-free, so every wave gets the same value.
__device__ __forceinline__ double wave_max_dpp(double x) {
  x = fmax(x, dpp_move<0xB1>(x));
  x = fmax(x, dpp_move<0x4E>(x));
  x = fmax(x, dpp_move<0x124>(x));
  x = fmax(x, dpp_move<0x128>(x));
  double a, b;
  pair_values<false>(x, a, b);
  x = fmax(a, b);
  pair_values<true>(x, a, b);
  return fmax(a, b);
}
__device__ __forceinline__ int wave_min_int_dpp(int x) {
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false));
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false));
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xF, 0xF, false));
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, false));
  return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

}  // namespace rif
