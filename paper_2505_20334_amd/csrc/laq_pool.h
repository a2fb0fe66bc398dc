// Sequence pooling of four neighbouring scores per lane, for the kernels that hold scores that way.
#pragma once

#include <type_traits>

#include "laq_internal.h"

namespace laq {

// Windows of up to SELECT_POOL_MAX_HALF scores to either side.  Scores are never negative: a zero stands for "not in the window",
// and leaves a maximum and an ascending sum as they are.
__device__ __forceinline__ float lane_before(float old, float x) {       // lane l: x of lane l - 1; lane 0: old
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_after(float old, float x) {        // lane l: x of lane l + 1; lane 63: old
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), 0x130, 0xf, 0xf, false));
}

// own: the lane's quad.  The quads beside it come from the neighbouring lanes; before1 and before2 are, for lane 0, the one before its own
// and the one before that, after1 and after2 for lane 63 those after.  Only the elements of the window are fetched, and a maximum shares
// what the four windows have in common.
template <int H>
__device__ __forceinline__ float4 pool_quad_of(float4 own, float4 before1, float4 before2, float4 after1, float4 after2, bool avg) {
  float w[20];                                   // w[8 .. 11]: own; of the others those in a window
  const float o[4] = {own.x, own.y, own.z, own.w}, b1[4] = {before1.x, before1.y, before1.z, before1.w},
              b2[4] = {before2.x, before2.y, before2.z, before2.w}, a1[4] = {after1.x, after1.y, after1.z, after1.w},
              a2[4] = {after2.x, after2.y, after2.z, after2.w};
#pragma unroll
  for (int c = 0; c < 4; ++c) w[8 + c] = o[c];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (4 + c >= 8 - H) w[4 + c] = lane_before(b1[c], o[c]);
    if (12 + c <= 11 + H) w[12 + c] = lane_after(a1[c], o[c]);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (c >= 8 - H) w[c] = lane_before(b2[c], w[4 + c]);
    if (16 + c <= 11 + H) w[16 + c] = lane_after(a2[c], w[12 + c]);
  }
  float r[4];
  if (avg) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float v = 0.f;
#pragma unroll
      for (int i = -H; i <= H; ++i) v += w[8 + c + i];
      r[c] = v / (float)(2 * H + 1);
    }
  } else if (H == 1) {
    const float m = fmaxf(w[9], w[10]);
    r[0] = fmaxf(fmaxf(w[7], w[8]), w[9]);
    r[1] = fmaxf(w[8], m);
    r[2] = fmaxf(m, w[11]);
    r[3] = fmaxf(fmaxf(w[10], w[11]), w[12]);
  } else {
    float m = w[11 - H];                         // 11 - H .. 8 + H: in all four
#pragma unroll
    for (int i = 12 - H; i <= 8 + H; ++i) m = fmaxf(m, w[i]);
    const float a = fmaxf(w[9 - H], w[10 - H]), b = fmaxf(w[9 + H], w[10 + H]);
    r[0] = fmaxf(fmaxf(m, w[8 - H]), a);
    r[1] = fmaxf(fmaxf(m, a), w[9 + H]);
    r[2] = fmaxf(fmaxf(m, w[10 - H]), b);
    r[3] = fmaxf(fmaxf(m, b), w[11 + H]);
  }
  return make_float4(r[0], r[1], r[2], r[3]);
}
// f(half as a constant): the window's width is the same for a whole launch, and a test per element would cost more than the copies of f
template <typename F>
__device__ __forceinline__ void for_half(int half, F&& f) {
  switch (half) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    default: return f(std::integral_constant<int, 8>{});
  }
}

}  // namespace laq
