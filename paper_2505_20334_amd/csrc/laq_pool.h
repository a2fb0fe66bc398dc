// Sequence pooling of four neighbouring scores per lane, for the kernels that hold scores that way.
#pragma once

#include "laq_internal.h"

namespace laq {

// Scores are never negative: a zero stands for "not in the window", and leaves a maximum and an ascending sum as they are.
constexpr int POOL_QUAD_MAX_HALF = 8;            // widest window: two quads beside a lane's own on either side

__device__ __forceinline__ float lane_before(float old, float x) {       // lane l: x of lane l - 1; lane 0: old
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_after(float old, float x) {        // lane l: x of lane l + 1; lane 63: old
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), 0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ float4 lane_before(float4 old, float4 x) {
  return make_float4(lane_before(old.x, x.x), lane_before(old.y, x.y), lane_before(old.z, x.z), lane_before(old.w, x.w));
}
__device__ __forceinline__ float4 lane_after(float4 old, float4 x) {
  return make_float4(lane_after(old.x, x.x), lane_after(old.y, x.y), lane_after(old.z, x.z), lane_after(old.w, x.w));
}

// q[2] is the lane's own quad, q[0] .. q[4] the five around it
template <int H>
__device__ __forceinline__ float4 pool_quad_of(const float4 (&q)[5], bool avg) {
  const float w[20] = {q[0].x, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y, q[1].z, q[1].w, q[2].x, q[2].y, q[2].z, q[2].w,
                       q[3].x, q[3].y, q[3].z, q[3].w, q[4].x, q[4].y, q[4].z, q[4].w};
  float r[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float v;
    if (avg) {
      v = 0.f;
#pragma unroll
      for (int o = -H; o <= H; ++o) v += w[8 + c + o];
      v /= (float)(2 * H + 1);
    } else {
      v = w[8 + c];
#pragma unroll
      for (int o = -H; o <= H; ++o) v = fmaxf(v, w[8 + c + o]);
    }
    r[c] = v;
  }
  return make_float4(r[0], r[1], r[2], r[3]);
}
// (the window's width is the same for a whole launch: the branch costs next to nothing, what it avoids is a test per element)
__device__ __forceinline__ float4 pool_quad(const float4 (&q)[5], int half, bool avg) {
  switch (half) {
    case 1: return pool_quad_of<1>(q, avg);
    case 2: return pool_quad_of<2>(q, avg);
    case 3: return pool_quad_of<3>(q, avg);
    case 4: return pool_quad_of<4>(q, avg);
    case 5: return pool_quad_of<5>(q, avg);
    case 6: return pool_quad_of<6>(q, avg);
    case 7: return pool_quad_of<7>(q, avg);
    default: return pool_quad_of<8>(q, avg);
  }
}

}  // namespace laq
