// Eight elements of a row of d as one lane of the decode-attention kernel holds them (one 16- or 32-byte piece): loads and the
// product of two pieces; and sums over groups of 8 or 16 lanes.
#ifndef LAQ_LANEGROUP_H
#define LAQ_LANEGROUP_H

#include "laq_internal.h"

namespace laq {

// Eight consecutive elements of a row: raw bits as loaded, widened to fp32 at the point of use.
struct Piece8F32 { float4 a, b; };
struct Piece8BF16 { uint4 r; };

__device__ __forceinline__ void fetch8(const float* p, Piece8F32& x) {
  x.a = *reinterpret_cast<const float4*>(p);
  x.b = *reinterpret_cast<const float4*>(p + 4);
}
__device__ __forceinline__ void fetch8(const uint16_t* p, Piece8BF16& x) { x.r = *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void clear8(Piece8F32& x) { x.a = x.b = make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ __forceinline__ void clear8(Piece8BF16& x) { x.r = make_uint4(0u, 0u, 0u, 0u); }

__device__ __forceinline__ void widen8(const Piece8F32& x, float (&f)[8]) {
  f[0] = x.a.x; f[1] = x.a.y; f[2] = x.a.z; f[3] = x.a.w;
  f[4] = x.b.x; f[5] = x.b.y; f[6] = x.b.z; f[7] = x.b.w;
}
__device__ __forceinline__ void widen8(const Piece8BF16& x, float (&f)[8]) {   // bf16 = the high half of fp32
  f[0] = __uint_as_float(x.r.x << 16); f[1] = __uint_as_float(x.r.x & 0xffff0000u);
  f[2] = __uint_as_float(x.r.y << 16); f[3] = __uint_as_float(x.r.y & 0xffff0000u);
  f[4] = __uint_as_float(x.r.z << 16); f[5] = __uint_as_float(x.r.z & 0xffff0000u);
  f[6] = __uint_as_float(x.r.w << 16); f[7] = __uint_as_float(x.r.w & 0xffff0000u);
}

// Product of two 8-element pieces.  bf16: four two-element dot-product instructions on the raw
// pairs (products and sums in fp32), no widening; fp32: eight fused multiply-adds.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), acc, false);
}
__device__ __forceinline__ float dot8(const Piece8BF16& a, const Piece8BF16& b) {
  float s = dot2_bf16(a.r.x, b.r.x, 0.f);
  s = dot2_bf16(a.r.y, b.r.y, s);
  s = dot2_bf16(a.r.z, b.r.z, s);
  return dot2_bf16(a.r.w, b.r.w, s);
}
__device__ __forceinline__ float dot8(const Piece8F32& a, const Piece8F32& b) {
  float s = a.a.x * b.a.x;
  s = fmaf(a.a.y, b.a.y, s); s = fmaf(a.a.z, b.a.z, s); s = fmaf(a.a.w, b.a.w, s);
  s = fmaf(a.b.x, b.b.x, s); s = fmaf(a.b.y, b.b.y, s); s = fmaf(a.b.z, b.b.z, s);
  return fmaf(a.b.w, b.b.w, s);
}

template <typename T> struct PieceOf;
template <> struct PieceOf<float> { using type = Piece8F32; };
template <> struct PieceOf<uint16_t> { using type = Piece8BF16; };

// lane selections within 16 lanes
template <int CTRL>
__device__ __forceinline__ float lane_select(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// One step of group_reduce: lanes whose BIT differs (lane selection CTRL) exchange half of N values, or, with
// one value left, add them.
template <int CTRL, int BIT, int N, int NV>
__device__ __forceinline__ void reduce_step(float (&x)[NV], int lane) {
  if constexpr (N > 1) {
    const bool upper = lane & BIT;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const float lo = x[i], hi = x[i + N / 2];
      const float keep = upper ? hi : lo, give = upper ? lo : hi;
      x[i] = keep + lane_select<CTRL>(give);
    }
  } else {
    x[0] += lane_select<CTRL>(x[0]);
  }
}
// Sums over the RP (8 or 16) lanes of a group for NV values: lane l of the group ends with value
// l * NV / RP (NV <= RP).
template <int RP, int NV>
__device__ __forceinline__ float group_reduce(float (&x)[NV], int lane) {
  static_assert(NV <= RP && (NV & (NV - 1)) == 0, "");
  constexpr int N8 = RP == 16 ? (NV > 1 ? NV / 2 : 1) : NV, N4 = N8 > 1 ? N8 / 2 : 1, N2 = N4 > 1 ? N4 / 2 : 1;
  if constexpr (RP == 16) reduce_step<0x128, 8, NV>(x, lane);      // rotate by 8: lane ^ 8
  reduce_step<0x141, 4, N8>(x, lane);                              // mirror of 8 lanes: lane ^ 7
  reduce_step<0x4E, 2, N4>(x, lane);                               // lane ^ 2
  reduce_step<0xB1, 1, N2>(x, lane);                               // lane ^ 1
  return x[0];
}

}  // namespace laq
#endif  // LAQ_LANEGROUP_H
