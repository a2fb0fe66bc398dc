// Products of key rows and score rows on the matrix cores, for the kernels that hold 32 key rows per wave in operand layout
// (lane l: row l % 32, the 16-byte pieces 2t + l / 32) and the score rows in LDS.
//
// fp32 takes six bf16 products: a float is the sum of three bf16 (split8), and the three products of parts that together reach
// 2^-24 of the whole at most are left out.
#pragma once

#include <cmath>

#include "laq_internal.h"
#include "laq_staging.h"

namespace laq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr float NEG_BIG = -1.0e30f;   // finite "minus infinity" for running maxima
// The exponential instruction returns 0 below 2^-126, where fp32 still tells scores apart: a score below TINY is summed again
// with the exponents of its terms raised (above it, what is lost is less than a rounding).
constexpr float TINY = 0x1p-90f;

// Row index (0..31) of accumulator register i for a lane in half hf of the 32x32 output layout.
__device__ __forceinline__ int acc_row(int i, int hf) { return 8 * (i >> 2) + 4 * hf + (i & 3); }

// Eight floats as the sums of three bf16 each, rounded to the nearest: the second part is at most 2^-8 and the third at most 2^-17
// of the float, nothing is left over, and the signs of the smaller parts do not follow that of the float.  (Cut off instead, the
// smaller parts reach 2^-7 and 2^-15 and what is left out of a product is up to 2^-21 of it, always to the side of its sign.  As many
// instructions, but slower ones: short heads 1.00 to 1.04 times as long, 64 heads x 8191 keys as long.)
struct Split { u32x4 p[3]; };
__device__ __forceinline__ Split split8(u32x4 a, u32x4 b) {
  float x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = __uint_as_float(i < 4 ? a[i] : b[i - 4]);
  Split s;
#pragma unroll
  for (int pl = 0; pl < 3; ++pl) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (pl == 2) {                       // (8 bits are left, at most)
        s.p[pl][i] = __builtin_amdgcn_perm(__float_as_uint(x[2 * i + 1]), __float_as_uint(x[2 * i]), 0x07060302u);
      } else {
        const unsigned both = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{x[2 * i], x[2 * i + 1]}), bf16x2));
        s.p[pl][i] = both;
        x[2 * i] -= __uint_as_float(both << 16);
        x[2 * i + 1] -= __uint_as_float(both & 0xffff0000u);
      }
    }
  }
  return s;
}
__device__ __forceinline__ f32x16 mfma(u32x4 a, u32x4 b, f32x16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

constexpr bool is_f32(float) { return true; }
constexpr bool is_f32(uint16_t) { return false; }

// from one staged score row to the next: bf16 as it is, fp32 as three rows of bf16
template <typename T> constexpr int row_stride(int d) { return staged_row(d, is_f32(T()) ? 3 : 1); }
template <typename T> constexpr int row16_stride(int d) { return staged_row16(d, is_f32(T()) ? 3 : 1); }

// The product of fp32 rows by the fp32 instruction, from memory: where the split one holds a NaN (a part of an infinity is one).
template <bool KEYS_AS_ROWS>
__device__ __forceinline__ f32x16 product_f32(const char* key, const char* q, int hf, int row_bytes) {
  f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int o = hf * 16; o < row_bytes + hf * 16; o += 32) {     // (both halves as often: the last piece of the upper one may be missing)
    f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
    if (o < row_bytes) {
      x = *reinterpret_cast<const f32x4*>(key + o);
      y = *reinterpret_cast<const f32x4*>(q + o);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc = KEYS_AS_ROWS ? __builtin_amdgcn_mfma_f32_32x32x2f32(x[j], y[j], acc, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x2f32(y[j], x[j], acc, 0, 0, 0);
  }
  return acc;
}

template <bool KEYS_AS_ROWS>
__device__ __forceinline__ f32x16 mm(u32x4 key, u32x4 q, f32x16 acc) { return KEYS_AS_ROWS ? mfma(key, q, acc) : mfma(q, key, acc); }

__device__ __forceinline__ void merge_stat(float& M, float& Z, float2 p) {
  const float Mn = fmaxf(M, p.x);
  Z = Z * __builtin_amdgcn_exp2f(M - Mn) + p.y * __builtin_amdgcn_exp2f(p.x - Mn);
  M = Mn;
}

// fp32 score rows are split into bf16 parts times 2^shift; their products then take scale2 * 2^-shift, which is 2^-28
// to 2^-27.  The parts of a float below 2^-103 reach numbers that bf16 does not hold or the matrix cores take for 0: an element loses
// less than 2^-126.  Times that scale and the other factor, a key or a staged element below 2^128, it is less than 2^-25 of an
// exponent whatever the magnitudes of keys, queries and scale.  What is larger is infinite, and taken from whole floats; the
// products become infinite at exponents from 2^100 on, beyond the smallest maximum the kernels know.  bf16: 0 and scale2.
// (An argument of its own: as members of the geometry they move the arguments of all kernels, and the single-read one took 2 us of 289 longer;
// made in the kernels it costs registers, 800 fp32 heads of 300 keys 60 us instead of 57.)
struct RowScale {
  int shift;
  float scale2;
};
template <typename T> RowScale row_scale_of(float scale2) {
  int exponent = 0;
  if (is_f32(T())) frexpf(scale2, &exponent);
  const int shift = is_f32(T()) ? 27 + exponent : 0;
  return RowScale{shift, ldexpf(scale2, -shift)};
}

// Score rows r0 .. r0 + n - 1 of a head to LDS, `stride` bytes apart (rows beyond R: the last one again); fp32: times
// 2^shift (RowScale).
template <typename T, bool FULL, int THREADS>
__device__ __forceinline__ void stage_rows(char* lds, const char* head_rows, int row_bytes, int plane, int stride, int R, int r0, int n,
                                           int shift) {
  const int tid = threadIdx.x, per = plane / 16, total = n * per;
#pragma unroll(is_f32(T()) ? 2 : 4)
  for (int p = tid; p < total; p += THREADS) {
    const int row = p / per, col = p - row * per;
    const char* src = head_rows + (size_t)min(r0 + row, R - 1) * row_bytes;
    if constexpr (!is_f32(T())) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (FULL || col * 16 < row_bytes) v = *reinterpret_cast<const u32x4*>(src + col * 16);
      *reinterpret_cast<u32x4*>(lds + row * stride + col * 16) = v;
    } else {
      // 8 elements as the key side has them: pieces 2t + hf and 2(t + 1) + hf
      const int a = (col >> 1) * 4 + (col & 1);
      u32x4 x = {0u, 0u, 0u, 0u}, y = {0u, 0u, 0u, 0u};
      if (FULL || a * 16 < row_bytes) x = *reinterpret_cast<const u32x4*>(src + a * 16);
      if (FULL || (a + 2) * 16 < row_bytes) y = *reinterpret_cast<const u32x4*>(src + (a + 2) * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = __float_as_uint(__builtin_amdgcn_ldexpf(__uint_as_float(x[i]), shift));
        y[i] = __float_as_uint(__builtin_amdgcn_ldexpf(__uint_as_float(y[i]), shift));
      }
      const Split s = split8(x, y);
#pragma unroll
      for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4*>(lds + row * stride + pl * plane + col * 16) = s.p[pl];
    }
  }
}

// ---- tiles of 16 x 16 (v_mfma_f32_16x16x32_bf16) ----
// 32 keys by 32 score rows as four of them, t[key half][row half].  Lane l supplies row l % 16 of either operand and the 16-byte pieces
// 4t + l / 16 of it, and holds, of column l % 16 of a tile, rows 4 (l / 16) .. + 3.
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <bool KEYS_AS_ROWS>
__device__ __forceinline__ f32x4 mm16(u32x4 key, u32x4 q, f32x4 acc) { return KEYS_AS_ROWS ? mfma16(key, q, acc) : mfma16(q, key, acc); }
struct Tile16 {
  f32x4 t[2][2];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
};
// Two values combined over the four lanes of the same number modulo 16: lanes 0 .. 31 end with the first one, the others with the second.
template <typename OP>
__device__ __forceinline__ float over_groups(float x, float y, OP op) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const float w = op(__uint_as_float(h[0]), __uint_as_float(h[1]));
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(w), __float_as_uint(w), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// product_f32() of the tiles: key[s], q[r] are this lane's rows
template <bool KEYS_AS_ROWS>
__device__ __forceinline__ Tile16 product16_f32(const char* const (&key)[2], const char* const (&q)[2], int grp, int row_bytes) {
  Tile16 a;
  a.clear();
#pragma unroll 1
  for (int o = grp * 16; o < row_bytes + grp * 16; o += 64) {   // (every group of lanes as often: the last pieces of some may be missing)
    f32x4 x[2], y[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      x[i] = y[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (o < row_bytes) {
        x[i] = *reinterpret_cast<const f32x4*>(key[i] + o);
        y[i] = *reinterpret_cast<const f32x4*>(q[i] + o);
      }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          a.t[s][r] = KEYS_AS_ROWS ? __builtin_amdgcn_mfma_f32_16x16x4f32(x[s][j], y[r][j], a.t[s][r], 0, 0, 0)
                                   : __builtin_amdgcn_mfma_f32_16x16x4f32(y[r][j], x[s][j], a.t[s][r], 0, 0, 0);
  }
  return a;
}

// stage_rows() for the products of 16 x 16 tiles
template <typename T, bool FULL, int THREADS>
__device__ __forceinline__ void stage_rows16(char* lds, const char* head_rows, int row_bytes, int plane, int stride, int R, int r0, int n,
                                           int shift) {
  const int tid = threadIdx.x, per = plane / 16, total = n * per;
#pragma unroll(is_f32(T()) ? 2 : 4)
  for (int p = tid; p < total; p += THREADS) {
    const int row = p / per, col = p - row * per;
    const char* src = head_rows + (size_t)min(r0 + row, R - 1) * row_bytes;
    if constexpr (!is_f32(T())) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (FULL || col * 16 < row_bytes) v = *reinterpret_cast<const u32x4*>(src + col * 16);
      *reinterpret_cast<u32x4*>(lds + row * stride + col * 16) = v;
    } else {
      // 8 elements as the key side has them: pieces 8t + grp and 8t + 4 + grp
      const int a = (col >> 2) * 8 + (col & 3);
      u32x4 x = {0u, 0u, 0u, 0u}, y = {0u, 0u, 0u, 0u};
      if (FULL || a * 16 < row_bytes) x = *reinterpret_cast<const u32x4*>(src + a * 16);
      if (FULL || (a + 4) * 16 < row_bytes) y = *reinterpret_cast<const u32x4*>(src + (a + 4) * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = __float_as_uint(__builtin_amdgcn_ldexpf(__uint_as_float(x[i]), shift));
        y[i] = __float_as_uint(__builtin_amdgcn_ldexpf(__uint_as_float(y[i]), shift));
      }
      const Split s = split8(x, y);
#pragma unroll
      for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4*>(lds + row * stride + pl * plane + col * 16) = s.p[pl];
    }
  }
}

}  // namespace laq
