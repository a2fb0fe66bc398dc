// A whole head in one workgroup: scores, pooling, selection and gather of a short cache in one launch.
//
// A workgroup of 8 or 16 waves holds all keys of one KV head in registers (operand layout, up to two tiles of 32
// per wave), K is read once, and nothing leaves the workgroup between the steps:
//   products with the score rows (lane = score row, registers = keys), e = exp2(s - m) against the wave's maximum m of the row (a whole number), (m, z) per
//   wave and row -> LDS -> weight exp2(m - M) / Z -> sum of e * weight over the rows, across lanes ->
//   raw scores in LDS -> one position per thread: pooled, ranked (counted in bins), listed -> gather.
// So where the registers hold the e of all score rows (kept_tiles); with more rows, c = M + log2 Z and products and exponentials a second time.
// What bounds it: the latency of one workgroup -- two trips to memory (keys; the rows of V) and a dozen barriers -- and, for fp32, the
// products and the splitting of the keys that the four waves of a SIMD share.  laq_evict, us, products of 32 x 32 and all of them twice : of 16 x 16 and kept:
// fp32, d = 64, 2 heads x 512 keys, 16 rows 15.9 : 13.2, 192 x 500, 64 rows 24.4 : 21.9, 96 x 1000, 32 rows 29.0 : 22.8; bf16, d = 128, 24 x 512, 32 rows
// 13.9 : 12.9, 96 x 1000 19.2 : 18.7, d = 96, 64 x 500, 64 rows 15.3 : 14.2.  Scores against 64 bits (2-norm), bf16, d = 128, 64 rows 1.8e-7 : 4.8e-8.
#include <algorithm>
#include <type_traits>

#include "laq_internal.h"
#include "laq_lanegroup.h"
#include "laq_products.h"
#include "laq_rank.h"

namespace laq {

namespace {

constexpr int MAX_TILES = 4;                 // 32-row tiles of score rows that are staged together
constexpr int MAX_ROWS = 256;                // score rows of a head
constexpr int MARGIN = SELECT_POOL_MAX_HALF;

struct HeadPlan {
  int group_tiles, groups;   // row tiles staged together
  int off_stat;              // bytes of the staged rows
  RowScale row_scale;
};

// the product of 32 keys, held as they lie in memory, with 16 * RH score rows (TIGHT: few registers are left for it)
template <typename T, int NP, bool FULL, bool TIGHT, int RH>
__device__ __forceinline__ Tile16 product16_raw(const u32x4 (&key)[NP], const char* lds, int stride, int plane, int steps) {
  constexpr int PER_ROW = NP / 2;
  Tile16 acc;
  acc.clear();
  if constexpr (is_f32(T())) {
#pragma unroll
    for (int u = 0; u < PER_ROW / 2; ++u) {
      if (FULL || u < steps) {
        // key halves whose parts are there at a time
        constexpr int AT_ONCE = TIGHT ? 1 : 2;
#pragma unroll
        for (int s0 = 0; s0 < 2; s0 += AT_ONCE) {
          Split x[AT_ONCE];
#pragma unroll
          for (int s = 0; s < AT_ONCE; ++s) {
            // (taken apart here, for every product: the registers do not hold the parts)
            u32x4 a = key[(s0 + s) * PER_ROW + 2 * u], b = key[(s0 + s) * PER_ROW + 2 * u + 1];
            asm volatile("" : "+v"(a));
            asm volatile("" : "+v"(b));
            x[s] = split8(a, b);
          }
          constexpr int PARTS[6][2] = {{2, 0}, {0, 2}, {1, 1}, {0, 1}, {1, 0}, {0, 0}};   // (of the key, of the row): the small ones first
#pragma unroll
          for (int r = 0; r < RH; ++r) {
#pragma unroll
            for (int i = 0; i < 6; ++i) {
              const u32x4 q = *reinterpret_cast<const u32x4*>(lds + r * 16 * stride + PARTS[i][1] * plane + u * 64);
#pragma unroll
              for (int s = 0; s < AT_ONCE; ++s) acc.t[s0 + s][r] = mm16<true>(x[s].p[PARTS[i][0]], q, acc.t[s0 + s][r]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < PER_ROW; ++u) {
      if (FULL || u < steps) {
#pragma unroll
        for (int r = 0; r < RH; ++r) {
          const u32x4 q = *reinterpret_cast<const u32x4*>(lds + r * 16 * stride + u * 64);
#pragma unroll
          for (int s = 0; s < 2; ++s) acc.t[s][r] = mm16<true>(key[s * PER_ROW + u], q, acc.t[s][r]);
        }
      }
      if (u % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
  }
  return acc;
}

// Tiles of 32 score rows whose exponentials a wave has registers for.  One more for fp32 with d > 64 or two key tiles per wave and for bf16 with two tiles of
// d > 64 spills 20 to 100 registers: fp32, d = 64, 96 heads x 1000 keys, 32 rows 22.8 -> 31.8 us, bf16, 512 x 400, 64 rows 29.4 -> 34.5.
template <typename T, int NP, int TPW> constexpr int kept_tiles() { return is_f32(T()) ? (NP > 8 || TPW > 1 ? 1 : 2) : TPW > 1 ? (NP > 4 ? 1 : 2) : NP > 8 ? 2 : 4; }

// the product of 32 keys held as they lie in memory
template <typename T, int NP, bool FULL, bool KEYS_AS_ROWS>
__device__ __forceinline__ f32x16 product_raw(u32x4 (&key)[NP], const char* lds, int plane, int steps) {
  f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if constexpr (is_f32(T())) {
#pragma unroll
    for (int u = 0; u < (NP + 1) / 2; ++u) {
      if (FULL || u < steps) {
        const u32x4 none = {0u, 0u, 0u, 0u};
        // (taken apart here, for every product: the registers do not hold the parts)
        asm volatile("" : "+v"(key[2 * u]));
        if (2 * u + 1 < NP) asm volatile("" : "+v"(key[2 * u + 1 < NP ? 2 * u + 1 : 0]));
        const Split s = split8(key[2 * u], 2 * u + 1 < NP ? key[2 * u + 1 < NP ? 2 * u + 1 : 0] : none);
        const u32x4 q0 = *reinterpret_cast<const u32x4*>(lds + u * 32);
        acc = mm<KEYS_AS_ROWS>(s.p[2], q0, acc);
        const u32x4 q2 = *reinterpret_cast<const u32x4*>(lds + 2 * plane + u * 32);
        acc = mm<KEYS_AS_ROWS>(s.p[0], q2, acc);
        const u32x4 q1 = *reinterpret_cast<const u32x4*>(lds + plane + u * 32);
        acc = mm<KEYS_AS_ROWS>(s.p[1], q1, acc);
        acc = mm<KEYS_AS_ROWS>(s.p[0], q1, acc);
        acc = mm<KEYS_AS_ROWS>(s.p[1], q0, acc);
        acc = mm<KEYS_AS_ROWS>(s.p[0], q0, acc);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      if (FULL || u < steps) acc = mm<KEYS_AS_ROWS>(key[u], *reinterpret_cast<const u32x4*>(lds + u * 32), acc);
      if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  return acc;
}

// Scores of a head of few score rows, whose exponentials stay in registers: into raw (prefix) and `scores` (the keys behind it).
template <typename T, int NP, bool FULL, int WAVES, int TPW>
__device__ __forceinline__ void scores_kept(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, const HeadPlan& pl, const T* __restrict__ q,
                                            const T* __restrict__ k, int inst, int head, char* smem, int* last, int* bins, float* raw, float* __restrict__ scores) {
  constexpr int THREADS = WAVES * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), grp = lane >> 4, n16 = lane & 15;
  const size_t hg = (size_t)inst * g.Hkv + head;
  const int row_bytes = FULL ? NP * 32 : g.d * (int)sizeof(T);
  const int plane = plane16_bytes(row_bytes / (int)sizeof(T)), stride = row16_stride<T>(row_bytes / (int)sizeof(T));
  const char* head_rows = reinterpret_cast<const char*>(q + hg * g.R * g.d);
  const RowScale row_scale = pl.row_scale;
  auto key_rows = [&](const char* (&rows)[2], int key0) {
    int r0 = key0;
    const char* p = reinterpret_cast<const char*>(k + (lay.table ? 0 : (int64_t)inst * lay.inst) + (int64_t)head * lay.head);
    if (lay.table) p += paged_tile_offset(lay, inst, key0, &r0) * (int64_t)sizeof(T);
#pragma unroll
    for (int s = 0; s < 2; ++s)                          // (keys beyond the last one are masked: any row will do)
      rows[s] = p + (int64_t)(r0 + min(16 * s + n16, g.L - 1 - key0)) * lay.row_bytes;
  };
  const int tiles16 = (g.R + 15) / 16;
  float2* stat = reinterpret_cast<float2*>(smem + pl.off_stat);            // [16 rows][wave][row]
  u32x4 key[TPW][NP];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int key0 = (i * WAVES + wave) * 32;
    if (key0 < g.L) {
      const char* p[2];
      key_rows(p, key0);
#pragma unroll
      for (int t = 0; t < NP; ++t) {
        const int piece = 4 * (t % (NP / 2)) + grp;
        if (!FULL) key[i][t] = u32x4{0u, 0u, 0u, 0u};
        if (FULL || piece * 16 < row_bytes) key[i][t] = *reinterpret_cast<const u32x4*>(p[t / (NP / 2)] + piece * 16);
      }
    }
  }
  for (int r = tid; r < tiles16 * 16; r += THREADS) last[r] = last_visible_key(g, qp, min(r, g.R - 1) % g.W);
  for (int i = tid; i < THREADS + 2 * MARGIN; i += THREADS) raw[i] = 0.f;
  bins[tid] = 0;
  stage_rows16<T, FULL, THREADS>(smem, head_rows, row_bytes, plane, stride, g.R, 0, tiles16 * 16, row_scale.shift);
  __syncthreads();
  const char* rows = smem + n16 * stride + grp * 16;
  const auto plus = [](float x, float y) { return x + y; };
  const auto greater = [](float x, float y) { return fmaxf(x, y); };
  // rows row0 .. + 16 RH - 1 that do not see a key of the tile key0
  auto mask = [&](Tile16& a, int row0, int row_halves, int key0) {
    if (key0 + 31 > g.qmin) {
#pragma unroll
      for (int r = 0; r < row_halves; ++r) {
        const int seen = last[row0 + 16 * r + n16] - key0 - 4 * grp;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (16 * (e >> 2) + (e & 3) > seen) a.t[e >> 2][r][e & 3] = -INFINITY;
      }
    }
  };
  // (m, z) of score rows row0 .. + 16 RH - 1 over the wave's keys, a tile after the other; tile i leaves its exponentials in e[i] and their
  // references, those of this lane's rows, in m[i]
  auto statistics = [&](auto row_halves, int row0, const char* at, Tile16 (&e)[TPW], float (&m)[TPW][2]) {
    constexpr int RH = decltype(row_halves)::value;
    float z_all = 0.f, m_all[2] = {NEG_BIG, NEG_BIG};
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int key0 = (i * WAVES + wave) * 32;
      if (key0 >= g.L) continue;
      Tile16 a = product16_raw<T, NP, FULL, (NP * TPW > 8), RH>(key[i], at, stride, plane, plane / 64);
      float scale = row_scale.scale2, z;
#pragma unroll 1
      for (bool again = false;; again = true) {
        mask(a, row0, RH, key0);
        float top[2];
#pragma unroll
        for (int r = 0; r < RH; ++r) {
          top[r] = a.t[0][r][0];
#pragma unroll
          for (int c = 1; c < 8; ++c) top[r] = fmaxf(top[r], a.t[c >> 2][r][c & 3]);
        }
        const float own = over_groups(top[0], top[RH - 1], greater);
        const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(own), __float_as_uint(own), false, false);
        float zr[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          // a whole number: what brings statistics together is an exact power of two (the logit scale is positive)
          m[i][r] = fmaxf(m_all[r], __builtin_ceilf(__uint_as_float(both[r]) * scale));
          zr[r] = 0.f;
        }
        Tile16& x = e[i];
#pragma unroll
        for (int r = 0; r < RH; ++r)
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            x.t[c >> 2][r][c & 3] = __builtin_amdgcn_exp2f(fmaf(a.t[c >> 2][r][c & 3], scale, -m[i][r]));
            zr[r] += x.t[c >> 2][r][c & 3];
          }
        z = over_groups(zr[0], zr[RH - 1], plus);
        if (!is_f32(T()) || again || __builtin_expect(!__any(z != z), 1)) break;
        const char *kr[2], *qr[2];
        key_rows(kr, key0);
#pragma unroll
        for (int r = 0; r < 2; ++r) qr[r] = head_rows + (size_t)min(row0 + 16 * r + n16, g.R - 1) * row_bytes;
        a = product16_f32<true>(kr, qr, grp, row_bytes);
        scale = g.scale2;
      }
      z_all = i == 0 ? z : fmaf(z_all, __builtin_amdgcn_exp2f(grp < 2 ? m_all[0] - m[i][0] : m_all[1] - m[i][1]), z);
      m_all[0] = m[i][0];
      m_all[1] = m[i][1];
    }
    if ((grp & 1) == 0 && (grp >> 1) < RH) stat[(row0 / 16 + (grp >> 1)) * WAVES * 16 + wave * 16 + n16] = make_float2(grp < 2 ? m_all[0] : m_all[1], z_all);
  };
  // M and Z of row n16 of 16 rows: the groups of lanes take a quarter of the waves each
  auto fold = [&](int t16) {
    const float2* s = stat + (t16 * WAVES + grp * (WAVES / 4)) * 16 + n16;
    float2 v[WAVES / 4];
    float M = NEG_BIG, Z = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES / 4; ++w) {
      v[w] = s[w * 16];
      M = fmaxf(M, v[w].x);
    }
    M = over_groups(M, M, greater);
#pragma unroll
    for (int w = 0; w < WAVES / 4; ++w) Z = fmaf(v[w].y, __builtin_amdgcn_exp2f(v[w].x - M), Z);
    return make_float2(M, over_groups(Z, Z, plus));
  };
  // Of more than 32 rows each wave folds 16 for all, into the first wave's place.  (Every wave all of them: laq_evict, us, that : this, bf16, 128 rows, 64 heads
  // x 400 keys, d = 64 15.9 : 13.9, 128 18.8 : 16.9, with products made twice 15.2, 18.7; 64 rows, 8 x 512, d = 128 14.9 : 14.0, 100 x 512, fp32, d = 64
  // 18.6 : 18.0.)
  constexpr int KT = kept_tiles<T, NP, TPW>();
  const bool once = KT > 1 && tiles16 > 2;
  auto folded = [&](int t16) { return once ? stat[t16 * WAVES * 16 + n16] : fold(t16); };
  using One = std::integral_constant<int, 1>;
  using Two = std::integral_constant<int, 2>;
  float sum[TPW][8];                       // of keys 16 (c / 4) + 4 grp + c % 4 of the tiles, over this lane's rows
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int c = 0; c < 8; ++c) sum[i][c] = 0.f;
  Tile16 kept[KT][TPW];
  float m[KT][TPW][2];
#pragma unroll
  for (int rt = 0; rt < KT; ++rt) {
    if (2 * rt + 1 < tiles16) statistics(Two{}, rt * 32, rows + rt * 32 * stride, kept[rt], m[rt]);
    else if (2 * rt < tiles16) statistics(One{}, rt * 32, rows + rt * 32 * stride, kept[rt], m[rt]);
  }
  __syncthreads();
  if (once) {
    static_assert(2 * KT <= WAVES, "");
    if (wave < tiles16) {
      const float2 f = fold(wave);
      if (grp == 0) stat[wave * WAVES * 16 + n16] = f;
    }
    __syncthreads();
  }
#pragma unroll
  for (int t16 = 0; t16 < 2 * KT; ++t16) {
    if (t16 >= tiles16) continue;
    const float2 f = folded(t16);
    const float per = t16 * 16 + n16 < g.R ? 1.f / f.y : 0.f;
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      if ((i * WAVES + wave) * 32 >= g.L) continue;
      const float weight = __builtin_amdgcn_exp2f(m[t16 / 2][i][t16 % 2] - f.x) * per;
#pragma unroll
      for (int c = 0; c < 8; ++c) sum[i][c] = fmaf(kept[t16 / 2][i].t[c >> 2][t16 % 2][c & 3], weight, sum[i][c]);
    }
  }
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int key0 = (i * WAVES + wave) * 32, c_own = (lane & 15) >> 1, j = key0 + 16 * (c_own >> 2) + 4 * grp + (c_own & 3);   // (two lanes a key)
    if (key0 >= g.L) continue;
    float both = group_reduce<16, 8>(sum[i], lane);
    if (__builtin_expect(__any((both < TINY || (is_f32(T()) && both != both)) && j < g.L), 0)) {
      // (score rows and keys from memory)
      float x_sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      const char* kr[2];
      key_rows(kr, key0);
#pragma unroll 1
      for (int t16 = 0; t16 < tiles16; ++t16) {
        const int row = t16 * 16 + n16;
        const char* const qr[2] = {head_rows + (size_t)min(row, g.R - 1) * row_bytes, head_rows + (size_t)min(row, g.R - 1) * row_bytes};
        Tile16 a;
        if constexpr (is_f32(T())) {
          a = product16_f32<true>(kr, qr, grp, row_bytes);
        } else {
          a.clear();
#pragma unroll 1
          for (int o = grp * 16; o < row_bytes + grp * 16; o += 64) {
            u32x4 x0 = {0u, 0u, 0u, 0u}, x1 = x0, y = x0;
            if (o < row_bytes) {
              x0 = *reinterpret_cast<const u32x4*>(kr[0] + o);
              x1 = *reinterpret_cast<const u32x4*>(kr[1] + o);
              y = *reinterpret_cast<const u32x4*>(qr[0] + o);
            }
            a.t[0][0] = mm16<true>(x0, y, a.t[0][0]);
            a.t[1][0] = mm16<true>(x1, y, a.t[1][0]);
          }
        }
        mask(a, t16 * 16, 1, key0);
        const float2 f = folded(t16);
        const float cr = row < g.R ? f.x + __builtin_amdgcn_logf(f.y) : INFINITY;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const float x = fmaf(a.t[c >> 2][0][c & 3], g.scale2, -cr);
          x_sum[c] += x < -126.f ? __builtin_amdgcn_exp2f(x + 64.f) * 0x1p-64f : __builtin_amdgcn_exp2f(x);
        }
      }
      both = group_reduce<16, 8>(x_sum, lane);
    }
    if ((lane & 1) == 0 && j < g.L) {
      if (j < g.P) raw[MARGIN + j] = both;
      else scores[j] = both;
    }
  }
  __syncthreads();
}

// The same where score rows are more: products and exponentials twice.
template <typename T, int NP, bool FULL, int WAVES, int TPW>
__device__ __forceinline__ void scores_again(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, const HeadPlan& pl, const T* __restrict__ q,
                                             const T* __restrict__ k, int inst, int head, char* smem, int* last, int* bins, float* raw, float* __restrict__ scores) {
  constexpr int THREADS = WAVES * 64;
  __shared__ __align__(16) float rowc[MAX_ROWS];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hf = lane >> 5, n32 = lane & 31;
  const size_t hg = (size_t)inst * g.Hkv + head;
  const int row_bytes = FULL ? NP * 32 : g.d * (int)sizeof(T);
  const int plane = plane_bytes(row_bytes / (int)sizeof(T)), stride = row_stride<T>(row_bytes / (int)sizeof(T));
  const char* head_rows = reinterpret_cast<const char*>(q + hg * g.R * g.d);
  const RowScale row_scale = pl.row_scale;
  auto key_row = [&](int key0) {
    int r0 = key0;
    const char* p = reinterpret_cast<const char*>(k + (lay.table ? 0 : (int64_t)inst * lay.inst) + (int64_t)head * lay.head);
    if (lay.table) p += paged_block_offset(lay, inst, key0, &r0) * (int64_t)sizeof(T);
    return p + (int64_t)(r0 + min(n32, g.L - 1 - key0)) * lay.row_bytes;     // (keys beyond the last one are masked: any row will do)
  };
  const int tiles = g.Rpad / 32;
  float2* stat = reinterpret_cast<float2*>(smem + pl.off_stat);            // [row tile][wave][row]
  u32x4 key[TPW][NP];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int key0 = (i * WAVES + wave) * 32;
    if (key0 < g.L) {
      const char* p = key_row(key0) + hf * 16;
#pragma unroll
      for (int t = 0; t < NP; ++t) {
        if (!FULL) key[i][t] = u32x4{0u, 0u, 0u, 0u};
        if (FULL || (2 * t + hf) * 16 < row_bytes) key[i][t] = *reinterpret_cast<const u32x4*>(p + t * 32);
      }
    }
  }
  for (int r = tid; r < tiles * 32; r += THREADS) last[r] = last_visible_key(g, qp, min(r, g.R - 1) % g.W);
  for (int i = tid; i < THREADS + 2 * MARGIN; i += THREADS) raw[i] = 0.f;
  bins[tid] = 0;
  stage_rows<T, FULL, THREADS>(smem, head_rows, row_bytes, plane, stride, g.R, 0, min(pl.group_tiles, tiles) * 32, row_scale.shift);
  __syncthreads();
  const char* rows = smem + n32 * stride + hf * 16;
  // ---- statistics ----
#pragma unroll 1
  for (int rt0 = 0; rt0 < tiles; rt0 += pl.group_tiles) {
    const int ntile = min(pl.group_tiles, tiles - rt0);
    if (rt0 > 0) {
      __syncthreads();
      stage_rows<T, FULL, THREADS>(smem, head_rows, row_bytes, plane, stride, g.R, rt0 * 32, ntile * 32, row_scale.shift);
      __syncthreads();
    }
#pragma unroll 1
    for (int rt = 0; rt < ntile; ++rt) {
      float M = NEG_BIG, Z = 0.f;
#pragma unroll
      for (int i = 0; i < TPW; ++i) {
        const int key0 = (i * WAVES + wave) * 32;
        if (key0 >= g.L) continue;
        float m, z, scale = row_scale.scale2;
        f32x16 s = product_raw<T, NP, FULL, true>(key[i], rows + rt * 32 * stride, plane, plane / 32);
#pragma unroll 1
        for (bool again = false;; again = true) {
          if (key0 + 31 > g.qmin) {
            const int seen = last[(rt0 + rt) * 32 + n32] - key0;
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (acc_row(e, hf) > seen) s[e] = -INFINITY;
          }
          m = s[0];
#pragma unroll
          for (int e = 1; e < 16; ++e) m = fmaxf(m, s[e]);
          const auto mh = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
          m = fmaxf(M, fmaxf(__uint_as_float(mh[0]), __uint_as_float(mh[1])) * scale);     // (the logit scale is positive)
          z = 0.f;
#pragma unroll
          for (int e = 0; e < 16; ++e) z += __builtin_amdgcn_exp2f(fmaf(s[e], scale, -m));
          const auto zh = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
          z = __uint_as_float(zh[0]) + __uint_as_float(zh[1]);
          if (!is_f32(T()) || again || __builtin_expect(!__any(z != z), 1)) break;
          s = product_f32<true>(key_row(key0), head_rows + (size_t)min((rt0 + rt) * 32 + n32, g.R - 1) * row_bytes, hf, row_bytes);
          scale = g.scale2;
        }
        Z = fmaf(Z, __builtin_amdgcn_exp2f(M - m), z);
        M = m;
      }
      if (hf == 0) stat[((rt0 + rt) * WAVES + wave) * 32 + n32] = make_float2(M, Z);
    }
  }
  __syncthreads();
  for (int r = tid; r < tiles * 32; r += THREADS) {
    const float2* s = stat + (r >> 5) * WAVES * 32 + (r & 31);
    float M = NEG_BIG, Z = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) M = fmaxf(M, s[w * 32].x);
#pragma unroll
    for (int w = 0; w < WAVES; ++w) Z = fmaf(s[w * 32].y, __builtin_amdgcn_exp2f(s[w * 32].x - M), Z);
    rowc[r] = r < g.R ? M + __builtin_amdgcn_logf(Z) : INFINITY;
  }
  __syncthreads();
  // ---- raw scores ----
  float sum[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) sum[i] = 0.f;
  auto masked = [&](f32x16 s, int row0, int key0) {
    if (key0 + 31 > g.qmin) {
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const i32x4 lv = *reinterpret_cast<const i32x4*>(last + row0 + 8 * gq + 4 * hf);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (key0 + n32 > lv[e]) s[4 * gq + e] = -INFINITY;
      }
    }
    return s;
  };
#pragma unroll 1
  for (int rt0 = 0; rt0 < tiles; rt0 += pl.group_tiles) {
    const int ntile = min(pl.group_tiles, tiles - rt0);
    if (pl.groups > 1) {
      __syncthreads();
      stage_rows<T, FULL, THREADS>(smem, head_rows, row_bytes, plane, stride, g.R, rt0 * 32, ntile * 32, row_scale.shift);
      __syncthreads();
    }
#pragma unroll 1
    for (int rt = 0; rt < ntile; ++rt) {
#pragma unroll
      for (int i = 0; i < TPW; ++i) {
        const int key0 = (i * WAVES + wave) * 32;
        if (key0 >= g.L) continue;
        const f32x16 s = masked(product_raw<T, NP, FULL, false>(key[i], rows + rt * 32 * stride, plane, plane / 32), (rt0 + rt) * 32, key0);
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const f32x4 c = *reinterpret_cast<const f32x4*>(rowc + (rt0 + rt) * 32 + 8 * gq + 4 * hf);
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[i] += __builtin_amdgcn_exp2f(fmaf(s[4 * gq + e], row_scale.scale2, -c[e]));
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int key0 = (i * WAVES + wave) * 32, j = key0 + n32;
    if (key0 >= g.L) continue;
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[i]), __float_as_uint(sum[i]), false, false);
    float both = __uint_as_float(halves[0]) + __uint_as_float(halves[1]);
    if (__builtin_expect(__any((both < TINY || (is_f32(T()) && both != both)) && j < g.L), 0)) {
      // (score rows and keys from memory: the staged rows may be another group's)
      float x_sum = 0.f;
#pragma unroll 1
      for (int rt = 0; rt < tiles; ++rt) {
        const char *kr = key_row(key0), *qr = head_rows + (size_t)min(rt * 32 + n32, g.R - 1) * row_bytes;
        f32x16 s;
        if constexpr (is_f32(T())) {
          s = product_f32<false>(kr, qr, hf, row_bytes);
        } else {
          s = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
          for (int o = hf * 16; o < row_bytes + hf * 16; o += 32) {
            u32x4 x = {0u, 0u, 0u, 0u}, y = x;
            if (o < row_bytes) {
              x = *reinterpret_cast<const u32x4*>(kr + o);
              y = *reinterpret_cast<const u32x4*>(qr + o);
            }
            s = mm<false>(x, y, s);
          }
        }
        s = masked(s, rt * 32, key0);
#pragma unroll 1
        for (int e = 0; e < 16; ++e) {
          const float x = fmaf(s[0], g.scale2, -rowc[rt * 32 + acc_row(e, hf)]);
          x_sum += x < -126.f ? __builtin_amdgcn_exp2f(x + 64.f) * 0x1p-64f : __builtin_amdgcn_exp2f(x);
          s = __builtin_shufflevector(s, s, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 0);
        }
      }
      both = x_sum + __shfl_xor(x_sum, 32);
    }
    if (hf == 0 && j < g.L) {
      if (j < g.P) raw[MARGIN + j] = both;
      else scores[j] = both;
    }
  }
  __syncthreads();
}

// `steps`: see HeadSteps.  fin.half: pooling of the scores, 0 for none.
template <typename T, int NP, bool FULL, int WAVES, int TPW, bool KEEP, typename TAB>
__global__ __launch_bounds__(WAVES * 64, 4) void head_kernel(ScoreGeom g, WindowPos qp, KvLayout lay, HeadPlan pl, int steps,
                                                              const T* __restrict__ q, const T* __restrict__ k, TAB tab,
                                                              int inst0, int32_t* __restrict__ idx, FinishArgs fin, int* __restrict__ status) {
  constexpr int THREADS = WAVES * 64;
  extern __shared__ __align__(16) char smem[];
  __shared__ __align__(16) int last[MAX_ROWS];           // last key the rows see
  __shared__ float raw[MARGIN + THREADS + MARGIN];       // raw scores of the prefix, zeros around them
  __shared__ int list[THREADS];
  __shared__ RankScratch<WAVES> rank;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int head = blockIdx.x, li = blockIdx.y, inst = inst0 + li;
  const size_t hg = (size_t)inst * g.Hkv + head;
  // (No wait to give up here.  In front of the keys' loads its address is a trip to memory that these are behind: bf16, and fp32 with d = 64 and a tile per wave, 2 to 80
  // heads x 300 to 800 keys, 16 and 32 rows, with the store behind the scores .97-1.00 of the time.  What the compiler makes of the other fp32 variants is 1.00-1.04
  // then.)
  constexpr bool STATUS_FIRST = is_f32(T()) && (NP > 8 || TPW > 1);
  const bool clears = head == 0 && inst == 0 && tid == 0;
  if (STATUS_FIRST && clears) *status = 0;
  float* scores = fin.pooled + hg * g.L;
  if constexpr (KEEP) scores_kept<T, NP, FULL, WAVES, TPW>(g, qp, lay, pl, q, k, inst, head, smem, last, rank.bins, raw, scores);
  else scores_again<T, NP, FULL, WAVES, TPW>(g, qp, lay, pl, q, k, inst, head, smem, last, rank.bins, raw, scores);
  if (!STATUS_FIRST && clears) *status = 0;
  // ---- pooling: position tid ----
  const int P = g.P, half = fin.half;
  float v = raw[MARGIN + tid];
  if (half > 0) {
    const float* w = raw + MARGIN + tid;
    if (fin.avg) {
      float acc = 0.f;
      for (int o = -half; o <= half; ++o) acc += w[o];
      v = acc / (float)(2 * half + 1);
    } else {
      for (int o = -half; o <= half; ++o) v = fmaxf(v, w[o]);
    }
  }
  if (tid < P) scores[tid] = v;
  if (steps == HEAD_SCORES) return;
  // ---- selection ----
  const int bk = tab.rows(li), ksel = bk - g.keep;
  const int64_t row0 = tab.first(li) + (int64_t)head * bk;
  int32_t* out = idx + row0;
  for (int w = tid; w < g.keep; w += THREADS) {
    list[ksel + w] = P + w;
    out[ksel + w] = P + w;
  }
  if (ksel >= P) {
    if (tid < P) {
      list[tid] = tid;
      out[tid] = tid;
    }
  } else if (ksel > 0) {
    const int at = rank_position<WAVES>(rank, tid < P ? max(order_key(v), 1u) : 0u, ksel, lane, wave);
    if (at >= 0) {
      list[at] = tid;
      out[at] = tid;
    }
  }
  if (steps == HEAD_LIST) return;
  __syncthreads();
  gather_rows<THREADS>(fin, inst, head, bk, row0, [&](int r) { return list[r]; });
}

template <typename T, int NP, bool FULL, int WAVES, int TPW, typename TAB>
hipError_t launch_one(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int steps, const T* q, const T* k, int n, int inst0,
                      const TAB& tab, int32_t* idx, const FinishArgs& fin, int* status, hipStream_t st) {
  HeadPlan pl;
  pl.row_scale = row_scale_of<T>(g.scale2);
  auto launch = [&](auto kernel, int lds) {
    hipLaunchKernelGGL(kernel, dim3(g.Hkv, n), dim3(WAVES * 64), lds, st, g, qp, lay, pl, steps, q, k, tab, inst0, idx, fin, status);
    return hipGetLastError();
  };
  const int tiles = g.Rpad / 32, tiles16 = (g.R + 15) / 16;
  if (tiles <= kept_tiles<T, NP, TPW>()) {
    pl.group_tiles = tiles;
    pl.groups = 1;
    pl.off_stat = tiles16 * 16 * row16_stride<T>(g.d);
    return launch(head_kernel<T, NP, FULL, WAVES, TPW, true, TAB>, pl.off_stat + tiles16 * WAVES * 16 * (int)sizeof(float2));
  }
  const int stride = row_stride<T>(g.d);
  const int stat = tiles * WAVES * 32 * (int)sizeof(float2), most = ((WAVES == 16 ? 150 : 74) << 10) - stat - 12 * 1024;
  pl.group_tiles = std::max(1, std::min(std::min(tiles, MAX_TILES), most / (32 * stride)));
  pl.groups = (tiles + pl.group_tiles - 1) / pl.group_tiles;
  pl.off_stat = pl.group_tiles * 32 * stride;
  return launch(head_kernel<T, NP, FULL, WAVES, TPW, false, TAB>, pl.off_stat + stat);
}

template <typename T, int NP, bool FULL, bool SHORT, typename TAB>
hipError_t launch_for_keys(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int steps, const T* q, const T* k, int n, int inst0,
                           const TAB& tab, int32_t* idx, const FinishArgs& fin, int* status, hipStream_t st) {
  if (g.L <= 512) {
    // one tile of keys per wave: the shortest way through one head; two per wave, half the waves: two heads per compute unit
    if (SHORT || (long long)g.n_inst * g.Hkv <= 256)
      return launch_one<T, NP, FULL, 16, 1, TAB>(g, qp, lay, steps, q, k, n, inst0, tab, idx, fin, status, st);
    if constexpr (!SHORT) return launch_one<T, NP, FULL, 8, 2, TAB>(g, qp, lay, steps, q, k, n, inst0, tab, idx, fin, status, st);
  }
  if constexpr (!SHORT) return launch_one<T, NP, FULL, 16, 2, TAB>(g, qp, lay, steps, q, k, n, inst0, tab, idx, fin, status, st);
  return hipErrorInvalidValue;
}

template <typename TAB>
hipError_t launch_for(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, int steps, const void* q, const void* k, int n, int inst0,
                      const TAB& tab, int32_t* idx, const FinishArgs& fin, int* status, hipStream_t st) {
  if (dtype == LAQ_F32) {
    const float *qq = static_cast<const float*>(q), *kk = static_cast<const float*>(k);
    if (g.d == 64) return launch_for_keys<float, 8, true, false>(g, qp, lay, steps, qq, kk, n, inst0, tab, idx, fin, status, st);
    if (g.d == 128) return launch_for_keys<float, 16, true, true>(g, qp, lay, steps, qq, kk, n, inst0, tab, idx, fin, status, st);
    return launch_for_keys<float, 16, false, true>(g, qp, lay, steps, qq, kk, n, inst0, tab, idx, fin, status, st);
  }
  const uint16_t *qq = static_cast<const uint16_t*>(q), *kk = static_cast<const uint16_t*>(k);
  if (g.d == 64) return launch_for_keys<uint16_t, 4, true, false>(g, qp, lay, steps, qq, kk, n, inst0, tab, idx, fin, status, st);
  if (g.d == 128) return launch_for_keys<uint16_t, 8, true, false>(g, qp, lay, steps, qq, kk, n, inst0, tab, idx, fin, status, st);
  if (g.d < 128) return launch_for_keys<uint16_t, 8, false, false>(g, qp, lay, steps, qq, kk, n, inst0, tab, idx, fin, status, st);
  if (g.d == 256) return launch_for_keys<uint16_t, 16, true, true>(g, qp, lay, steps, qq, kk, n, inst0, tab, idx, fin, status, st);
  return launch_for_keys<uint16_t, 16, false, true>(g, qp, lay, steps, qq, kk, n, inst0, tab, idx, fin, status, st);
}

}  // namespace

bool head_supported(const ScoreGeom& g, int dtype) {
  const bool two_tiles = dtype == LAQ_F32 ? g.d == 64 : g.d <= 128;      // that a wave has registers for
  return g.R <= MAX_ROWS && g.d <= (dtype == LAQ_F32 ? 128 : 256) && g.L <= (two_tiles ? 1024 : 512);
}

// (the variants as launch_for() and launch_for_keys() choose them)
bool head_keeps(const ScoreGeom& g, int dtype) {
  const bool two = g.L > 512 || (long long)g.n_inst * g.Hkv > 256;       // tiles per wave, where the variant has registers for them
  int kept;
  if (dtype == LAQ_F32) kept = g.d != 64 ? kept_tiles<float, 16, 1>() : two ? kept_tiles<float, 8, 2>() : kept_tiles<float, 8, 1>();
  else if (g.d == 64) kept = two ? kept_tiles<uint16_t, 4, 2>() : kept_tiles<uint16_t, 4, 1>();
  else if (g.d <= 128) kept = two ? kept_tiles<uint16_t, 8, 2>() : kept_tiles<uint16_t, 8, 1>();
  else kept = kept_tiles<uint16_t, 16, 1>();
  return g.Rpad / 32 <= kept;
}

hipError_t launch_head(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, int steps, const void* q, const void* k, int n, int inst0,
                       const InstTable& tab, int32_t* idx, const FinishArgs& fin, int* status, hipStream_t st) {
  return launch_for(g, qp, lay, dtype, steps, q, k, n, inst0, tab, idx, fin, status, st);
}
hipError_t launch_head(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, int steps, const void* q, const void* k, int n, int inst0,
                       const UniformInst& tab, int32_t* idx, const FinishArgs& fin, int* status, hipStream_t st) {
  return launch_for(g, qp, lay, dtype, steps, q, k, n, inst0, tab, idx, fin, status, st);
}

// every variant that launch_for() names
template <typename T, int NP, bool FULL, int WAVES, int TPW> hipError_t init_one() {
  hipError_t e;
  for (const void* f : {(const void*)&head_kernel<T, NP, FULL, WAVES, TPW, true, InstTable>, (const void*)&head_kernel<T, NP, FULL, WAVES, TPW, true, UniformInst>,
                        (const void*)&head_kernel<T, NP, FULL, WAVES, TPW, false, InstTable>, (const void*)&head_kernel<T, NP, FULL, WAVES, TPW, false, UniformInst>})
    if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 144 << 10)) != hipSuccess) return e;
  return hipSuccess;
}
template <typename T, int NP, bool FULL, bool SHORT> hipError_t init_keys() {
  hipError_t e = init_one<T, NP, FULL, 16, 1>();
  if constexpr (!SHORT) {
    if (e == hipSuccess) e = init_one<T, NP, FULL, 8, 2>();
    if (e == hipSuccess) e = init_one<T, NP, FULL, 16, 2>();
  }
  return e;
}
hipError_t head_init() {
  for (hipError_t e : {init_keys<float, 8, true, false>(), init_keys<float, 16, true, true>(), init_keys<float, 16, false, true>(), init_keys<uint16_t, 4, true, false>(),
                       init_keys<uint16_t, 8, true, false>(), init_keys<uint16_t, 8, false, false>(), init_keys<uint16_t, 16, true, true>(),
                       init_keys<uint16_t, 16, false, true>()})
    if (e != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace laq
