// Scoring in two passes over K without a barrier between keys: every head size up to 256, any number of score
// rows, fp32 or bf16, on the matrix cores (v_mfma_f32_16x16x32_bf16).
//
// Kernel 1 leaves the softmax statistics (m, z) of every score row over a segment of a head's keys, kernel 2 folds
// the segments' (or finds them folded by row_constants_kernel, where they are many) and sums the probabilities
// exp2(s - M) / Z over the rows: raw scores.
//
// A workgroup of four waves stages the head's score rows (up to 128 of them) in LDS once and then walks its segment
// of keys, 128 at a time; a wave takes 32 of these in registers, straight from memory in operand layout (lane l: rows
// l % 16 and 16 + l % 16, the 16-byte pieces 4t + l / 16), while the next 32 are on their way into others.  Nothing that a wave does
// per key waits for another wave, so loads and arithmetic of the 8 to 20 waves of a compute unit mix freely.
//   (1) D = K * Q^T: lane = two score rows, registers = 8 keys: sum (and, where it is needed, maximum) in registers, the wave's running (m, z) in LDS.
//   (2) D = Q * K^T: lane = two keys, registers = 8 rows: the sum over the rows in registers.
// Score rows beyond R repeat the last one and get the weight 0, so that they add nothing.
//
// 32 keys by 32 rows are four products of 16 x 16 and not one of 32 x 32: as many operations and operand reads, but a fifth less traffic between
// matrix core and registers, four chains instead of one, 64 bytes of a row per load instruction instead of 32, and half the reads of row constants.
// laq_evict, us, with 32 x 32 : so: bf16, 128 rows, 256 heads x 32768 keys 937 : 900, 112 rows, 112 x 20123 295 : 288, d = 96, 128 rows, 96 x 16000
// 152.9 : 147.6; 64 rows and fewer 0.99-1.01; fp32, 64 rows, 64 x 8191 152 : 147, d = 64 and 96 1.04, d = 104 1.06, 128 rows, 64 x 4000 144.5 : 136.
//
// References M are whole numbers and the rows' weights 1 / Z are multiplied in, so that everything which brings statistics together is an exact power
// of two and no logarithm of Z is rounded at the size of M.  Scores, error against 64 bits (2-norm), logits of deviation 1 / 4, with exp2(s - (M + log2 Z)) :
// so: bf16, d = 128, 128 rows, 32 heads x 5000 keys 2.0e-7 / 6.1e-7 : 6.0e-8 / 4.9e-7; fp32, 64 rows, 24 x 9000 2.0e-7 / 7.1e-7 : 6.2e-8 / 6.1e-7.
//
// fp32 takes six bf16 products: a float is the sum of three bf16 (split8), and the three products of parts that together reach
// 2^-24 of the whole at most are left out.  The sums are fp32, those of the small products apart from those of the large ones: fewer
// roundings than the fp32 instruction makes, and 2.7 times its rate.  Rows of a single
// element (no sum, one rounding) are where it is not the closer one: 2.34e-8 of a logit rms, 9e-8 at most, against 2.31e-8 and 6e-8.
//
// What bounds it: for up to 64 score rows the two reads of K (64 heads x 8192 to 16384 keys: 5.6 TB/s of 6.2), with 128 the
// matrix cores and the exponentials at the clock they leave, for fp32 the matrix cores.  Scoring, us, before : now: the streaming kernels
// that stood here (256 keys of a head in LDS at a time, two barriers each, five launches): bf16, d = 128, 128 rows, 256 heads x
// 32768 keys 864 : 850; 112 rows, 28 heads x 6143 38 : 31; d = 64, 64 rows, 8 heads x 28227 35 : 28.  The one-chunk kernels: bf16,
// d = 96, 64 rows, 1656 heads x 796 keys 145 : 85; d = 96, 128 rows, 264 x 5815 194 : 135; fp32, d = 128, 64 rows, 64 x 8191 195 : 122;
// d = 96, 128 rows, 368 x 1255 264 : 141.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "laq_internal.h"
#include "laq_products.h"

namespace laq {

namespace {

constexpr int WAVES = 4, THREADS = WAVES * 64;
constexpr int BLOCK_KEYS = WAVES * 32;       // keys that the waves of a workgroup hold at a time
constexpr int MAX_TILES = 4;                 // 32-row tiles of score rows that are staged together
// Segments of a head whose statistics every workgroup of the second kernel folds itself.
constexpr int FOLD_SEGMENTS = 32;
// The work of a wave: segment `seg` of a head's keys, tiles of 32 from `first` to `last_tile`, every BLOCK_KEYS keys one.
// NP: pairs of 16-byte pieces a row may have (32 bytes each); FULL: it has exactly that many.
template <typename T, int NP, bool FULL> struct Wave {
  static constexpr bool F32 = is_f32(T());
  int grp, n16, wave;
  int row_bytes, stride, plane;
  int inst;
  int64_t src_row;         // bytes between key rows
  const char *head_keys, *head_rows;
  int first, last_tile, end;
  bool some;

  __device__ __forceinline__ Wave(const ScoreGeom& g, const KvLayout& lay, const T* q, const T* k, int inst_, int head, int seg, int seg_blocks) {
    const int lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    grp = lane >> 4;
    n16 = lane & 15;
    inst = inst_;
    row_bytes = FULL ? NP * 32 : g.d * (int)sizeof(T);
    plane = plane16_bytes(row_bytes / (int)sizeof(T));
    stride = row16_stride<T>(row_bytes / (int)sizeof(T));
    src_row = lay.row_bytes;
    head_keys = reinterpret_cast<const char*>(k + (lay.table ? 0 : (int64_t)inst * lay.inst) + (int64_t)head * lay.head);
    head_rows = reinterpret_cast<const char*>(q + ((size_t)inst * g.Hkv + head) * g.R * g.d);
    const int block0 = seg * seg_blocks;
    end = min((block0 + seg_blocks) * BLOCK_KEYS, g.L);
    first = block0 * BLOCK_KEYS + wave * 32;
    last_tile = (end - 1) / BLOCK_KEYS * BLOCK_KEYS + wave * 32;
    if (last_tile >= end) last_tile -= BLOCK_KEYS;
    some = first <= last_tile;
  }
  // this lane's rows of the tile of keys key0 .. key0 + 31: n16 and 16 + n16
  __device__ __forceinline__ void key_rows(const char* (&rows)[2], const ScoreGeom& g, const KvLayout& lay, int key0) const {
    int r0 = key0;
    const char* p = head_keys;
    if (lay.table) p += paged_tile_offset(lay, inst, key0, &r0) * (int64_t)sizeof(T);       // (a block holds whole tiles)
#pragma unroll
    for (int s = 0; s < 2; ++s)                          // (keys beyond the last one are masked: any row will do)
      rows[s] = p + (int64_t)(r0 + min(16 * s + n16, g.L - 1 - key0)) * src_row;
  }
  __device__ __forceinline__ void load(u32x4 (&key)[NP], const ScoreGeom& g, const KvLayout& lay, int key0) const {
    const char* rows[2];
    key_rows(rows, g, lay, key0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int t = 0; t < NP / 2; ++t) {
        const char* p = rows[s] + grp * 16 + t * 64;
        u32x4& x = key[s * (NP / 2) + t];
        if (FULL) {
          x = *reinterpret_cast<const u32x4*>(p);
        } else {
          x = u32x4{0u, 0u, 0u, 0u};
          if ((4 * t + grp) * 16 < row_bytes) x = *reinterpret_cast<const u32x4*>(p);
        }
      }
  }

  // this lane's score rows of a tile, in memory
  __device__ __forceinline__ void score_rows(const char* (&rows)[2], const ScoreGeom& g, int rt) const {
#pragma unroll
    for (int r = 0; r < 2; ++r) rows[r] = head_rows + (size_t)min(rt * 32 + 16 * r + n16, g.R - 1) * row_bytes;
  }
};

// A key tile as the products take it; fp32: split into its three parts.
template <typename T, int NP, bool FULL> struct Operand {
  static constexpr bool F32 = is_f32(T());
  static constexpr int PER_ROW = NP / 2, STEPS = F32 ? PER_ROW / 2 : PER_ROW, PARTS = F32 ? 3 : 1;
  static_assert(NP % (F32 ? 4 : 2) == 0, "");
  u32x4 v[2][STEPS * PARTS];
  __device__ __forceinline__ void from(const u32x4 (&key)[NP]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int u = 0; u < STEPS; ++u) {
        if constexpr (F32) {
          const Split x = split8(key[s * PER_ROW + 2 * u], key[s * PER_ROW + 2 * u + 1]);
#pragma unroll
          for (int pl = 0; pl < 3; ++pl) v[s][3 * u + pl] = x.p[pl];
        } else {
          v[s][u] = key[s * PER_ROW + u];
        }
      }
  }
  // against the score rows at `lds` (this lane's row and piece); `steps` of 64 bytes a row has, `plane` bytes between its parts
  // RH: row halves, 1 where the tile's last 16 rows are beyond R
  template <bool KEYS_AS_ROWS, int RH>
  __device__ __forceinline__ Tile16 product(const char* lds, int stride, int plane, int steps) const {
    Tile16 acc;
    acc.clear();
    const char* lds1 = lds + 16 * stride;
    if constexpr (F32) {
      Tile16 low;
      low.clear();
      u32x4 q[2][3];
      auto fetch = [&](int u) {
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
          q[0][pl] = *reinterpret_cast<const u32x4*>(lds + pl * plane + u * 64);
          if (RH > 1) q[1][pl] = *reinterpret_cast<const u32x4*>(lds1 + pl * plane + u * 64);
        }
      };
      auto add = [&](Tile16& to, int u, int key_part, int row_part) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int r = 0; r < RH; ++r) to.t[s][r] = mm16<KEYS_AS_ROWS>(v[s][3 * u + key_part], q[r][row_part], to.t[s][r]);
      };
#pragma unroll
      for (int u = 0; u < STEPS; ++u) {
        if (FULL || u < steps) {
          fetch(u);
          add(low, u, 2, 0);
          add(acc, u, 0, 0);
          add(low, u, 0, 2);
          add(low, u, 1, 1);
          add(low, u, 1, 0);
          add(low, u, 0, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < RH; ++r) acc.t[s][r] += low.t[s][r];
    } else {
#pragma unroll
      for (int u = 0; u < STEPS; ++u) {
        if (FULL || u < steps) {
          u32x4 q[RH];
#pragma unroll
          for (int r = 0; r < RH; ++r) q[r] = *reinterpret_cast<const u32x4*>((r ? lds1 : lds) + u * 64);
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int r = 0; r < RH; ++r) acc.t[s][r] = mm16<KEYS_AS_ROWS>(v[s][u], q[r], acc.t[s][r]);
        }
        if (u % 2 == 1) __builtin_amdgcn_sched_barrier(0);                 // (at most four operands of Q requested ahead: registers)
      }
    }
    return acc;
  }
};

// work(tile, first key) for a wave's key tiles first, first + BLOCK_KEYS .. last; the next one travels while one is worked on
template <typename T, int NP, bool FULL, typename LOAD, typename WORK>
__device__ __forceinline__ void walk_tiles(u32x4 (&A)[NP], int first, int last, LOAD load, WORK work) {
  Operand<T, NP, FULL> op;
  if constexpr (is_f32(T())) {
    for (int t = first; t <= last; t += BLOCK_KEYS) {
      op.from(A);
      load(A, min(t + BLOCK_KEYS, last));
      work(op, t);
    }
  } else {
    u32x4 B[NP];
    for (int t = first; t <= last; t += 2 * BLOCK_KEYS) {
      load(B, min(t + BLOCK_KEYS, last));
      op.from(A);
      work(op, t);
      if (t + BLOCK_KEYS > last) break;
      load(A, min(t + 2 * BLOCK_KEYS, last));
      op.from(B);
      work(op, t + BLOCK_KEYS);
    }
  }
}

struct WavePlan {
  int segs;                // workgroups that share a head's keys
  int seg_blocks;          // blocks of BLOCK_KEYS keys each of them takes
  int group_tiles;         // row tiles staged together
  int groups;
  // The second kernel's workgroups (., y, z) take head head0 + way * y of instance inst0 + way * z: the heads in the first one's order, or in the other.
  // (Numbers and no flag: a flag, and the sizes of the grid behind it, are two waits for memory before anything else.  Kernel 2, us, a flag : so: 64 heads x 2042
  // to 4042 keys 0.2 to 0.25 less of 12 to 16.5.)
  int head0, inst0, way;
  RowScale row_scale;
};

// Waves per SIMD the kernels are built for: as many as their registers (and 32 of the score rows per workgroup in LDS) allow.  (d = 96, bf16: five waves
// spill 13 registers in the second kernel; 64 rows, 192 heads x 8001 152 us, with four 134.5.)
template <typename T, int NP> constexpr int waves_per_simd() { return is_f32(T()) ? (NP <= 8 ? 3 : 2) : (NP <= 4 ? 5 : NP <= 8 ? 4 : 2); }
// (The first kernel of bf16 with d > 128 or a head size without a variant of its own: 168 registers.  With 176, two waves, 448 rows, 3000 heads x 120 keys,
// d = 16 342 us : 298, d = 104 616 : 546.)
template <typename T, int NP> constexpr int stats_waves_per_simd() { return !is_f32(T()) && NP > 8 ? 3 : waves_per_simd<T, NP>(); }

// Row tiles, of those staged from rt0 on, that are taken whole.  fp32 leaves the second half of a last one out where it has no rows: laq_evict, us, 112
// rows, 48 heads x 9000 keys 221 : 209.  bf16 does not: its passes are not bound by products, and the code for it makes others slower (112 rows, 112 x 20123
// 292 : 290, but 128 rows, 256 x 32768 912 : 930, d = 64, 32 rows, 320 x 9000 181 : 190; fp32 of
// head sizes without a variant of their own, whose kernels spill: d = 104, 64 rows, 96 x 5000 141.5 : 145).
template <bool HALVES> __device__ __forceinline__ int whole_tiles(const ScoreGeom& g, int rt0, int ntile) {
  return HALVES ? min(ntile, (g.R - rt0 * 32 + 15) / 32) : ntile;
}

// A wave's sums of exponentials refer to a number near the row's maximum, not to the maximum itself: HEADROOM above that of the first
// tile, and moved only where a tile's sum reaches OUTGROWN of it (then, and where a row does not see all keys of a tile, or a sum is no
// number, the maximum of the tile is made).  The terms that count have exponents between -8 and 7, as with a maximum that most keys stay
// some powers of two below.  A gain in instructions rather than in time: 16 of 87 vector instructions per product of 32 keys and 32 rows less
// (SQ_INSTS_VALU), and the whole eviction of 256 heads x 32768 keys, 128 rows, was not faster beyond noise (934 : 927 us): it is bound by memory and by
// the power that memory and matrix cores take.  Whole numbers, see above.
constexpr float HEADROOM = 3.f, OUTGROWN = 128.f;
// exp2(s * scale - m) of a lane's two rows over the tile's keys: eight of them here, the others in the lanes of the same number modulo 16.
// Lanes 0 .. 31 end with the sum of row n16, the others with that of row 16 + n16 (RH 1: of row n16 too).
template <int RH>
__device__ __forceinline__ float tile_sum(const Tile16& a, float scale, float m0, float m1) {
  float z0 = 0.f, z1 = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float x0 = __builtin_amdgcn_exp2f(fmaf(a.t[e >> 2][0][e & 3], scale, -m0));
    z0 = e == 0 ? x0 : z0 + x0;
    if (RH > 1) {
      const float x1 = __builtin_amdgcn_exp2f(fmaf(a.t[e >> 2][RH - 1][e & 3], scale, -m1));
      z1 = e == 0 ? x1 : z1 + x1;
    }
  }
  return over_groups(z0, RH > 1 ? z1 : z0, [](float x, float y) { return x + y; });
}

// The greater of two numbers, none where one of them is none.  (fmaxf() takes two instructions more for each that it cannot see the origin of.)
__device__ __forceinline__ float greater(float x, float y) { return __builtin_elementwise_maximum(x, y); }
// A lane's own row's number (lanes 0 .. 31: row n16, the others: 16 + n16) -> those of both its rows.  From lane to lane and not by way of LDS, where a lane
// would read what another one wrote with nothing between; and the reference is made once for the lane's row, not twice.  Kernel 1, us, numbers read from
// LDS, two references : so: 128 rows, 67 heads x 2042 keys 17.1 : 16.7, d = 64, 67 x 4042 15.2 : 14.5.
struct RowPair { float m0, m1; };
template <int RH>
__device__ __forceinline__ RowPair both_rows(float own) {
  if constexpr (RH == 1) return {own, own};
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(own), __float_as_uint(own), false, false);
  return {__uint_as_float(h[0]), __uint_as_float(h[1])};
}

// Pass 1: part[head][segment][row] = (m, z) of a score row over the segment's visible keys, in log2 units.
template <typename T, int NP, bool FULL>
__global__ __launch_bounds__(THREADS, (stats_waves_per_simd<T, NP>())) void wave_stats_kernel(ScoreGeom g, WindowPos qp, KvLayout lay, WavePlan pl,
                                                                               const T* __restrict__ q, const T* __restrict__ k,
                                                                               float2* __restrict__ part) {
  extern __shared__ __align__(16) char smem[];
  const int group = blockIdx.x / pl.segs, seg = blockIdx.x - group * pl.segs;
  const int rt0 = group * pl.group_tiles, ntile = min(pl.group_tiles, g.Rpad / 32 - rt0);
  const int whole = whole_tiles<is_f32(T()) && FULL>(g, rt0, ntile);
  const Wave<T, NP, FULL> w(g, lay, q, k, blockIdx.z, blockIdx.y, seg, pl.seg_blocks);
  const RowScale row_scale = pl.row_scale;
  u32x4 key[NP];
  if (w.some) w.load(key, g, lay, w.first);
  stage_rows16<T, FULL, THREADS>(smem, w.head_rows, w.row_bytes, w.plane, w.stride, g.R, rt0 * 32, ntile * 32, row_scale.shift);
  float2* stat = reinterpret_cast<float2*>(smem + pl.group_tiles * 32 * w.stride);       // [row tile][wave][row]
  for (int i = threadIdx.x; i < ntile * WAVES * 32; i += THREADS) stat[i] = make_float2(NEG_BIG, 0.f);
  __syncthreads();
  auto work = [&](const Operand<T, NP, FULL>& op, int key0) {
    const bool plain = key0 + 31 <= g.qmin;              // every row sees every key
    const char* rows = smem + w.n16 * w.stride + w.grp * 16;
    float2* mine = stat + w.wave * 32 + w.n16;           // this lane's first row; the second: 16 further on
    auto tile = [&](auto row_halves, int rt) {
      constexpr int RH = decltype(row_halves)::value;
      const int own = RH > 1 ? w.grp >> 1 << 4 : 0;      // the one whose sum it ends with: the only word of `stat` that the lane reads and writes
      const float2 old = mine[own];
      Tile16 a = op.template product<true, RH>(rows, w.stride, w.plane, w.plane / 64);
      float z = INFINITY;
      if (plain && key0 != w.first) {
        const RowPair r = both_rows<RH>(old.x);
        z = tile_sum<RH>(a, row_scale.scale2, r.m0, r.m1);
      }
      if (__builtin_expect(!__any(!(z <= OUTGROWN)), 1)) {
        mine[own].y = old.y + z;
      } else {
        float m, scale = row_scale.scale2;
#pragma unroll 1
        for (bool again = false;; again = true) {
          if (!plain) {
            int n = threadIdx.x & 63, W = g.W;
            asm volatile("" : "+v"(n));                  // (computed here: the common case has no registers for it)
            if constexpr (!is_f32(T())) asm volatile("" : "+s"(W));   // (nor for what a division by W has ready: bf16, d = 256; fp32, d = 64: 2 spills with this)
#pragma unroll
            for (int r = 0; r < RH; ++r) {
              const int row = (rt0 + rt) * 32 + 16 * r + (n & 15), last = last_visible_key(g, qp, min(row, g.R - 1) % W) - key0 - 4 * (n >> 4);
#pragma unroll
              for (int e = 0; e < 8; ++e)
                if (16 * (e >> 2) + (e & 3) > last) a.t[e >> 2][r][e & 3] = -INFINITY;
            }
          }
          float m0 = greater(a.t[0][0][0], a.t[0][0][1]), m1 = greater(a.t[0][RH - 1][0], a.t[0][RH - 1][1]);
#pragma unroll
          for (int e = 2; e < 8; ++e) {
            m0 = greater(m0, a.t[e >> 2][0][e & 3]);
            m1 = greater(m1, a.t[e >> 2][RH - 1][e & 3]);
          }
          // (the logit scale is positive)
          m = fmaxf(old.x, __builtin_ceilf(fmaf(over_groups(m0, m1, [](float x, float y) { return greater(x, y); }), scale, HEADROOM)));
          const RowPair r = both_rows<RH>(m);
          z = tile_sum<RH>(a, scale, r.m0, r.m1);
          if (!is_f32(T()) || again || __builtin_expect(!__any(z != z), 1)) break;
          const char *kr[2], *qr[2];
          w.key_rows(kr, g, lay, key0);
          w.score_rows(qr, g, rt0 + rt);
          a = product16_f32<true>(kr, qr, w.grp, w.row_bytes);
          scale = g.scale2;
        }
        mine[own] = make_float2(m, fmaf(old.y, __builtin_amdgcn_exp2f(old.x - m), z));
      }
    };
#pragma unroll 1
    for (int rt = 0; rt < whole; ++rt) {
      tile(std::integral_constant<int, 2>{}, rt);
      rows += 32 * w.stride;
      mine += WAVES * 32;
    }
    if (is_f32(T()) && FULL && whole < ntile) tile(std::integral_constant<int, 1>{}, whole);
  };
  if (w.some) walk_tiles<T, NP, FULL>(key, w.first, w.last_tile, [&](u32x4 (&x)[NP], int key0) { w.load(x, g, lay, key0); }, work);
  __syncthreads();
  float2* out = part + (((size_t)blockIdx.z * g.Hkv + blockIdx.y) * pl.segs + seg) * g.Rpad + rt0 * 32;
  if (threadIdx.x < ntile * 32) {
    const int r = threadIdx.x;
    const float2* s = stat + (r >> 5) * WAVES * 32 + (r & 31);
    float M = NEG_BIG, Z = 0.f;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) M = fmaxf(M, s[i * 32].x);
#pragma unroll
    for (int i = 0; i < WAVES; ++i) Z = fmaf(s[i * 32].y, __builtin_amdgcn_exp2f(s[i * 32].x - M), Z);
    out[r] = make_float2(M, Z);
  }
}

// The (m, z) of segments first, first + by, .. of a row, TURN at a time: the greatest reference of these first, then the sums, which whole numbers bring
// together by exact powers of two.  (No segment: NEG_BIG, 0.)  It is what a workgroup of kernel 2 begins with.  laq_evict, us, each segment merged into the
// ones before : so: 64 rows, 67 heads x 2042 keys 36.4 : 36.0, d = 64 24.9 : 24.5; 130 x 1100, d = 64, 128 rows 28.8 : 28.5.
template <int TURN>
__device__ __forceinline__ float2 fold_row(const float2* __restrict__ p, int first, int by, int segs, int Rpad) {
  float M = NEG_BIG, Z = 0.f;
#pragma unroll 1
  for (int i = first; i < segs; i += by * TURN) {
    float2 v[TURN];
    float top = M;
#pragma unroll
    for (int b = 0; b < TURN; ++b) v[b] = p[(size_t)min(i + b * by, segs - 1) * Rpad];
#pragma unroll
    for (int b = 0; b < TURN; ++b) {
      if (i + b * by >= segs) v[b] = make_float2(NEG_BIG, 0.f);
      top = fmaxf(top, v[b].x);
    }
    Z *= __builtin_amdgcn_exp2f(M - top);
#pragma unroll
    for (int b = 0; b < TURN; ++b) Z = fmaf(v[b].y, __builtin_amdgcn_exp2f(v[b].x - top), Z);
    M = top;
  }
  return make_float2(M, Z);
}

// M and the weight 1 / Z of the score rows r0 .. r0 + n - 1 from the statistics of the head's segments: THREADS / n threads share
// a row, fixed order.  (The caller's next barrier completes it.)
template <int TURN>
__device__ __forceinline__ void fold_segments(const float2* __restrict__ part, int segs, int Rpad, int R, int r0, int n, float2* fold, float* rowm, float* roww) {
  const int subs = THREADS / n, r = threadIdx.x % n, sub = threadIdx.x / n;
  if (sub < subs) fold[threadIdx.x] = fold_row<TURN>(part + r0 + r, sub, subs, segs, Rpad);
  __syncthreads();
  if (sub == 0) {
    float M = NEG_BIG, Z = 0.f;
    for (int i = 0; i < subs; ++i) merge_stat(M, Z, fold[i * n + r]);
    rowm[r] = M;
    roww[r] = r0 + r < R ? 1.f / Z : 0.f;
  }
}

// Pass 2: raw[j] = sum over the score rows of exp2(s - M) / Z, a group of row tiles after the other.  folded: the first segment's place in
// `part` holds (M, 1 / Z); else they are made here.
template <typename T, int NP, bool FULL>
__global__ __launch_bounds__(THREADS, (waves_per_simd<T, NP>())) void wave_score_kernel(ScoreGeom g, WindowPos qp, KvLayout lay, WavePlan pl,
                                                                               const T* __restrict__ q, const T* __restrict__ k,
                                                                               const float2* __restrict__ part,
                                                                               bool folded, float* __restrict__ raw, int* __restrict__ status) {
  extern __shared__ __align__(16) char smem[];
  __shared__ __align__(16) float rowm[MAX_TILES * 32], roww[MAX_TILES * 32];
  __shared__ __align__(16) int last[MAX_TILES * 32];     // last key the rows see
  const int tid = threadIdx.x;
  const int inst = pl.inst0 + pl.way * (int)blockIdx.z, head = pl.head0 + pl.way * (int)blockIdx.y;
  const size_t hg = (size_t)inst * g.Hkv + head;
  if (blockIdx.x == 0 && hg == 0 && tid == 0) *status = 0;    // (these kernels have no wait to give up)
  const Wave<T, NP, FULL> w(g, lay, q, k, inst, head, blockIdx.x, pl.seg_blocks);
  const RowScale row_scale = pl.row_scale;
  constexpr int TURN = is_f32(T()) ? 4 : 8;              // (fp32, d = 64: 8 spill two registers)
  float* out = raw + hg * g.L;
  u32x4 key[NP];
#pragma unroll 1
  for (int rt0 = 0; rt0 < g.Rpad / 32; rt0 += pl.group_tiles) {
    const int ntile = min(pl.group_tiles, g.Rpad / 32 - rt0), whole = whole_tiles<is_f32(T()) && FULL>(g, rt0, ntile);
    if (w.some) w.load(key, g, lay, w.first);
    if (rt0 > 0) __syncthreads();
    stage_rows16<T, FULL, THREADS>(smem, w.head_rows, w.row_bytes, w.plane, w.stride, g.R, rt0 * 32, ntile * 32, row_scale.shift);
    if (tid < ntile * 32) {
      const int row = rt0 * 32 + tid;
      last[tid] = last_visible_key(g, qp, min(row, g.R - 1) % g.W);
      if (folded) {
        const float2 c = part[hg * pl.segs * g.Rpad + row];
        rowm[tid] = c.x;
        roww[tid] = c.y;
      }
    }
    if (!folded)
      fold_segments<TURN>(part + hg * pl.segs * g.Rpad, pl.segs, g.Rpad, g.R, rt0 * 32, ntile * 32,
                    reinterpret_cast<float2*>(smem + pl.group_tiles * 32 * w.stride), rowm, roww);
    __syncthreads();
    const char* rows = smem + w.n16 * w.stride + w.grp * 16;
    auto work = [&](const Operand<T, NP, FULL>& op, int key0) {
      const bool plain = key0 + 31 <= g.qmin;
      auto masked = [&](Tile16& a, int rt, int row_halves) {
        if (!plain) {
#pragma unroll
          for (int r = 0; r < row_halves; ++r) {
            const i32x4 lv = *reinterpret_cast<const i32x4*>(last + rt * 32 + 16 * r + 4 * w.grp);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              if (key0 + 16 * (e >> 2) + w.n16 > lv[e & 3]) a.t[e >> 2][r][e & 3] = -INFINITY;
              if (is_f32(T()) && FULL) __builtin_amdgcn_sched_barrier(0);    // (one comparison at a time: registers)
            }
          }
        }
      };
      float sum0 = 0.f, sum1 = 0.f;                      // of keys n16 and 16 + n16 of the tile
      auto tile = [&](auto row_halves, int rt) {
        constexpr int RH = decltype(row_halves)::value;
        Tile16 a = op.template product<false, RH>(rows + rt * 32 * w.stride, w.stride, w.plane, w.plane / 64);
        masked(a, rt, RH);
#pragma unroll
        for (int r = 0; r < RH; ++r) {
          const f32x4 m = *reinterpret_cast<const f32x4*>(rowm + rt * 32 + 16 * r + 4 * w.grp);
          const f32x4 wt = *reinterpret_cast<const f32x4*>(roww + rt * 32 + 16 * r + 4 * w.grp);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            sum0 = fmaf(__builtin_amdgcn_exp2f(fmaf(a.t[0][r][i], row_scale.scale2, -m[i])), wt[i], sum0);
            sum1 = fmaf(__builtin_amdgcn_exp2f(fmaf(a.t[1][r][i], row_scale.scale2, -m[i])), wt[i], sum1);
          }
        }
      };
#pragma unroll 1
      for (int rt = 0; rt < whole; ++rt) tile(std::integral_constant<int, 2>{}, rt);
      if (is_f32(T()) && FULL && whole < ntile) tile(std::integral_constant<int, 1>{}, whole);
      const auto plus = [](float x, float y) { return x + y; };
      float both = over_groups(sum0, sum1, plus);
      const int j = key0 + (w.grp >> 1 << 4) + w.n16;    // the key whose sum this lane ends with
      if (__builtin_expect(__any((both < TINY || (is_f32(T()) && both != both)) && j < g.L), 0)) {
        sum0 = sum1 = 0.f;
#pragma unroll 1
        for (int rt = 0; rt < ntile; ++rt) {
          Tile16 a;
          if constexpr (is_f32(T())) {
            const char *kr[2], *qr[2];
            w.key_rows(kr, g, lay, key0);
            w.score_rows(qr, g, rt0 + rt);
            a = product16_f32<false>(kr, qr, w.grp, w.row_bytes);
          } else {
            a = op.template product<false, 2>(rows + rt * 32 * w.stride, w.stride, w.plane, w.plane / 64);
          }
          masked(a, rt, 2);
#pragma unroll 1
          for (int e = 0; e < 8; ++e) {                  // rows 16 (e / 4) + 4 grp + e % 4
            const int row = rt * 32 + 16 * (e >> 2) + 4 * w.grp + (e & 3);
            const float c = rowm[row] - __builtin_amdgcn_logf(roww[row]);                  // (no weight: infinite)
            const float x0 = fmaf(a.t[0][0][0], g.scale2, -c), x1 = fmaf(a.t[1][0][0], g.scale2, -c);
            sum0 += x0 < -126.f ? __builtin_amdgcn_exp2f(x0 + 64.f) * 0x1p-64f : __builtin_amdgcn_exp2f(x0);
            sum1 += x1 < -126.f ? __builtin_amdgcn_exp2f(x1 + 64.f) * 0x1p-64f : __builtin_amdgcn_exp2f(x1);
#pragma unroll
            for (int s = 0; s < 2; ++s) {                // the next element to the front
              const float first = a.t[s][1][0];
              a.t[s][0] = f32x4{a.t[s][0][1], a.t[s][0][2], a.t[s][0][3], first};
              a.t[s][1] = f32x4{a.t[s][1][1], a.t[s][1][2], a.t[s][1][3], 0.f};
            }
          }
        }
        both = over_groups(sum0, sum1, plus);
      }
      if ((w.grp & 1) == 0 && j < w.end) out[j] = rt0 > 0 ? out[j] + both : both;
    };
    if (w.some) walk_tiles<T, NP, FULL>(key, w.first, w.last_tile, [&](u32x4 (&x)[NP], int key0) { w.load(x, g, lay, key0); }, work);
  }
}

// Combine the (m, z) of all segments of a head, one workgroup per (head, 32-row tile): 8 threads share a row and split the segments; fixed
// merge order.  rowc: c = M + log2 Z per score row; null: (M, 1 / Z) take the place of the first segment's.
__global__ __launch_bounds__(256) void row_constants_kernel(ScoreGeom g, float2* part, float* __restrict__ rowc) {
  __shared__ float2 stat[256];
  const int hg = blockIdx.x, rt = blockIdx.y, tid = threadIdx.x;
  const int r = rt * 32 + (tid & 31), sel = tid >> 5;
  float2* p = part + (size_t)hg * g.nchunk * g.Rpad + r;
  stat[tid] = fold_row<16>(p, sel, 8, g.nchunk, g.Rpad);
  __syncthreads();
  if (tid < 32) {
    float M = stat[tid].x, Z = stat[tid].y;
    for (int s2 = 1; s2 < 8; ++s2) merge_stat(M, Z, stat[s2 * 32 + tid]);
    if (rowc) rowc[(size_t)hg * g.Rpad + r] = (r < g.R) ? M + __builtin_amdgcn_logf(Z) : 1.0e30f;
    else *p = make_float2(M, r < g.R ? 1.f / Z : 0.f);
  }
}

constexpr int MAX_LDS = 160 << 10, STATIC_LDS = 3 * MAX_TILES * 32 * 4;   // (the second kernel's arrays; the first has none)

// How a call's keys are cut into segments.  A segment costs its blocks and about three more (the score rows' way to LDS, the first keys'
// to the registers).  Where a workgroup has few blocks, the cut with the least of that over the rounds of resident workgroups it takes
// (and a little per segment, which the second kernel folds, or a launch that does): 64 heads x 8191 keys, fp32, 512 resident workgroups: 8, 16,
// 32 segments (1, 2, 4 rounds) 122, 144, 169 us.  Where a workgroup has many, segments of 10 to 16 blocks, so that workgroups which get ahead of
// others take more of them: 1800 heads x 20259 keys, d = 64: 1, 3, 5, 16, 80 segments 2047, 1936, 1862, 1844, 2102 us.
// Where these are few rounds, what the last one leaves idle counts: a round that is not full takes 0.6 of one at least, and a single one, which nothing
// evens out, 1.08; a segment its blocks and 1.5 (of 8 to 20 blocks).  laq_evict, us, by segments (rounds): 112 rows, 112 heads x 20123 keys 9 (0.98) 277, 16
// (1.75) 266.5, 18 (1.97) 273; fp32, 128 x 8191 4 (1) 251, 5 (1.25) 279.5, 8 (2) 253, 16 (4) 273; d = 64, 64 rows, 160 x 16384 8 (1) 140.7, 10 (1.25) 146.3,
// 16 (2) 140.3; 32 rows, 320 x 9000 4 (1) 163, 7 (1.75) 168, 8 (2) 161, 12 (3) 164.
// Fewer segments than these 10 to 16 blocks make are not taken for it: token-major caches, d = 64, 32 rows, 280 heads x 19097 keys 15 (3.28) 292, 8 (1.75) 342; 1008 x 3759 3 (2.36)
// 234, 2 (1.57) 265; fp32, d = 96, 64 rows, 144 x 15336 10 (2.81) 396, 6 (1.69) 420; d = 64, 32 rows, 112 x 26356 19 (2.77) 306.5, 11 (1.60) 321.5.  (66 such calls
// .85-1.05 of the time with the more of them, two 1.05-1.11.)
// More score rows than are staged together are other workgroups' in the first kernel, but in the second the same one takes a group after the other.
// Its rounds count that often; but where not all workgroups that fit are there, those that are get on faster: a share `enough` of them
// does what all do (bf16 1.25 waves per SIMD, fp32 2), though never less than the first kernel's.  laq_evict, the second counted as
// the first : so, us: fp32, 256 rows, d = 128, 64 heads x 3300 285 : 212,
// 16 x 4000 114.5 : 87.9, 300 x 3000 866 : 787; 448 rows, d = 96, 16 x 8000 220 : 173.  With all the workgroups that fit counted as needed: bf16, 160 rows,
// d = 128, 256 x 1500 81 : 91; 224 rows, d = 256, 128 x 1100 80 : 91.
WavePlan plan_of(const ScoreGeom& g, int resident, double enough, int lds, int first_per_simd, int stride) {
  WavePlan pl;
  const int ntile = g.Rpad / 32, blocks = (g.L + BLOCK_KEYS - 1) / BLOCK_KEYS;
  const long long heads = (long long)g.n_inst * g.Hkv;
  int fit = std::min(lds / (32 * stride + WAVES * 32 * (int)sizeof(float2)), (lds - STATIC_LDS - THREADS * (int)sizeof(float2)) / (32 * stride));
  fit = std::max(1, std::min(fit, MAX_TILES));
  // Heads of one block: row tiles so few that as many of the first kernel's workgroups fit as its registers allow.  laq_evict, us, four tiles : three, 448 rows, d = 168,
  // 1000 heads x 60 keys 202 : 183.5, x 120 245 : 232, 300 x 60 88 : 79; d = 192, 1000 x 60 215.5 : 202.5.  (Longer heads are read once more by the second kernel.)
  const int first_fit = MAX_LDS / first_per_simd / (32 * stride + WAVES * 32 * (int)sizeof(float2));
  if (blocks == 1 && first_fit >= 3) fit = std::min(fit, first_fit);
  pl.groups = (ntile + fit - 1) / fit;
  pl.group_tiles = (ntile + pl.groups - 1) / pl.groups;
  pl.groups = (ntile + pl.group_tiles - 1) / pl.group_tiles;
  const int most = std::min(blocks, g.nchunk);           // (the workspace has room for a segment per 256 keys)
  int best = 1;
  if (heads * blocks >= 15LL * resident) {
    best = std::max(1, std::min(most, blocks / (8 + 2 * pl.group_tiles)));
    if (pl.groups == 1 && 2 * heads * best < 9 * resident) {
      const int before = best;
      double least = 1e30;
      for (int sb = 8; sb <= 20; ++sb) {
        const int used = (blocks + sb - 1) / sb;
        if (used > most || used < before) continue;
        const double load = (double)(heads * used) / resident, rounds = std::floor(load), rest = load - rounds;
        const double cost = (load <= 1.0 ? 1.08 : rest > 0.0 ? rounds + std::max(rest, 0.6) : rounds) * (sb + 1.5);
        if (cost < least) { least = cost; best = used; }
      }
    }
  } else {
    double least = 1e30;
    for (const double share : {0.0, 0.25, 0.35, 0.5, 0.7, 1.0, 1.5, 2.0, 3.0}) {
      const int s = std::max(1, std::min(most, (int)(share * resident / heads)));
      const int sb = (blocks + s - 1) / s, used = (blocks + sb - 1) / sb;
      const long long first = (heads * used * pl.groups + resident - 1) / resident;
      double second = first;
      if (pl.groups > 1) {
        const double load = (double)(heads * used) / resident;
        second = std::max(second, pl.groups * (load <= 1.0 ? std::max(load, enough) : std::ceil(load)));
      }
      const double cost = 0.5 * (first + second) * (sb + 3.0) + 0.1 * sb + 0.12 * used + (used > FOLD_SEGMENTS ? 3.0 : 0.0);
      if (cost < least) { least = cost; best = s; }
    }
  }
  pl.seg_blocks = (blocks + best - 1) / best;
  pl.segs = (blocks + pl.seg_blocks - 1) / pl.seg_blocks;
  return pl;
}

template <typename T, int NP, bool FULL>
hipError_t launch_wave(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, const T* q, const T* k, float* raw,
                       const Workspace& ws, hipStream_t st) {
  constexpr int per_simd = waves_per_simd<T, NP>();
  const int stride = row16_stride<T>(g.d);
  WavePlan pl = plan_of(g, 256 * per_simd, (is_f32(T()) ? 2.0 : 1.25) / per_simd, MAX_LDS / per_simd, stats_waves_per_simd<T, NP>(), stride);
  pl.row_scale = row_scale_of<T>(g.scale2);
  // Where the keys do not fit the last-level cache (256 MiB), the second kernel begins with the heads that the first one read last.  laq_evict, us, in the
  // same order : so, on the same cache every time; on one that no earlier call has read:
  //   bf16, 128 rows, heads x 8192 keys  250 MiB 119 : 118.5, 126.5 : 127;  280 MiB 139.5 : 135, 148 : 144;  500 MiB 243 : 228, 242 : 233
  //   d = 64, 64 rows, x 8192            230 MiB 98 : 98.5, 111 : 111.5;  280 MiB 140 : 137, 151 : 146;  500 MiB 246 : 224, 243.5 : 230.5
  //   d = 96, 64 rows, x 4000            230 MiB 107 : 109, 121 : 120.5;  280 MiB 135 : 130, 148 : 140.5;  350 MiB 181 : 165, 185 : 174
  //   fp32, 64 rows, x 8191              250 MiB 125 : 125, 137 : 138;  280 MiB 153.5 : 152, 161 : 159;  500 MiB 261 : 250, 262 : 257
  // In small calls the same workgroup numbers find their keys in the L2 of their XCD: d = 64, 64 rows, 24 x 8192, 24 MiB, 28.4 : 30.0, 31.7 : 32.9.
  const bool other = (double)g.n_inst * g.Hkv * g.L * g.d * sizeof(T) > (double)(256 << 20);
  pl.way = other ? -1 : 1;
  pl.head0 = other ? g.Hkv - 1 : 0;
  pl.inst0 = other ? g.n_inst - 1 : 0;
  const int rows = pl.group_tiles * 32;
  hipLaunchKernelGGL((wave_stats_kernel<T, NP, FULL>), dim3(pl.segs * pl.groups, g.Hkv, g.n_inst), dim3(THREADS),
                     rows * (stride + WAVES * (int)sizeof(float2)), st, g, qp, lay, pl, q, k, ws.part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool fold = pl.segs <= FOLD_SEGMENTS;
  if (!fold) {
    ScoreGeom gs = g;
    gs.nchunk = pl.segs;
    if ((e = launch_row_constants(gs, ws, nullptr, st)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL((wave_score_kernel<T, NP, FULL>), dim3(pl.segs, g.Hkv, g.n_inst), dim3(THREADS), rows * stride + THREADS * (int)sizeof(float2),
                     st, g, qp, lay, pl, q, k, ws.part, !fold, raw, ws.status);
  return hipGetLastError();
}

template <typename T, int NP, bool FULL> hipError_t init_wave() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wave_stats_kernel<T, NP, FULL>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     MAX_LDS - STATIC_LDS);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&wave_score_kernel<T, NP, FULL>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             MAX_LDS - STATIC_LDS);
}

}  // namespace

// c = M + log2 Z of every score row from the statistics of g.nchunk segments of every head into rowc; null: (M, 1 / Z) into the statistics'
// first segment
hipError_t launch_row_constants(const ScoreGeom& g, const Workspace& ws, float* rowc, hipStream_t st) {
  const long long n_heads = (long long)g.n_inst * g.Hkv;
  hipLaunchKernelGGL(row_constants_kernel, dim3((unsigned)n_heads, g.Rpad / 32), dim3(256), 0, st, g, ws.part, rowc);
  return hipGetLastError();
}

hipError_t score_wave_init() {
  hipError_t e;
  if ((e = init_wave<uint16_t, 4, true>()) != hipSuccess || (e = init_wave<uint16_t, 6, true>()) != hipSuccess ||
      (e = init_wave<uint16_t, 8, true>()) != hipSuccess || (e = init_wave<uint16_t, 16, true>()) != hipSuccess ||
      (e = init_wave<uint16_t, 16, false>()) != hipSuccess || (e = init_wave<float, 8, true>()) != hipSuccess ||
      (e = init_wave<float, 12, true>()) != hipSuccess || (e = init_wave<float, 16, true>()) != hipSuccess)
    return e;
  return init_wave<float, 16, false>();
}

bool score_wave_supported(const ScoreGeom& g, int dtype) { return dtype == LAQ_BF16 || g.d <= 128; }

bool score_wave_own_size(const ScoreGeom& g, int dtype) {
  return g.d == 64 || g.d == 96 || g.d == 128 || (dtype == LAQ_BF16 && g.d == 256);
}

hipError_t launch_score_wave(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, const void* q, const void* k,
                             float* raw, const Workspace& ws, hipStream_t st) {
  if (dtype == LAQ_F32) {
    const float *qq = static_cast<const float*>(q), *kk = static_cast<const float*>(k);
    if (g.d == 64) return launch_wave<float, 8, true>(g, qp, lay, qq, kk, raw, ws, st);
    if (g.d == 96) return launch_wave<float, 12, true>(g, qp, lay, qq, kk, raw, ws, st);
    if (g.d == 128) return launch_wave<float, 16, true>(g, qp, lay, qq, kk, raw, ws, st);
    return launch_wave<float, 16, false>(g, qp, lay, qq, kk, raw, ws, st);
  }
  const uint16_t *qq = static_cast<const uint16_t*>(q), *kk = static_cast<const uint16_t*>(k);
  if (g.d == 64) return launch_wave<uint16_t, 4, true>(g, qp, lay, qq, kk, raw, ws, st);
  if (g.d == 96) return launch_wave<uint16_t, 6, true>(g, qp, lay, qq, kk, raw, ws, st);
  if (g.d == 128) return launch_wave<uint16_t, 8, true>(g, qp, lay, qq, kk, raw, ws, st);
  if (g.d == 256) return launch_wave<uint16_t, 16, true>(g, qp, lay, qq, kk, raw, ws, st);
  return launch_wave<uint16_t, 16, false>(g, qp, lay, qq, kk, raw, ws, st);
}

}  // namespace laq
