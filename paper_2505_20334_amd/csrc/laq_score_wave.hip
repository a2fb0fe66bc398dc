// Scoring in two passes over K without a barrier between keys: every head size up to 256, any number of score
// rows, fp32 or bf16, on the matrix cores (v_mfma_f32_32x32x16_bf16).
//
// Kernel 1 leaves the softmax statistics (m, z) of every score row over a segment of a head's keys, kernel 2 folds
// the segments' (or finds them folded by row_constants_kernel, where they are many) and sums the probabilities
// exp2(s - c), c = M + log2 Z, over the rows: raw scores.
//
// A workgroup of four waves stages the head's score rows (up to 128 of them) in LDS once and then walks its segment
// of keys, 128 at a time; a wave takes 32 of these in registers, straight from memory in operand layout (lane l: row
// l % 32, the 16-byte pieces 2t + l / 32), while the next 32 are on their way into others.  Nothing that a wave does
// per key waits for another wave, so loads and arithmetic of the 8 to 20 waves of a compute unit mix freely.
//   (1) D = K * Q^T: lane = score row, registers = 16 keys: sum (and, where it is needed, maximum) in registers, the wave's running (m, z) in LDS.
//   (2) D = Q * K^T: lane = key, registers = 16 rows: the sum over the rows in registers.
// Score rows beyond R repeat the last one and get c = inf, so that they add nothing.
//
// fp32 takes six bf16 products: a float is the sum of three bf16 (split8), and the three products of parts that together reach
// 2^-24 of the whole at most are left out.  The sums are fp32, those of the small products apart from those of the large ones: fewer
// roundings than the fp32 instruction makes.  Error against 64 bits (2-norm of the scores, d = 64, 96, 104, 128, logits of standard
// deviation 1 / 4): 1.85-1.9e-7 / 4.5-4.9e-7, with the fp32 instruction 1.9e-7 / 7.9-9.7e-7; and 2.7 times its rate.  Rows of a single
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
  int hf, n32, wave;
  int row_bytes, stride, plane;
  int inst;
  int64_t src_row;         // bytes between key rows
  const char *head_keys, *head_rows;
  int first, last_tile, end;
  bool some;

  __device__ __forceinline__ Wave(const ScoreGeom& g, const KvLayout& lay, const T* q, const T* k, int seg, int seg_blocks) {
    const int lane = threadIdx.x & 63, head = blockIdx.y;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    hf = lane >> 5;
    n32 = lane & 31;
    inst = blockIdx.z;
    row_bytes = FULL ? NP * 32 : g.d * (int)sizeof(T);
    plane = plane_bytes(row_bytes / (int)sizeof(T));
    stride = row_stride<T>(row_bytes / (int)sizeof(T));
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
  // this lane's row of the tile of keys key0 .. key0 + 31
  __device__ __forceinline__ const char* key_row(const ScoreGeom& g, const KvLayout& lay, int key0) const {
    int r0 = key0;
    const char* p = head_keys;
    if (lay.table) p += paged_block_offset(lay, inst, key0, &r0) * (int64_t)sizeof(T);      // (a block holds whole tiles)
    const int row = min(n32, g.L - 1 - key0);            // (keys beyond the last one are masked: any row will do)
    return p + (int64_t)(r0 + row) * src_row;
  }
  __device__ __forceinline__ void load(u32x4 (&key)[NP], const ScoreGeom& g, const KvLayout& lay, int key0) const {
    const char* p = key_row(g, lay, key0) + hf * 16;
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      if (FULL) {
        key[t] = *reinterpret_cast<const u32x4*>(p + t * 32);
      } else {
        key[t] = u32x4{0u, 0u, 0u, 0u};
        if ((2 * t + hf) * 16 < row_bytes) key[t] = *reinterpret_cast<const u32x4*>(p + t * 32);
      }
    }
  }

  // this lane's score row of a tile, in memory
  __device__ __forceinline__ const char* score_row(const ScoreGeom& g, int rt) const {
    return head_rows + (size_t)min(rt * 32 + n32, g.R - 1) * row_bytes;
  }
};

// A key tile as the products take it; fp32: split into its three parts.
template <typename T, int NP, bool FULL> struct Operand {
  static constexpr bool F32 = is_f32(T());
  static constexpr int STEPS = F32 ? (NP + 1) / 2 : NP;
  u32x4 v[F32 ? 3 * STEPS : STEPS];
  __device__ __forceinline__ void from(const u32x4 (&key)[NP]) {
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
      if constexpr (F32) {
        const u32x4 none = {0u, 0u, 0u, 0u};
        const Split s = split8(key[2 * u], 2 * u + 1 < NP ? key[2 * u + 1 < NP ? 2 * u + 1 : 0] : none);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) v[3 * u + pl] = s.p[pl];
      } else {
        v[u] = key[u];
      }
    }
  }
  // against the score rows at `lds` (this lane's row and half); `steps` of 32 bytes a row has, `plane` bytes between its parts
  template <bool KEYS_AS_ROWS>
  __device__ __forceinline__ f32x16 product(const char* lds, int plane, int steps) const {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc = zero;
    if constexpr (F32) {
      f32x16 low = zero;
      u32x4 q0, q1, q2;
      auto fetch = [&](int u) {
        q0 = *reinterpret_cast<const u32x4*>(lds + u * 32);
        q1 = *reinterpret_cast<const u32x4*>(lds + plane + u * 32);
        q2 = *reinterpret_cast<const u32x4*>(lds + 2 * plane + u * 32);
      };
      fetch(0);
#pragma unroll
      for (int u = 0; u < STEPS; ++u) {
        if (FULL || u < steps) {
          const u32x4 a0 = q0, a1 = q1, a2 = q2;
          if (u + 1 < STEPS && (FULL || u + 1 < steps)) fetch(u + 1);      // one step ahead of the products
          __builtin_amdgcn_sched_barrier(0);
          low = mm<KEYS_AS_ROWS>(v[3 * u + 2], a0, low);
          acc = mm<KEYS_AS_ROWS>(v[3 * u], a0, acc);
          low = mm<KEYS_AS_ROWS>(v[3 * u], a2, low);
          low = mm<KEYS_AS_ROWS>(v[3 * u + 1], a1, low);
          low = mm<KEYS_AS_ROWS>(v[3 * u + 1], a0, low);
          low = mm<KEYS_AS_ROWS>(v[3 * u], a1, low);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      acc += low;
    } else {
#pragma unroll
      for (int u = 0; u < STEPS; ++u) {
        if (FULL || u < steps) acc = mm<KEYS_AS_ROWS>(v[u], *reinterpret_cast<const u32x4*>(lds + u * 32), acc);
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);                 // (at most four operands of Q requested ahead: registers)
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
  RowScale row_scale;
};

// Waves per SIMD the kernels are built for: as many as their registers (and 32 of the score rows per workgroup in LDS) allow.
template <typename T, int NP> constexpr int waves_per_simd() { return is_f32(T()) ? (NP <= 8 ? 3 : 2) : (NP <= 6 ? 5 : NP <= 8 ? 4 : 2); }

// A wave's sums of exponentials refer to a number near the row's maximum, not to the maximum itself: HEADROOM above that of the first
// tile, and moved only where a tile's sum reaches OUTGROWN of it (then, and where a row does not see all keys of a tile, or a sum is no
// number, the maximum of the tile is made).  The terms that count have exponents between -8 and 7, as with a maximum that most keys stay
// some powers of two below.  A gain in error and in instructions rather than in time: scores against 64 bits (2-norm, logits of deviation 1)
// bf16 3.0e-7 -> 2.0e-7, fp32 2.2e-7 -> 1.9e-7; 71 instead of 87 vector instructions per product of 32 keys and 32 rows (SQ_INSTS_VALU); the whole
// eviction of 256 heads x 32768 keys, 128 rows, is not faster beyond noise (934 : 927 us): it is bound by memory and by the power that memory and
// matrix cores take.
constexpr float HEADROOM = 3.f, OUTGROWN = 128.f;
// exp2(s * scale - m) of a lane's 16 keys and of the 16 that the other half of the wave has of the same row, summed
__device__ __forceinline__ float tile_sum(const f32x16& s, float scale, float m) {
  float z[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i & 1] += __builtin_amdgcn_exp2f(fmaf(s[i], scale, -m));
  z[0] += z[1];
  const auto zh = __builtin_amdgcn_permlane32_swap(__float_as_uint(z[0]), __float_as_uint(z[0]), false, false);
  return __uint_as_float(zh[0]) + __uint_as_float(zh[1]);
}

// Pass 1: part[head][segment][row] = (m, z) of a score row over the segment's visible keys, in log2 units.
template <typename T, int NP, bool FULL>
__global__ __launch_bounds__(THREADS, (waves_per_simd<T, NP>())) void wave_stats_kernel(ScoreGeom g, WindowPos qp, KvLayout lay, WavePlan pl,
                                                                               const T* __restrict__ q, const T* __restrict__ k,
                                                                               float2* __restrict__ part) {
  extern __shared__ __align__(16) char smem[];
  const int group = blockIdx.x / pl.segs, seg = blockIdx.x - group * pl.segs;
  const int rt0 = group * pl.group_tiles, ntile = min(pl.group_tiles, g.Rpad / 32 - rt0);
  const Wave<T, NP, FULL> w(g, lay, q, k, seg, pl.seg_blocks);
  const RowScale row_scale = pl.row_scale;
  u32x4 key[NP];
  if (w.some) w.load(key, g, lay, w.first);
  stage_rows<T, FULL, THREADS>(smem, w.head_rows, w.row_bytes, w.plane, w.stride, g.R, rt0 * 32, ntile * 32, row_scale.shift);
  float2* stat = reinterpret_cast<float2*>(smem + pl.group_tiles * 32 * w.stride);       // [row tile][wave][row]
  for (int i = threadIdx.x; i < ntile * WAVES * 32; i += THREADS) stat[i] = make_float2(NEG_BIG, 0.f);
  __syncthreads();
  auto work = [&](const Operand<T, NP, FULL>& op, int key0) {
    const bool plain = key0 + 31 <= g.qmin;              // every row sees every key
    const char* rows = smem + w.n32 * w.stride + w.hf * 16;
    float2* mine = stat + w.wave * 32 + w.n32;
#pragma unroll 1
    for (int rt = 0; rt < ntile; ++rt) {
      const float2 old = *mine;
      f32x16 s = op.template product<true>(rows, w.plane, w.plane / 32);
      float z = plain && key0 != w.first ? tile_sum(s, row_scale.scale2, old.x) : INFINITY;
      if (__builtin_expect(!__any(!(z <= OUTGROWN)), 1)) {
        mine->y = old.y + z;
      } else {
        float m, scale = row_scale.scale2;
#pragma unroll 1
        for (bool again = false;; again = true) {
          if (!plain) {
            int n = threadIdx.x & 63;
            asm volatile("" : "+v"(n));                  // (computed here: the common case has no registers for it)
            const int row = (rt0 + rt) * 32 + (n & 31), last = last_visible_key(g, qp, min(row, g.R - 1) % g.W) - key0;
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (acc_row(i, n >> 5) > last) s[i] = -INFINITY;
          }
          m = s[0];
#pragma unroll
          for (int i = 1; i < 16; ++i) m = fmaxf(m, s[i]);
          const auto mh = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
          m = fmaxf(old.x, fmaf(fmaxf(__uint_as_float(mh[0]), __uint_as_float(mh[1])), scale, HEADROOM));    // (the logit scale is positive)
          z = tile_sum(s, scale, m);
          if (!is_f32(T()) || again || __builtin_expect(!__any(z != z), 1)) break;
          s = product_f32<true>(w.key_row(g, lay, key0), w.score_row(g, rt0 + rt), w.hf, w.row_bytes);
          scale = g.scale2;
        }
        *mine = make_float2(m, fmaf(old.y, __builtin_amdgcn_exp2f(old.x - m), z));
      }
      rows += 32 * w.stride;
      mine += WAVES * 32;
    }
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

// c = M + log2 Z of the score rows r0 .. r0 + n - 1 from the statistics of the head's segments: THREADS / n threads share
// a row, fixed order.  (The caller's next barrier completes it.)
__device__ __forceinline__ void fold_segments(const float2* __restrict__ part, int segs, int Rpad, int R, int r0, int n, float2* fold, float* rowc) {
  constexpr int TURN = 8;
  const int subs = THREADS / n, r = threadIdx.x % n, sub = threadIdx.x / n;
  if (sub < subs) {
    const float2* p = part + r0 + r;
    float M = NEG_BIG, Z = 0.f;
#pragma unroll 1
    for (int i = sub; i < segs; i += subs * TURN) {
      float2 v[TURN];
#pragma unroll
      for (int b = 0; b < TURN; ++b) v[b] = p[(size_t)min(i + b * subs, segs - 1) * Rpad];
#pragma unroll
      for (int b = 0; b < TURN; ++b)
        if (i + b * subs < segs) merge_stat(M, Z, v[b]);
    }
    fold[threadIdx.x] = make_float2(M, Z);
  }
  __syncthreads();
  if (sub == 0) {
    float M = NEG_BIG, Z = 0.f;
    for (int i = 0; i < subs; ++i) merge_stat(M, Z, fold[i * n + r]);
    rowc[r] = r0 + r < R ? M + __builtin_amdgcn_logf(Z) : INFINITY;
  }
}

// Pass 2: raw[j] = sum over the score rows of exp2(s - c[row]), a group of row tiles after the other.  rowc_all: the heads' row
// constants, or null: folded here.
template <typename T, int NP, bool FULL>
__global__ __launch_bounds__(THREADS, (waves_per_simd<T, NP>())) void wave_score_kernel(ScoreGeom g, WindowPos qp, KvLayout lay, WavePlan pl,
                                                                               const T* __restrict__ q, const T* __restrict__ k,
                                                                               const float2* __restrict__ part,
                                                                               const float* __restrict__ rowc_all,
                                                                               float* __restrict__ raw, int* __restrict__ status) {
  extern __shared__ __align__(16) char smem[];
  __shared__ __align__(16) float rowc[MAX_TILES * 32];
  __shared__ __align__(16) int last[MAX_TILES * 32];     // last key the rows see
  const int tid = threadIdx.x;
  const size_t hg = (size_t)blockIdx.z * g.Hkv + blockIdx.y;
  if (blockIdx.x == 0 && hg == 0 && tid == 0) *status = 0;    // (these kernels have no wait to give up)
  const Wave<T, NP, FULL> w(g, lay, q, k, blockIdx.x, pl.seg_blocks);
  const RowScale row_scale = pl.row_scale;
  float* out = raw + hg * g.L;
  u32x4 key[NP];
#pragma unroll 1
  for (int rt0 = 0; rt0 < g.Rpad / 32; rt0 += pl.group_tiles) {
    const int ntile = min(pl.group_tiles, g.Rpad / 32 - rt0);
    if (w.some) w.load(key, g, lay, w.first);
    if (rt0 > 0) __syncthreads();
    stage_rows<T, FULL, THREADS>(smem, w.head_rows, w.row_bytes, w.plane, w.stride, g.R, rt0 * 32, ntile * 32, row_scale.shift);
    if (tid < ntile * 32) {
      const int row = rt0 * 32 + tid;
      last[tid] = last_visible_key(g, qp, min(row, g.R - 1) % g.W);
      if (rowc_all) rowc[tid] = row < g.R ? rowc_all[hg * g.Rpad + row] : INFINITY;
    }
    if (!rowc_all)
      fold_segments(part + hg * pl.segs * g.Rpad, pl.segs, g.Rpad, g.R, rt0 * 32, ntile * 32,
                    reinterpret_cast<float2*>(smem + pl.group_tiles * 32 * w.stride), rowc);
    __syncthreads();
    const char* rows = smem + w.n32 * w.stride + w.hf * 16;
    auto work = [&](const Operand<T, NP, FULL>& op, int key0) {
      const bool plain = key0 + 31 <= g.qmin;
      const int j = key0 + w.n32;
      auto masked = [&](f32x16 s, int rt) {
        if (!plain) {
#pragma unroll
          for (int gq = 0; gq < 4; ++gq) {
            const i32x4 lv = *reinterpret_cast<const i32x4*>(last + rt * 32 + 8 * gq + 4 * w.hf);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (j > lv[i]) s[4 * gq + i] = -INFINITY;
          }
        }
        return s;
      };
      float sum = 0.f;
#pragma unroll 1
      for (int rt = 0; rt < ntile; ++rt) {
        const f32x16 s = masked(op.template product<false>(rows + rt * 32 * w.stride, w.plane, w.plane / 32), rt);
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const f32x4 c = *reinterpret_cast<const f32x4*>(rowc + rt * 32 + 8 * gq + 4 * w.hf);
#pragma unroll
          for (int i = 0; i < 4; ++i) sum += __builtin_amdgcn_exp2f(fmaf(s[4 * gq + i], row_scale.scale2, -c[i]));
        }
      }
      const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
      float both = __uint_as_float(halves[0]) + __uint_as_float(halves[1]);
      if (__builtin_expect(__any((both < TINY || (is_f32(T()) && both != both)) && j < g.L), 0)) {
        sum = 0.f;
#pragma unroll 1
        for (int rt = 0; rt < ntile; ++rt) {
          f32x16 s;
          if constexpr (is_f32(T())) s = product_f32<false>(w.key_row(g, lay, key0), w.score_row(g, rt0 + rt), w.hf, w.row_bytes);
          else s = op.template product<false>(rows + rt * 32 * w.stride, w.plane, w.plane / 32);
          s = masked(s, rt);
#pragma unroll 1
          for (int i = 0; i < 16; ++i) {
            const float x = fmaf(s[0], g.scale2, -rowc[rt * 32 + acc_row(i, w.hf)]);
            sum += x < -126.f ? __builtin_amdgcn_exp2f(x + 64.f) * 0x1p-64f : __builtin_amdgcn_exp2f(x);
            s = __builtin_shufflevector(s, s, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 0);
          }
        }
        both = sum + __shfl_xor(sum, 32);
      }
      if (w.hf == 0 && j < w.end) out[j] = rt0 > 0 ? out[j] + both : both;
    };
    if (w.some) walk_tiles<T, NP, FULL>(key, w.first, w.last_tile, [&](u32x4 (&x)[NP], int key0) { w.load(x, g, lay, key0); }, work);
  }
}

// Combine the (m, z) of all segments of a head into c = M + log2 Z per score row.  One workgroup per
// (head, 32-row tile): 8 threads share a row and split the segments; fixed merge order.
__global__ __launch_bounds__(256) void row_constants_kernel(ScoreGeom g, const float2* __restrict__ part,
                                                            float* __restrict__ rowc) {
  __shared__ float2 stat[256];
  const int hg = blockIdx.x, rt = blockIdx.y, tid = threadIdx.x;
  const int r = rt * 32 + (tid & 31), sel = tid >> 5;
  const float2* p = part + (size_t)hg * g.nchunk * g.Rpad + r;
  float M = NEG_BIG, Z = 0.f;
  constexpr int B = 16;
  for (int c0 = sel; c0 < g.nchunk; c0 += 8 * B) {
    float2 buf[B];
#pragma unroll
    for (int b = 0; b < B; ++b) buf[b] = p[(size_t)min(c0 + 8 * b, g.nchunk - 1) * g.Rpad];
#pragma unroll
    for (int b = 0; b < B; ++b)
      if (c0 + 8 * b < g.nchunk) merge_stat(M, Z, buf[b]);
  }
  stat[tid] = make_float2(M, Z);
  __syncthreads();
  if (tid < 32) {
    for (int s2 = 1; s2 < 8; ++s2) merge_stat(M, Z, stat[s2 * 32 + tid]);
    rowc[(size_t)hg * g.Rpad + r] = (r < g.R) ? M + __builtin_amdgcn_logf(Z) : 1.0e30f;
  }
}

// How a call's keys are cut into segments.  A segment costs its blocks and about three more (the score rows' way to LDS, the first keys'
// to the registers).  Where a workgroup has few blocks, the cut with the least of that over the rounds of resident workgroups it takes
// (and a little per segment, which the second kernel folds, or a launch that does): 64 heads x 8191 keys, fp32, 512 resident workgroups: 8, 16,
// 32 segments (1, 2, 4 rounds) 122, 144, 169 us.  Where a workgroup has many, segments of 10 to 16 blocks, so that workgroups which get ahead of
// others take more of them: 1800 heads x 20259 keys, d = 64: 1, 3, 5, 16, 80 segments 2047, 1936, 1862, 1844, 2102 us.
// More score rows than are staged together are other workgroups' in the first kernel, but in the second the same one takes a group after the other.
// Its rounds count that often; but where not all workgroups that fit are there, those that are get on faster: a share `enough` of them
// does what all do (bf16 1.25 waves per SIMD, fp32 2), though never less than the first kernel's.  laq_evict, the second counted as
// the first : so, us: fp32, 256 rows, d = 128, 64 heads x 3300 285 : 212,
// 16 x 4000 114.5 : 87.9, 300 x 3000 866 : 787; 448 rows, d = 96, 16 x 8000 220 : 173.  With all the workgroups that fit counted as needed: bf16, 160 rows,
// d = 128, 256 x 1500 81 : 91; 224 rows, d = 256, 128 x 1100 80 : 91.
WavePlan plan_of(const ScoreGeom& g, int resident, double enough, int lds, int stride) {
  WavePlan pl;
  const int ntile = g.Rpad / 32, blocks = (g.L + BLOCK_KEYS - 1) / BLOCK_KEYS;
  const long long heads = (long long)g.n_inst * g.Hkv;
  int fit = std::min(lds / (32 * stride + WAVES * 32 * (int)sizeof(float2)), (lds - THREADS * (int)sizeof(float2)) / (32 * stride));
  fit = std::max(1, std::min(fit, MAX_TILES));
  pl.groups = (ntile + fit - 1) / fit;
  pl.group_tiles = (ntile + pl.groups - 1) / pl.groups;
  pl.groups = (ntile + pl.group_tiles - 1) / pl.group_tiles;
  const int most = std::min(blocks, g.nchunk);           // (the workspace has room for a segment per 256 keys)
  int best = 1;
  if (heads * blocks >= 15LL * resident) {
    best = std::max(1, std::min(most, blocks / (8 + 2 * pl.group_tiles)));
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

constexpr int MAX_LDS = 160 << 10, STATIC_LDS = 2 * MAX_TILES * 32 * 4;

template <typename T, int NP, bool FULL>
hipError_t launch_wave(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, const T* q, const T* k, float* raw,
                       const Workspace& ws, hipStream_t st) {
  constexpr int per_simd = waves_per_simd<T, NP>();
  const int stride = row_stride<T>(g.d);
  WavePlan pl = plan_of(g, 256 * per_simd, (is_f32(T()) ? 2.0 : 1.25) / per_simd, (MAX_LDS / per_simd - STATIC_LDS) & ~255, stride);
  pl.row_scale = row_scale_of<T>(g.scale2);
  const int rows = pl.group_tiles * 32;
  hipLaunchKernelGGL((wave_stats_kernel<T, NP, FULL>), dim3(pl.segs * pl.groups, g.Hkv, g.n_inst), dim3(THREADS),
                     rows * (stride + WAVES * (int)sizeof(float2)), st, g, qp, lay, pl, q, k, ws.part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool fold = pl.segs <= FOLD_SEGMENTS;
  if (!fold) {
    ScoreGeom gs = g;
    gs.nchunk = pl.segs;
    if ((e = launch_row_constants(gs, ws, st)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL((wave_score_kernel<T, NP, FULL>), dim3(pl.segs, g.Hkv, g.n_inst), dim3(THREADS), rows * stride + THREADS * (int)sizeof(float2),
                     st, g, qp, lay, pl, q, k, ws.part, fold ? (const float*)nullptr : ws.rowc, raw, ws.status);
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

// c = M + log2 Z of every score row from the statistics of g.nchunk segments of every head
hipError_t launch_row_constants(const ScoreGeom& g, const Workspace& ws, hipStream_t st) {
  const long long n_heads = (long long)g.n_inst * g.Hkv;
  hipLaunchKernelGGL(row_constants_kernel, dim3((unsigned)n_heads, g.Rpad / 32), dim3(256), 0, st, g, ws.part, ws.rowc);
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
