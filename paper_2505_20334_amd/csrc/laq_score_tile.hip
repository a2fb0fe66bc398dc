// Scoring, one 256-key chunk per workgroup: every head size up to 256 and any number of score rows, fp32 or
// bf16, on the matrix cores (v_mfma_f32_32x32x2_f32, v_mfma_f32_32x32x16_bf16: products of the stored values,
// fp32 sums).  Used for small calls: a workgroup per chunk, and up to four for its row tiles, fill the device where the
// segments of laq_score_wave.hip would not; and for most calls of head sizes that those kernels have no variant of their own for
// (tile_wanted() has both sides' times).
//
// Two kernels: (1) per-row softmax statistics (m, z) of each chunk, (2) after folding the statistics of a
// head's chunks (by every workgroup itself when they are few, else by row_constants_kernel), the sum over
// the rows of exp2(s - c): raw scores.
//
// A wave holds 32 key rows in registers in operand layout (lane l: row l % 32, the 16-byte pieces 2t + l / 32)
// and walks the score rows in tiles of 32 that the workgroup stages in LDS, one tile ahead.  The reduction
// index of a product may run in any order as long as both operands agree, so fp32 takes the four elements
// of a piece in four instructions: lanes below 32 supply elements 8g + j, the others 8g + 4 + j.
//   (1) D = K * Q^T: lane = score row, registers = 16 keys: maximum and sum in registers.
//   (2) D = Q * K^T: lane = key, registers = 16 rows: the sum over the rows in registers.
//
// What bounds it: latency, of two launches and of load -> LDS -> products -> reduction in each (8 heads x 4096 keys, bf16: 5.3 + 6.6 us);
// fp32 pays the fp32 instruction's rate for both products, which larger calls do not (laq_score_wave.hip).
#include "laq_internal.h"
#include "laq_products.h"

namespace laq {

namespace {

constexpr int WAVES = CHUNK_ROWS / 32, THREADS = WAVES * 64;
// Row tiles of a chunk that are worked on side by side where there are too few chunks to fill the device.
constexpr int MAX_SPLIT = 4;
// Every workgroup of the second kernel folds the statistics of its head itself where that is little next to
// its keys and the workgroups are few (one launch less); otherwise row_constants_kernel does it once.
constexpr int FOLD_CHUNKS = 32, FOLD_WORKGROUPS = 512;
// bytes between rows of the staged score rows: pairs of 16-byte pieces (the second half of the last one may be
// padding, zeros) and one more, so that 128-bit reads of 16 consecutive rows fall on distinct banks
__host__ __device__ inline int q_stride(int row_bytes) { return (row_bytes + 31) / 32 * 32 + 16; }

// acc += A * B over one piece (16 bytes) per lane of either operand
__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 acc, uint16_t) { return mfma(a, b, acc); }
__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 acc, float) {
  const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
  for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[j], y[j], acc, 0, 0, 0);
  return acc;
}

// (in a scalar register: what follows from it costs none of the vector registers, of which these kernels have none to spare)
__device__ __forceinline__ int wave_number() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// The thread's number; TIGHT: by a way that keeps what is computed from it inside the loop that uses it.  (Kept in registers
// over the loop, it cost waves, or pushed keys out to memory, and waiting for those is waiting for the score rows asked for
// before them too.  64 score rows, 64 heads x 8191 keys: fp32, d = 128 201.5 -> 189.6 us, bf16, d = 96 55.1 -> 49.8, d = 256 126.5 ->
// 108; fp32, d = 256, which has two waves and registers left, 114.5 -> 117.)
template <bool TIGHT>
__device__ __forceinline__ int thread_here() {
  int t = threadIdx.x;
  if (TIGHT) asm volatile("" : "+v"(t));
  return t;
}

// What both kernels do around their products.  NP: pairs of 16-byte pieces a row may have (32 bytes each); FULL:
// it has exactly that many.
template <typename T, int NP, bool FULL> struct Chunk {
  u32x4 key[NP];           // this lane's pieces of its key row
  int np;                  // pairs of pieces a row has, the last one possibly half
  int row_bytes, stride;   // of a score row in memory / in LDS
  int lane, hf, n32, wave;
  int k0;                  // the wave's first key

  // keys first .. first + 31 of the head, for this wave
  __device__ __forceinline__ void load_keys(const ScoreGeom& g, const KvLayout& lay, const T* __restrict__ k, int first,
                                            int head, int inst) {
    const int tid = threadIdx.x;
    lane = tid & 63; hf = lane >> 5; n32 = lane & 31; wave = wave_number();
    row_bytes = FULL ? NP * 32 : g.d * (int)sizeof(T);
    stride = q_stride(row_bytes);
    np = FULL ? NP : (row_bytes + 31) / 32;
    k0 = first;
    int64_t off = (int64_t)inst * lay.inst;
    int r0 = first;
    if (lay.table && first < g.L) off = paged_block_offset(lay, inst, first, &r0);      // (a block holds whole chunks)
    const char* p = reinterpret_cast<const char*>(k + off + (int64_t)head * lay.head + (int64_t)(r0 + n32) * lay.row);
    const bool there = first + n32 < g.L;
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      key[t] = u32x4{0u, 0u, 0u, 0u};
      if (there && (FULL || (2 * t + hf) * 16 < row_bytes)) key[t] = *reinterpret_cast<const u32x4*>(p + (2 * t + hf) * 16);
    }
  }
  // score rows rt * 32 .. + 31 of the group (rows beyond R: zeros), memory -> registers -> LDS
  static constexpr int PER_THREAD = (32 * NP * 2 + THREADS - 1) / THREADS;
  __device__ __forceinline__ void fetch_rows(u32x4 (&v)[PER_THREAD], const T* __restrict__ qg, int R, int rt) const {
    const int per_row = 2 * np, tid = thread_here<(NP <= 16)>();
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int p = tid + i * THREADS, row = p / per_row, col = p - row * per_row;
      v[i] = u32x4{0u, 0u, 0u, 0u};
      if (row < 32 && rt * 32 + row < R && col * 16 < row_bytes)
        v[i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(qg) + (size_t)(rt * 32 + row) * row_bytes + col * 16);
    }
  }
  __device__ __forceinline__ void stage_rows(char* lds, const u32x4 (&v)[PER_THREAD]) const {
    const int per_row = 2 * np, tid = thread_here<(NP <= 16)>();
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int p = tid + i * THREADS, row = p / per_row, col = p - row * per_row;
      if (row < 32) *reinterpret_cast<u32x4*>(lds + row * stride + col * 16) = v[i];
    }
  }
  template <bool KEYS_AS_ROWS>
  __device__ __forceinline__ f32x16 product(const char* lds) const {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc = zero;
    const char* p = lds + n32 * stride + hf * 16;
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      if (FULL || t < np) {                              // (the same in every lane)
        const u32x4 q = *reinterpret_cast<const u32x4*>(p + t * 32);
        acc = KEYS_AS_ROWS ? mma(key[t], q, acc, T()) : mma(q, key[t], acc, T());
      }
      if (t % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (at most four operands of Q requested ahead: registers)
    }
    return acc;
  }
};

// Pass 1: part[head][chunk][row] = (m, z) of a score row over the chunk's visible keys, in log2 units.  split
// workgroups share the row tiles of a chunk.
template <typename T, int NP, bool FULL>
__global__ __launch_bounds__(THREADS, NP > 16 ? 2 : 4) void tile_stats_kernel(ScoreGeom g, WindowPos qp, KvLayout lay, int split,
                                                             const T* __restrict__ q, const T* __restrict__ k,
                                                             float2* __restrict__ part) {
  extern __shared__ __align__(16) char smem[];           // two tiles of score rows
  __shared__ float2 stat[WAVES][32];
  const int chunk = blockIdx.x / split, first = blockIdx.x - chunk * split, head = blockIdx.y, inst = blockIdx.z, tid = threadIdx.x;
  Chunk<T, NP, FULL> c;
  c.load_keys(g, lay, k, chunk * CHUNK_ROWS + wave_number() * 32, head, inst);
  const T* qg = q + ((size_t)inst * g.Hq + (size_t)head * g.G) * g.W * g.d;
  float2* out = part + (((size_t)inst * g.Hkv + head) * g.nchunk + chunk) * g.Rpad;
  const int ntile = g.Rpad / 32, tile_bytes = 32 * c.stride;
  u32x4 v[Chunk<T, NP, FULL>::PER_THREAD];
  c.fetch_rows(v, qg, g.R, first);
  c.stage_rows(smem, v);
  const bool plain = c.k0 + 31 <= g.qmin;                // seen by every row
  int turn = 0;
  for (int rt = first; rt < ntile; rt += split, turn ^= 1) {
    if (rt + split < ntile) c.fetch_rows(v, qg, g.R, rt + split);
    __syncthreads();
    f32x16 s = c.template product<true>(smem + turn * tile_bytes);
    if (!plain) {
      const int row = rt * 32 + c.n32, last = row < g.R ? last_visible_key(g, qp, row % g.W) : g.L - 1;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (c.k0 + acc_row(i, c.hf) > last) s[i] = -INFINITY;
    }
    float m = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) m = fmaxf(m, s[i]);
    m = fmaxf(m, __shfl_xor(m, 32));
    m = fmaxf(m, NEG_BIG) * g.scale2;                    // (the logit scale is positive)
    float z = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) z += __builtin_amdgcn_exp2f(fmaf(s[i], g.scale2, -m));
    z += __shfl_xor(z, 32);
    if (c.hf == 0) stat[c.wave][c.n32] = make_float2(m, z);
    if (rt + split < ntile) c.stage_rows(smem + (turn ^ 1) * tile_bytes, v);
    __syncthreads();
    if (tid < 32) {
      float M = stat[0][tid].x, Z = 0.f;
#pragma unroll
      for (int w = 1; w < WAVES; ++w) M = fmaxf(M, stat[w][tid].x);
#pragma unroll
      for (int w = 0; w < WAVES; ++w) Z = fmaf(stat[w][tid].y, __builtin_amdgcn_exp2f(stat[w][tid].x - M), Z);
      out[rt * 32 + tid] = make_float2(M, Z);
    }
  }
}

// c = M + log2 Z of the score rows rt * 32 .. + 31 from the statistics of all chunks of the head: thread
// (sub, row) takes the chunks sub, sub + WAVES * 2, ...; fixed order.
template <bool TIGHT>
__device__ __forceinline__ void fold_rows(const ScoreGeom& g, const float2* __restrict__ part, int rt, float2 (*fold)[32], float* rowc) {
  const int tid = thread_here<TIGHT>(), row = tid & 31, sub = tid >> 5;
  float M = NEG_BIG, Z = 0.f;
#pragma unroll 1
  for (int ch = sub; ch < g.nchunk; ch += WAVES * 2) {
    const float2 mz = part[(size_t)ch * g.Rpad + rt * 32 + row];
    const float Mn = fmaxf(M, mz.x);
    Z = Z * __builtin_amdgcn_exp2f(M - Mn) + mz.y * __builtin_amdgcn_exp2f(mz.x - Mn);
    M = Mn;
  }
  fold[sub][row] = make_float2(M, Z);
  __syncthreads();
  if (tid < 32) {
    M = fold[0][tid].x; Z = 0.f;
#pragma unroll 4
    for (int w = 1; w < WAVES * 2; ++w) M = fmaxf(M, fold[w][tid].x);
#pragma unroll 4
    for (int w = 0; w < WAVES * 2; ++w) Z = fmaf(fold[w][tid].y, __builtin_amdgcn_exp2f(fold[w][tid].x - M), Z);
    rowc[tid] = rt * 32 + tid < g.R ? M + __builtin_amdgcn_logf(Z) : 1.0e30f;      // (rows beyond R: any finite number)
  }
  __syncthreads();                                       // (`fold` may be written again)
}

// Pass 2: raw[j] = sum over the score rows of exp2(s - c[row]).  The workgroup has CHUNK_ROWS / split keys; wave
// (row group rg, key tile) takes the row tiles rg, rg + split, ...  rowc_all: the heads' row constants, or
// null: folded here.
template <typename T, int NP, bool FULL>
__global__ __launch_bounds__(THREADS, NP > 16 ? 2 : 4) void tile_score_kernel(ScoreGeom g, WindowPos qp, KvLayout lay, int split,
                                                             const T* __restrict__ q, const T* __restrict__ k,
                                                             const float2* __restrict__ part, const float* __restrict__ rowc_all,
                                                             float* __restrict__ raw, int* __restrict__ status) {
  extern __shared__ __align__(16) char smem[];           // two tiles of score rows per row group
  __shared__ __align__(16) float rowc[2][MAX_SPLIT][32];
  __shared__ __align__(16) int last[2][MAX_SPLIT][32];   // last key the rows see
  __shared__ float2 fold[WAVES * 2][32];
  __shared__ float sums[WAVES][32];
  const int head = blockIdx.y, inst = blockIdx.z, tid = threadIdx.x;
  const size_t hg = (size_t)inst * g.Hkv + head;
  if (blockIdx.x == 0 && hg == 0 && tid == 0) *status = 0;    // (these kernels have no wait to give up)
  const int key_waves = WAVES / split, rg = wave_number() / key_waves, kw = wave_number() - rg * key_waves;
  Chunk<T, NP, FULL> c;
  c.load_keys(g, lay, k, (int)blockIdx.x * key_waves * 32 + kw * 32, head, inst);
  const T* qg = q + ((size_t)inst * g.Hq + (size_t)head * g.G) * g.W * g.d;
  const int ntile = g.Rpad / 32, tile_bytes = 32 * c.stride;
  u32x4 v[Chunk<T, NP, FULL>::PER_THREAD];
  auto constants = [&](int turn, int rt) {
    const int tid = thread_here<(NP <= 16)>();
#pragma unroll 1
    for (int i = 0; i < split && rt + i < ntile; ++i) {
      if (tid < 32) {
        const int row = (rt + i) * 32 + tid;
        last[turn][i][tid] = row < g.R ? last_visible_key(g, qp, row % g.W) : -1;
      }
      if (rowc_all == nullptr) fold_rows<(NP <= 16)>(g, part + hg * g.nchunk * g.Rpad, rt + i, fold, rowc[turn][i]);
      else if (tid < 32) rowc[turn][i][tid] = rowc_all[hg * g.Rpad + (rt + i) * 32 + tid];
    }
  };
  auto stage = [&](int turn, int rt) {                   // (the first of the next tiles is in v)
    c.stage_rows(smem + turn * split * tile_bytes, v);
#pragma unroll 1
    for (int i = 1; i < split; ++i) {
      c.fetch_rows(v, qg, g.R, rt + i);
      c.stage_rows(smem + (turn * split + i) * tile_bytes, v);
    }
    constants(turn, rt);
  };
  c.fetch_rows(v, qg, g.R, 0);
  stage(0, 0);
  const int key = c.k0 + c.n32;
  const bool seen = c.k0 + 31 <= g.qmin;
  float sum = 0.f;
  int turn = 0;
  for (int rt = 0; rt < ntile; rt += split, turn ^= 1) {
    if (rt + split < ntile) c.fetch_rows(v, qg, g.R, rt + split);
    __syncthreads();
    if (rt + rg < ntile) {
      f32x16 s = c.template product<false>(smem + (turn * split + rg) * tile_bytes);
      // rows beyond R see no key: their product with one that is not finite would be a NaN
      if (!seen || (rt + rg + 1) * 32 > g.R) {
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const i32x4 lv = *reinterpret_cast<const i32x4*>(last[turn][rg] + 8 * gq + 4 * c.hf);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (key > lv[j]) s[4 * gq + j] = -INFINITY;
        }
      }
      const float* rc = rowc[turn][rg];
      float tile_sum = 0.f;
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const f32x4 cc = *reinterpret_cast<const f32x4*>(rc + 8 * gq + 4 * c.hf);
#pragma unroll
        for (int j = 0; j < 4; ++j) tile_sum += __builtin_amdgcn_exp2f(fmaf(s[4 * gq + j], g.scale2, -cc[j]));
      }
      // (over both lanes' rows: one lane's may all pad, or not see the key)
      const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(tile_sum), __float_as_uint(tile_sum), false, false);
      const float both = __uint_as_float(halves[0]) + __uint_as_float(halves[1]);
      if (__builtin_expect(__any(both < TINY && key < g.L), 0)) {      // (what the exponential lost is added)
#pragma unroll 1
        for (int i = 0; i < 16; ++i) {                   // (few instructions: what follows them is fetched sooner)
          const float x = fmaf(s[0], g.scale2, -rc[acc_row(i, c.hf)]);
          if (x < -126.f) tile_sum = fmaf(__builtin_amdgcn_exp2f(x + 64.f), 0x1p-64f, tile_sum);
          s = __builtin_shufflevector(s, s, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 0);
        }
      }
      sum += tile_sum;
    }
    if (rt + split < ntile) stage(turn ^ 1, rt + split);
  }
  sum += __shfl_xor(sum, 32);
  if (split > 1) {                                       // the row groups' sums, in their order
    if (c.hf == 0) sums[c.wave][c.n32] = sum;
    __syncthreads();
    if (rg != 0) return;
    for (int i = 1; i < split; ++i) sum += sums[kw + i * key_waves][c.n32];
  }
  if (c.hf == 0 && key < g.L) raw[hg * g.L + key] = sum;
}

constexpr int MAX_LDS = 128 << 10;                       // of the staged score rows

template <typename T, int NP, bool FULL>
hipError_t launch_tile(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, const T* q, const T* k, float* raw,
                       const Workspace& ws, hipStream_t st) {
  const int bytes = 2 * 32 * q_stride(g.d * (int)sizeof(T)), ntile = g.Rpad / 32;
  const long long units = (long long)g.nchunk * g.Hkv * g.n_inst;
  // As far as each of the 256 compute units still gets one workgroup at most: more of them read the keys and the score
  // rows again for nothing (fp32, d = 128, 64 score rows: 192 chunks took 43.2 us in 384 workgroups, 256 take
  // 37.3 in 256 and 44.0 in 512).
  int split = 1;
  while (split < MAX_SPLIT && 2 * split <= ntile && units * split * 2 <= 256) split *= 2;
  hipLaunchKernelGGL((tile_stats_kernel<T, NP, FULL>), dim3(g.nchunk * split, g.Hkv, g.n_inst), dim3(THREADS), bytes, st, g, qp, lay, split, q,
                     k, ws.part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool fold = g.nchunk <= FOLD_CHUNKS && units <= FOLD_WORKGROUPS;
  if (!fold && (e = launch_row_constants(g, ws, ws.rowc, st)) != hipSuccess) return e;
  if (split * bytes > MAX_LDS) split = 1;
  const int keys = CHUNK_ROWS / split;
  hipLaunchKernelGGL((tile_score_kernel<T, NP, FULL>), dim3((g.L + keys - 1) / keys, g.Hkv, g.n_inst), dim3(THREADS), split * bytes, st, g, qp, lay,
                     split, q, k, ws.part, fold ? (const float*)nullptr : ws.rowc, raw, ws.status);
  return hipGetLastError();
}

template <typename T, int NP, bool FULL> hipError_t init_tile() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tile_stats_kernel<T, NP, FULL>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, MAX_LDS);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&tile_score_kernel<T, NP, FULL>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, MAX_LDS);
}

}  // namespace

hipError_t score_tile_init() {
  hipError_t e;
  if ((e = init_tile<uint16_t, 4, true>()) != hipSuccess || (e = init_tile<uint16_t, 8, true>()) != hipSuccess ||
      (e = init_tile<uint16_t, 8, false>()) != hipSuccess || (e = init_tile<uint16_t, 16, true>()) != hipSuccess ||
      (e = init_tile<uint16_t, 16, false>()) != hipSuccess || (e = init_tile<float, 8, true>()) != hipSuccess ||
      (e = init_tile<float, 16, true>()) != hipSuccess || (e = init_tile<float, 16, false>()) != hipSuccess ||
      (e = init_tile<float, 32, true>()) != hipSuccess)
    return e;
  return init_tile<float, 32, false>();
}

hipError_t launch_score_tile(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, const void* q, const void* k,
                             float* raw, const Workspace& ws, hipStream_t st) {
  if (dtype == LAQ_F32) {
    const float *qq = static_cast<const float*>(q), *kk = static_cast<const float*>(k);
    if (g.d == 64) return launch_tile<float, 8, true>(g, qp, lay, qq, kk, raw, ws, st);
    if (g.d == 128) return launch_tile<float, 16, true>(g, qp, lay, qq, kk, raw, ws, st);
    if (g.d == 256) return launch_tile<float, 32, true>(g, qp, lay, qq, kk, raw, ws, st);
    if (g.d < 128) return launch_tile<float, 16, false>(g, qp, lay, qq, kk, raw, ws, st);
    return launch_tile<float, 32, false>(g, qp, lay, qq, kk, raw, ws, st);
  }
  const uint16_t *qq = static_cast<const uint16_t*>(q), *kk = static_cast<const uint16_t*>(k);
  if (g.d == 64) return launch_tile<uint16_t, 4, true>(g, qp, lay, qq, kk, raw, ws, st);
  if (g.d == 128) return launch_tile<uint16_t, 8, true>(g, qp, lay, qq, kk, raw, ws, st);
  if (g.d == 256) return launch_tile<uint16_t, 16, true>(g, qp, lay, qq, kk, raw, ws, st);
  if (g.d < 128) return launch_tile<uint16_t, 8, false>(g, qp, lay, qq, kk, raw, ws, st);
  return launch_tile<uint16_t, 16, false>(g, qp, lay, qq, kk, raw, ws, st);
}

}  // namespace laq
