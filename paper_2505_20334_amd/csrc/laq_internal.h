// Internal declarations shared by the HIP translation units of the LAQ library.
// Not part of the public boundary (that is include/laq.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "laq.h"

namespace laq {

// The one-chunk scoring kernels give every workgroup CHUNK_ROWS consecutive key rows of one KV head; a head is
// covered by nchunk = ceil(L / CHUNK_ROWS) chunks.  The other two-pass kernels cut a head into at most as many segments.
constexpr int CHUNK_ROWS = 256;
constexpr int MAX_POOL = 63;
constexpr int MAX_INST_PER_LAUNCH = 256;   // size of the per-instance tables passed as kernel arguments

constexpr int MAX_QPOS = 512;              // explicit query positions a call may carry
// The single-read scoring kernel: key rows per workgroup, and the number of its workgroups on the
// device at once that the exchange memory of a workspace is sized for.
constexpr int FUSED_ROWS = 512;
constexpr int FUSED_MAX_RESIDENT = 1024;
// Whether scoring may take the single-read kernel at all (single_read_wanted() tells where it is the faster one).
constexpr bool SINGLE_READ_ENABLED = true;

struct ScoreGeom {
  int n_inst, Hq, Hkv, d, L, W;
  int G, R;
  int keep;      // trailing keys always retained
  int P;         // L - keep: the prefix that is ranked and pooled
  int Rpad;      // R rounded up to a multiple of 32
  int nchunk;    // ceil(L / CHUNK_ROWS)
  int pos0;      // trailing-window layout: query w sees keys j <= pos0 + w (pos0 = L - W)
  int explicit_pos;   // 1: positions come from the QueryPos table instead
  int qmin;      // smallest last-visible key over the W queries: keys up to here need no mask
  float scale2;  // scale * log2(e): logits are kept in base-2 units
};

// Last key each window query sees, where positions are explicit (already clamped to L-1); passed by value
// to the kernels.  Launch arguments cost host time per byte, so only short windows travel in them; a
// longer one's table (up to MAX_QPOS entries) is written to the workspace first.
constexpr int WINDOW_INLINE = 32;
struct WindowPos {
  int32_t last[WINDOW_INLINE];
  const int32_t* table;
};
__device__ __forceinline__ int last_visible_key(const ScoreGeom& g, const WindowPos& qp, int w) {
  if (!g.explicit_pos) return g.pos0 + w;
  return g.W <= WINDOW_INLINE ? qp.last[w] : qp.table[w];
}
struct QueryPos {                          // host side
  int32_t last[MAX_QPOS];
};

// Workspace carving: [partials | row constants | raw scores]
//   part:  float2 (m, z) per (instance, KV head, chunk, padded row): softmax statistics of a chunk or segment
//   rowc:  float c = M + log2(Z) per (instance, KV head, padded row): the one-chunk kernels with many chunks
//   raw:   float per (instance, KV head, key): unpooled scores in front of a pooling or selecting kernel; the single-read
//          kernel with the max pool keeps the edge records of its workgroups' boundaries here instead
//   pooled: float per (instance, KV head, key): the hand-over plane between scoring and selection
//          when laq_evict is called without a scores buffer
struct Workspace {
  float2* part;
  float* rowc;
  float* raw;
  float* pooled;
  void* fused;      // exchange memory of the single-read kernel (fused_sync_bytes)
  int32_t* window;  // position table of a window longer than WINDOW_INLINE (MAX_QPOS entries)
  int* status;      // != 0 after a call whose single-read kernel gave up a wait (results invalid)
  int* started;     // counters of the single-read kernel's workgroups
};

size_t workspace_bytes(const ScoreGeom& g);
Workspace carve_workspace(const ScoreGeom& g, void* ws);

// Where the rows of k and v lie: element strides between instances and KV heads, and between
// consecutive key rows (row_bytes is the latter in bytes).  dense = [n_inst, Hkv, L, d].
struct KvLayout {
  int64_t inst, head, row;
  int32_t row_bytes;
  int32_t dense;
  // paged cache (table != nullptr): key row j of instance i is row j % block_rows of block
  // table[i * blocks_per_inst + j / block_rows]; blocks lie `block` elements apart, head / row are
  // the strides inside a block, inst is not used
  const int32_t* table;
  int32_t blocks_per_inst;
  int32_t block_rows;
  int64_t block;
};

// Where the packed outputs of an instance lie, for select / compact (passed by value as a kernel argument):
// a table, or, where all instances keep the same number of rows, its arithmetic.
struct InstTable {
  int32_t bk[MAX_INST_PER_LAUNCH];      // rows kept per KV head
  int64_t row0[MAX_INST_PER_LAUNCH];    // first packed output row (sum of Hkv * Bk of earlier instances)
  __device__ int rows(int i) const { return bk[i]; }
  __device__ int64_t first(int i) const { return row0[i]; }
};
struct UniformInst {
  int32_t bk;
  int64_t row0, per_inst;
  __device__ int rows(int) const { return bk; }
  __device__ int64_t first(int i) const { return row0 + i * per_inst; }
};
// The gather's own table: its grid covers exactly the rows of every instance, so a workgroup finds
// its instance by the first workgroup of each (blk0 ascending, blk0[n] = all workgroups).
struct CompactTable {
  int32_t bk[MAX_INST_PER_LAUNCH];
  int64_t row0[MAX_INST_PER_LAUNCH];
  int32_t blk0[MAX_INST_PER_LAUNCH + 1];
};
// What the selection kernel does besides: it pools the raw scores it is given (max or mean over half positions to either
// side) and writes the pooled ones; and, where it finishes a small eviction in one launch, it gathers the rows it has
// selected.
struct PoolArgs {
  float* pooled;
  int32_t half, avg;
};
struct FinishArgs : PoolArgs {
  const char *k, *v;
  char *k_out, *v_out;
  int64_t inst_bytes, head_bytes;
  int32_t row_bytes, src_row_bytes, elem_bytes;
  KvLayout lay;
};
constexpr int SELECT_POOL_MAX_HALF = 8;         // widest pooling it does (laq_pool.h): two quads of scores beside a lane's own on either side
constexpr int SELECT_POOL_MAX_KEYS = 32 * 1024; // longest prefix it pools
constexpr int SELECT_MANY_HEADS = 768;          // heads of a launch from which on several workgroups share a compute unit,
constexpr int SELECT_POOL_MANY_KEYS = 8 * 1024; // and the longest prefix it pools there (a longer one leaves no registers for it)
constexpr int FINISH_MAX_KEYS = 16 * 1024;      // longest prefix of a finishing launch
// How many scores the rows of a launch start behind a 16-byte boundary, at most.  Only where they do does a variant of the
// selection kernel hold fewer keys than its registers: 32768 keys of aligned rows taken for 32771 went to the kernel that holds
// none (8, 256, 2048 heads: 43.6, 51.0 and 366 us against 15.6, 17.1 and 116 for 32764), 2048 of them to the next
// larger one (2048 heads: 27.8 us against 10.5 for 2044).
inline int row_shift(const float* scores, int L) {
  return L % 4 == 0 ? (int)(reinterpret_cast<uintptr_t>(scores) / sizeof(float) % 4) : 3;
}

// Pooled score at prefix position pos, the one arithmetic every pooling site uses: the
// maximum over the part of the window inside [0, P), or (avg) the fp32 sum over it in
// ascending position divided by the kernel size 2*half+1 (zeros outside the prefix).
__device__ __forceinline__ float pool_window(const float* __restrict__ s, int pos, int P, int half, bool avg) {
  if (half == 0) return s[pos];
  const int lo = max(pos - half, 0), hi = min(pos + half, P - 1);
  if (avg) {
    float acc = 0.f;
    for (int i = lo; i <= hi; ++i) acc += s[i];
    return acc / (float)(2 * half + 1);
  }
  float v = s[pos];
  for (int i = lo; i <= hi; ++i) v = fmaxf(v, s[i]);
  return v;
}

#ifdef __HIPCC__
// Paged caches: element offset, from the pool's start, of the block that holds key row j of an
// instance, and the row's number inside that block.
__device__ __forceinline__ int64_t paged_block_offset(const KvLayout& lay, int inst, int j, int* row_in_block) {
  const int b = j / lay.block_rows;
  *row_in_block = j - b * lay.block_rows;
  return (int64_t)lay.table[(size_t)inst * lay.blocks_per_inst + b] * lay.block;
}
// The same for a key row that all lanes of a wave share (no kernel writes the table): as constant memory, through the scalar cache.  A
// vector load returns behind every key load issued before it, so that a tile's loads waited for the tile in front of it: laq_evict,
// 112 rows, 28 instances x 4 heads x 20123 keys in blocks of 256, 289 us, so 284.
__device__ __forceinline__ int64_t paged_tile_offset(const KvLayout& lay, int inst, int j, int* row_in_block) {
  typedef __attribute__((address_space(4))) const int32_t* ConstTable;
  const int b = j / lay.block_rows;
  *row_in_block = j - b * lay.block_rows;
  return (int64_t)((ConstTable)(unsigned long long)lay.table)[(size_t)inst * lay.blocks_per_inst + b] * lay.block;
}
#endif

// Two packed index lists side by side, for up to MAX_PAIR_PER_LAUNCH instances.
constexpr int MAX_PAIR_PER_LAUNCH = 128;
struct PairTable {
  int32_t bk_a[MAX_PAIR_PER_LAUNCH], bk_b[MAX_PAIR_PER_LAUNCH];       // row lengths
  int64_t row_a[MAX_PAIR_PER_LAUNCH], row_b[MAX_PAIR_PER_LAUNCH];     // first packed row of the instance
};

// The rows kept per KV head if that is the same number for instances i0 .. i0+n-1, else 0.
inline int uniform_rows(int L, const int32_t* budget, int i0, int n) {
  const int bk = budget[i0] < L ? budget[i0] : L;
  for (int i = 1; i < n; ++i)
    if ((budget[i0 + i] < L ? budget[i0 + i] : L) != bk) return 0;
  return bk;
}

// launchers (each returns hipGetLastError() after its last launch); `raw` receives unpooled scores
hipError_t launch_score_tile(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, const void* q,
                             const void* k, float* raw, const Workspace& ws, hipStream_t st);
hipError_t score_tile_init();
bool score_wave_supported(const ScoreGeom& g, int dtype);
bool score_wave_own_size(const ScoreGeom& g, int dtype);      // a head size that these kernels have a variant of its own for
hipError_t launch_score_wave(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, const void* q,
                             const void* k, float* raw, const Workspace& ws, hipStream_t st);
hipError_t score_wave_init();
hipError_t launch_row_constants(const ScoreGeom& g, const Workspace& ws, float* rowc, hipStream_t st);
// kernel attributes and residency of the single-read scoring kernel on device `dev`, which must be
// the current device; idempotent
hipError_t score_fused_init(int dev);
size_t fused_sync_bytes(const ScoreGeom& g);
bool score_fused_supported(const ScoreGeom& g, const KvLayout& lay, int dtype);
hipError_t score_fused_applies(const ScoreGeom& g, const KvLayout& lay, int dtype, bool* yes);
// 0: where the rule for its launches (laq_team.h) does not hold; else the number of counters that its teams draw from (st null: on a
// stream of normal priority that may use all compute units)
int score_fused_counters(const ScoreGeom& g, const KvLayout& lay, int dtype, const hipStream_t* st);
// single-read scoring (K streamed once); *done = false: not launched, take the two-pass kernels
hipError_t launch_score_fused(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int pool, const void* q,
                              const void* k, float* scores, const Workspace& ws, hipStream_t st, bool* done);
// pooled scores of the prefix keys within `half` of a boundary between two chunks of chunk_rows keys,
// from the chunks' edge records
hipError_t launch_pool_boundaries(const ScoreGeom& g, int half, int nchunk, int chunk_rows, const float* edge,
                                  float* scores, hipStream_t st);
hipError_t launch_pool(const ScoreGeom& g, int pool, bool avg, const float* raw, float* pooled, hipStream_t st);
hipError_t launch_select(int n_inst, int inst0, int Hkv, int L, int keep, int pool, bool avg, const float* scores,
                         const InstTable& tab, int32_t* idx, hipStream_t st);
hipError_t launch_select(int n_inst, int inst0, int Hkv, int L, int keep, int pool, bool avg, const float* scores,
                         const UniformInst& tab, int32_t* idx, hipStream_t st);
// the same from raw scores, pooled on the way
hipError_t launch_select_pooling(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const InstTable& tab, int32_t* idx,
                                 const PoolArgs& pool, hipStream_t st);
hipError_t launch_select_pooling(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const UniformInst& tab, int32_t* idx,
                                 const PoolArgs& pool, hipStream_t st);
hipError_t launch_finish(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const InstTable& tab, int32_t* idx,
                         const FinishArgs& fin, hipStream_t st);
hipError_t launch_finish(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const UniformInst& tab, int32_t* idx,
                         const FinishArgs& fin, hipStream_t st);
// all of a short head in one workgroup: scores (pooled by fin.half / fin.avg into fin.pooled), with HEAD_LIST the selection too, with HEAD_ROWS that and the
// gather
enum HeadSteps { HEAD_SCORES, HEAD_LIST, HEAD_ROWS };
bool head_supported(const ScoreGeom& g, int dtype);
bool head_keeps(const ScoreGeom& g, int dtype);   // its products and exponentials are made once: the registers hold those of all score rows
hipError_t head_init();
hipError_t launch_head(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, int steps, const void* q, const void* k, int n_inst,
                       int inst0, const InstTable& tab, int32_t* idx, const FinishArgs& fin, int* status, hipStream_t st);
hipError_t launch_head(const ScoreGeom& g, const WindowPos& qp, const KvLayout& lay, int dtype, int steps, const void* q, const void* k, int n_inst,
                       int inst0, const UniformInst& tab, int32_t* idx, const FinishArgs& fin, int* status, hipStream_t st);
hipError_t launch_sink_recent(int n_inst, int Hkv, int L, int n_sink, const InstTable& tab, int32_t* idx,
                              hipStream_t st);
hipError_t launch_recall(int n_inst, int inst0, int Hkv, const PairTable& tab, const int32_t* idx_pred,
                         const int32_t* idx_gold, int32_t* overlap, float* recall, hipStream_t st);
int decode_head_batch(int Hq, int Hkv, int dtype);   // query heads of a KV head that one decode workgroup serves
int decode_part_rows(int n, int L, int Hq, int Hkv, int dtype, const int32_t* budget);   // the limit of the parts' rows, before they are evened out
size_t decode_partial_bytes(int n, int L, int Hq, int Hkv, int d, int dtype, const int32_t* budget);
hipError_t launch_decode(int n_inst, int L, int Hq, int Hkv, int d, int dtype, float scale2, int rows_per_part, const int32_t* budget,
                         const void* q, const void* kc, const void* vc, float* out, void* ws, hipStream_t st);
hipError_t launch_qcache_store(long long rows, int W, int t, int row_bytes, const void* q_step, void* q_cache,
                               hipStream_t st);
constexpr int COMPACT_THREADS = 256;      // one 16-byte piece of an output row per thread
hipError_t launch_compact(int n_inst, int inst0, int Hkv, int L, int row_bytes, const KvLayout& lay,
                          const void* k, const void* v, const int32_t* idx, const CompactTable& tab, void* k_out,
                          void* v_out, hipStream_t st);
hipError_t launch_compact(int n_inst, int inst0, int Hkv, int L, int row_bytes, const KvLayout& lay,
                          const void* k, const void* v, const int32_t* idx, const UniformInst& tab, void* k_out,
                          void* v_out, hipStream_t st);

}  // namespace laq
