// C ABI of the LAQ re-eviction library (declared in include/laq.h): argument checks,
// geometry, kernel dispatch.  No device memory is allocated here.
#include <math.h>
#include <string.h>

#include <atomic>

#include "laq_internal.h"

namespace laq {

static bool pool_ok(int pool) { return pool >= 1 && pool <= MAX_POOL && (pool % 2) == 1; }
static bool pool_avg(const laq_shape* s) { return s->pool_mode == LAQ_POOL_AVG; }

// Geometry of a call.  Returns LAQ_OK, LAQ_ERR_INVALID or LAQ_ERR_UNSUPPORTED; fills the query
// position table (qp may be null for calls that do not score) when positions are explicit.
static int make_geom(const laq_shape* s, ScoreGeom* g, QueryPos* qp = nullptr) {
  if (!s) return LAQ_ERR_INVALID;
  if (s->n_inst < 1 || s->Hq < 1 || s->Hkv < 1 || s->d < 8 || s->d > 256 || (s->d % 8) != 0) return LAQ_ERR_INVALID;
  if (s->L < 1 || s->W < 1 || (s->Hq % s->Hkv) != 0) return LAQ_ERR_INVALID;
  if ((!s->q_pos || s->keep < 0) && s->W > s->L) return LAQ_ERR_INVALID;   // trailing-window defaults need W <= L
  if (s->keep > s->L) return LAQ_ERR_INVALID;
  if (s->dtype != LAQ_F32 && s->dtype != LAQ_BF16) return LAQ_ERR_INVALID;
  if (s->pool_mode != LAQ_POOL_MAX && s->pool_mode != LAQ_POOL_AVG) return LAQ_ERR_INVALID;
  if (!(s->scale == s->scale) || isinf(s->scale)) return LAQ_ERR_INVALID;
  g->n_inst = s->n_inst; g->Hq = s->Hq; g->Hkv = s->Hkv; g->d = s->d; g->L = s->L; g->W = s->W;
  g->G = s->Hq / s->Hkv;
  g->R = g->G * s->W;
  g->keep = s->keep < 0 ? s->W : s->keep;
  g->P = s->L - g->keep;
  g->pos0 = s->L - s->W;
  g->explicit_pos = s->q_pos ? 1 : 0;
  g->qmin = g->pos0;
  if (s->q_pos) {
    if (s->W > MAX_QPOS) return LAQ_ERR_UNSUPPORTED;
    int qmin = s->L - 1;
    for (int w = 0; w < s->W; ++w) {
      if (s->q_pos[w] < 0) return LAQ_ERR_INVALID;
      const int last = s->q_pos[w] < s->L - 1 ? s->q_pos[w] : s->L - 1;
      if (qp) qp->last[w] = last;
      if (last < qmin) qmin = last;
    }
    g->qmin = qmin;
  }
  g->Rpad = (g->R + 31) / 32 * 32;
  g->nchunk = (s->L + CHUNK_ROWS - 1) / CHUNK_ROWS;
  const float sc = s->scale > 0.f ? s->scale : 1.0f / sqrtf((float)s->d);
  g->scale2 = sc * 1.44269504088896340736f;
  return LAQ_OK;
}

// Layout of k / v from the shape's strides (all zero: dense).  LAQ_ERR_INVALID on strides that are
// not 16-byte multiples, overlap a row, or mix zero and non-zero.
static int make_layout(const laq_shape* s, const ScoreGeom& g, KvLayout* lay) {
  const int eb = s->dtype == LAQ_F32 ? 4 : 2;
  const int64_t si = s->kv_stride_inst, sh = s->kv_stride_head, sr = s->kv_stride_row;
  lay->table = nullptr;
  lay->blocks_per_inst = 0;
  lay->block_rows = 0;
  lay->block = 0;
  if (s->block_table) {
    // a pool of blocks: strides inside a block, and between blocks
    const int64_t br = s->block_rows, sb = s->kv_stride_block;
    if (br < 256 || br % 256 || br > (1 << 24)) return LAQ_ERR_INVALID;
    if ((sh == 0) != (sr == 0)) return LAQ_ERR_INVALID;
    lay->row = sr ? sr : g.d;
    lay->head = sh ? sh : br * g.d;
    if (lay->row < g.d || lay->head < 1 || sb < 1 || (lay->row * eb) % 16 || (lay->head * eb) % 16 || (sb * eb) % 16)
      return LAQ_ERR_INVALID;
    if (lay->row * eb > 0x7fffffffLL) return LAQ_ERR_INVALID;
    lay->inst = 0;
    lay->dense = 0;
    lay->table = s->block_table;
    lay->blocks_per_inst = (int32_t)((g.L + br - 1) / br);
    lay->block_rows = (int32_t)br;
    lay->block = sb;
    lay->row_bytes = (int32_t)(lay->row * eb);
    return LAQ_OK;
  }
  if (s->block_rows != 0 || s->kv_stride_block != 0) return LAQ_ERR_INVALID;
  if (si == 0 && sh == 0 && sr == 0) {
    lay->row = g.d;
    lay->head = (int64_t)g.L * g.d;
    lay->inst = (int64_t)g.Hkv * g.L * g.d;
    lay->dense = 1;
  } else {
    if (sr < g.d || sh < 1 || si < 1 || (sr * eb) % 16 || (sh * eb) % 16 || (si * eb) % 16) return LAQ_ERR_INVALID;
    if (sr * eb > 0x7fffffffLL) return LAQ_ERR_INVALID;
    lay->row = sr;
    lay->head = sh;
    lay->inst = si;
    lay->dense = (sr == g.d && sh == (int64_t)g.L * g.d && si == (int64_t)g.Hkv * g.L * g.d) ? 1 : 0;
  }
  lay->row_bytes = (int32_t)(lay->row * eb);
  return LAQ_OK;
}

static size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t workspace_bytes(const ScoreGeom& g) {
  const size_t heads = (size_t)g.n_inst * g.Hkv;
  return round256(heads * g.nchunk * g.Rpad * sizeof(float2)) + round256(heads * g.Rpad * sizeof(float)) +
         2 * round256(heads * g.L * sizeof(float)) + round256(fused_sync_bytes(g)) + 256;
}

Workspace carve_workspace(const ScoreGeom& g, void* ws) {
  const size_t heads = (size_t)g.n_inst * g.Hkv;
  char* base = static_cast<char*>(ws);
  Workspace w;
  w.part = reinterpret_cast<float2*>(base);
  base += round256(heads * g.nchunk * g.Rpad * sizeof(float2));
  w.rowc = reinterpret_cast<float*>(base);
  base += round256(heads * g.Rpad * sizeof(float));
  w.raw = reinterpret_cast<float*>(base);
  base += round256(heads * g.L * sizeof(float));
  w.pooled = reinterpret_cast<float*>(base);
  base += round256(heads * g.L * sizeof(float));
  w.fused = base;
  base += round256(fused_sync_bytes(g));
  w.window = reinterpret_cast<int32_t*>(base - MAX_QPOS * sizeof(int32_t));   // (the end of that area, see make_plan() of the single-read kernel)
  w.status = reinterpret_cast<int*>(base) + 8;
  w.started = reinterpret_cast<int*>(base) + 32;     // (not in the cache line of the status)
  return w;
}

// The positions of a long explicit window, from launch arguments to the workspace.
__global__ void window_table_kernel(QueryPos qp, int W, int32_t* table) {
  for (int w = threadIdx.x; w < W; w += blockDim.x) table[w] = qp.last[w];
}

// What the scoring kernels get of the window's positions.
static hipError_t window_positions(const ScoreGeom& g, const QueryPos& qp, const Workspace& w, hipStream_t st, WindowPos* out) {
  memset(out, 0, sizeof *out);
  if (!g.explicit_pos) return hipSuccess;
  if (g.W <= WINDOW_INLINE) {
    memcpy(out->last, qp.last, g.W * sizeof(int32_t));
    return hipSuccess;
  }
  out->table = w.window;
  hipLaunchKernelGGL(window_table_kernel, dim3(1), dim3(256), 0, st, qp, g.W, w.window);
  return hipGetLastError();
}

// Fill the per-instance table for instances [i0, i0+n) and return the largest Bk among them.
static int fill_table(int Hkv, int L, const int32_t* budget, int i0, int n, int64_t row_base,
                      InstTable* tab, int64_t* rows_after) {
  int bk_max = 0;
  int64_t row = row_base;
  for (int i = 0; i < n; ++i) {
    const int bk = budget[i0 + i] < L ? budget[i0 + i] : L;
    tab->bk[i] = bk;
    tab->row0[i] = row;
    row += (int64_t)Hkv * bk;
    if (bk > bk_max) bk_max = bk;
  }
  *rows_after = row;
  return bk_max;
}

// The same for the gather, whose grid covers the rows of every instance exactly.
static void fill_compact_table(int Hkv, int L, int pieces_per_row, const int32_t* budget, int i0, int n,
                               int64_t row_base, CompactTable* tab, int64_t* rows_after) {
  int64_t row = row_base, blk = 0;
  for (int i = 0; i < n; ++i) {
    const int bk = budget[i0 + i] < L ? budget[i0 + i] : L;
    tab->bk[i] = bk;
    tab->row0[i] = row;
    tab->blk0[i] = (int32_t)blk;
    row += (int64_t)Hkv * bk;
    blk += ((int64_t)Hkv * bk * pieces_per_row + COMPACT_THREADS - 1) / COMPACT_THREADS;
  }
  tab->blk0[n] = (int32_t)blk;
  *rows_after = row;
}

static bool budgets_ok(const laq_shape* s, const ScoreGeom& g, const int32_t* budget) {
  if (!budget) return false;
  for (int i = 0; i < s->n_inst; ++i)
    if (budget[i] < g.keep || budget[i] < 1) return false;
  return true;
}

// ---- per-device set-up ---------------------------------------------------------------------
// Kernel attributes and residency of the scoring kernels on the current device, and the address of
// the library's own scratch array there.  `scratch` is the workspace of laq_evict_static: in host
// code its name is only a handle, and every device holds its own copy at its own address, which is
// looked up once per device (with that device current) and used from then on.
static __device__ __align__(256) unsigned char scratch[LAQ_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static std::atomic<void*> scratch_of[MAX_DEVICES];

static int init_current_device(int* dev_out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return LAQ_ERR_DEVICE;
  if (dev_out) *dev_out = dev;
  if (scratch_of[dev].load(std::memory_order_acquire)) return LAQ_OK;
  if (score_fused_init(dev) != hipSuccess || score_tile_init() != hipSuccess || score_wave_init() != hipSuccess || head_init() != hipSuccess) return LAQ_ERR_DEVICE;
  void* ptr = nullptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LAQ_ERR_DEVICE;
  scratch_of[dev].store(ptr, std::memory_order_release);
  return LAQ_OK;
}

// bf16 and one of the head sizes 64 and 128, with byte offsets inside a head (or block) that fit 31 bits: what laq_score_kernel
// tells apart from the other shapes.
static bool usual_shape(const ScoreGeom& g, const KvLayout& lay, int dtype) {
  return dtype == LAQ_BF16 && (g.d == 128 || g.d == 64) && g.W <= MAX_QPOS && g.n_inst * (long long)g.Hkv <= 0x7fffffff &&
         ((long long)(lay.table ? lay.block_rows : g.L) + CHUNK_ROWS) * lay.row_bytes < 0x7fffffffLL;
}

// The single-read kernel's serial start costs more than the launches of the two passes; from some size of the call on it is the
// faster one (21-27 % at 1 GiB and more).
// laq_evict, bf16, the two passes : this one, us:
//   64 rows  36 MiB 1100 to 5000 keys 1.06-1.09, 2 x 8 heads x 8200 35.4 : 36.5;  43 MiB 3100 keys 41.0 : 35.7, 1100 keys 49.8 : 41.5;  49 to 70 MiB
//            1.08-1.29;  94 to 120 MiB 1.12-1.31
//   32 rows  36 MiB 1300 to 5000 keys 1.04-1.13, 8200 keys 34.6 : 34.8;  48 to 54 MiB 1300 to 30011 keys 1.02-1.22;  62 to 70 MiB .98 (8200 keys), 1.00-1.24;
//            94 to 120 MiB 1.06-1.34;  1100 keys (a team's second workgroup nearly empty) 37 MiB .88, 64 MiB .99, 97 MiB 1.05
// Teams of one counter (laq_team.h) from 128 MiB on.  Captured calls take the same kernel, so that a replay gives the eager bits; a graph of one call, the
// two passes : this one: 8 heads x 24000 46.9 : 47.9, x 30011 53.1 : 51.1, 200 x 1100 59.1 : 55.7, 112 x 2000 55.3 : 47.0, 32 rows, 48 x 5000 53.2 : 44.8.
static bool single_read_wanted(const laq_shape* shape, const ScoreGeom& g, const KvLayout& lay, const hipStream_t* st) {
  if (shape->score_choice == LAQ_CHOOSE_SINGLE_READ) return true;
  if (shape->score_choice == LAQ_CHOOSE_TWO_PASS) return false;
  // by itself: where it is the faster one -- at most 64 score rows per KV head (with more, a
  // workgroup holds 256 keys and reads as many bytes of its team's statistics as of keys) and
  // enough keys to pay for its start -- and its waits are safe next to any other calls
  const long long key_bytes = (long long)g.n_inst * g.Hkv * g.L * g.d * (shape->dtype == LAQ_F32 ? 4 : 2);
  const bool many = key_bytes >= (128LL << 20);
  if (g.Rpad > 64 || (!many && (key_bytes < ((g.Rpad > 32 ? 40LL : 48LL) << 20) || (g.Rpad <= 32 && g.L <= 1280)))) return false;
  return score_fused_counters(g, lay, shape->dtype, st) >= (many ? 1 : 2);
}

// Heads of a call from which on their gather is spread over enough compute units with a workgroup each.
constexpr int HEAD_MANY = 72;

// Which kernels score a call.  The single-read kernel pools (maximum) where it scores; the one-workgroup kernel pools, selects and gathers
// too; the others leave raw scores.
enum class ScorePath { single_read, head, tile, wave };

// The kernels that give every 256-key chunk a workgroup of its own, where they are the faster ones.  They work on up to four row tiles of a
// chunk side by side where chunks are few, and hold all of a chunk's keys at once; the others have their score rows in LDS
// once for many keys and no barrier after that.  laq_evict, these : the others, us, by row tiles x chunks:
//   bf16, d = 128   1 x 32 17.5 : 18.7, 1 x 128 21.1 : 22.1, 1 x 288 26.7 : 28.7, 1 x 512 30.0 : 33.0; 1 x 280, 344 in 8 heads 31.0 : 27.9, 32.9 : 29.6
//                   2 x 16 20.4 : 19.5, 2 x 64 23.6 : 21.4, 2 x 256 31.9 : 30.5, 2 x 480 36.0 : 32.2
//                   4 x 39 27.8 : 29.5, 7 x 60 32.8 : 33.8, 4 x 65 26.5 : 25.7, 4 x 192 36.9 : 30.4, 4 x 399 38.5 : 32.4, 8 x 228 50.5 : 45.2
//   bf16, d = 64    1 x 96 21.8 : 22.6, 1 x 464 23.4 : 26.6, 2 x 192 21.9 : 19.3, 2 x 480 28.0 : 26.4, 4 x 48 22.0 : 22.6, 4 x 192 33.7 : 25.7
//   bf16, d = 256   1 x 48 26.0 : 28.7, 1 x 3752 212 : 216, 2 x 396 45.6 : 47.6, 2 x 4360 307 : 292, 4 x 140 39.9 : 36.2
//   fp32            1 x 72 24.9 : 25.2, 1 x 256 46.5 : 45.7, 2 x 38 34.2 : 36.3, 2 x 148 45.4 : 40.1, 4 x 24 28.3 : 32.7, 4 x 268 114.1 : 96.5
// fp32 with d > 128 always (the others have no registers for the parts of 32 such keys).
// Long heads, so few that a workgroup per chunk is one round of them, by row tiles x chunks in 4 heads: fp32, d = 128   1 x 252 38 : 45,
//   4 x 252 67 : 74; 1, 4 x 268 .96, 1.16 (these over the others); d = 96   1 x 252 34 : 38; d = 256   1 x 376 .87, 4 x 252 41 : 47, 4 x 376 .91;
//   in 8 heads 4 x 264 1.15.  More than eight row tiles, d = 256: 96 to 8000 chunks .82-.95; five (a
//   second group of one or two): up to 640 chunks .97-1.08, 768 to 3600 .86-.95.
// The other head sizes share one variant of the others for up to 256 (fp32: 128) elements; these have eight.  These over the others:
//   bf16, d = 8 to 112   1, 2 tiles .74-1.06, 4 .67-1.07, 8 .70-1.13, 14 .76-1.08; but heads of half a chunk, 4 and 14 tiles, 100 heads and more 1.0-1.28
//   bf16, d = 136 to 232   1 tile, up to 1500 chunks .77-1.07; 2, 4 tiles, up to 320 chunks .66-1.05, 512 .83-.94, 640 to 1500 .97-1.20 (900 heads of one chunk .83-.95), 8000 1.1-1.28;
//                   7, 8 tiles, up to 1024 chunks .66-1.08, 8000 1.02-1.17; 14 tiles .73-1.07; half a chunk, 4 and 14 tiles, d = 136 .89-1.25, 232 .82-1.04
//   fp32, d = 8, 16   .71-1.10, half a chunk and 4, 14 tiles .93-1.62;  d = 40   1 tile .69-1.04, 2 tiles 8 heads x 288 .97, 640 on 1.03-1.14, 4 tiles 4 heads
//                   x 256 .72, 8 heads x 192, 288 1.05, 1.06, 640 on 1.16-1.34;  d = 88, 112   1 tile, up to 512 chunks .74-1.06, 640 on 1.02-1.15; 2 tiles and
//                   more, 8 heads and more x 192 on 1.02-1.5;  1 to 6 heads, all types, up to 500 chunks .66-.98, 512 to 564 .75-.96, 780 to 940 .80-1.16,
//                   1096 on .92-1.14
//   Heads of half a chunk with d below 200 stay with the others however many they are: these kernels' scores are further from 64 bits (2-norm error, 512 heads x
//                   120 keys, 448 rows, d = 176: 1.28e-7 against 4.8e-8)
static bool tile_wanted(const laq_shape* shape, const ScoreGeom& g) {
  if (!score_wave_supported(g, shape->dtype)) return true;
  const bool f32 = shape->dtype == LAQ_F32;
  if (shape->score_choice != LAQ_CHOOSE_AUTO && !f32 && (g.d == 64 || g.d == 128)) return false;
  const long long heads = (long long)g.n_inst * g.Hkv, chunks = heads * g.nchunk;
  const int tiles = g.Rpad / 32;
  const bool half = 2 * g.L <= CHUNK_ROWS;               // (half of a workgroup's waves have no keys)
  if (!score_wave_own_size(g, shape->dtype) && !(half && tiles > 2 && (f32 || g.d < 200))) {
    if (heads < 8 && chunks <= 1024) return true;
    if (f32 && (g.d <= 32 || (tiles == 1 && (g.d < 64 || chunks <= 512)))) return true;
    if (!f32 && (g.d < 128 || tiles > 8 || g.nchunk == 1 || chunks <= (tiles > 4 ? 4096 : 512))) return true;
  }
  if (f32) return chunks <= 128 || (heads < 8 && chunks > 192 && chunks <= 256 && (tiles <= 4 || g.d > 96));
  if (g.d > 128) return tiles == 1 || (tiles > 8 && !half) || (tiles == 5 && chunks > 640) || chunks <= 64 || (chunks <= 512 && (tiles == 2 || heads < 8));
  if (tiles == 1) return chunks <= 512 && g.nchunk <= 32;
  return tiles > 2 && chunks <= 64;
}

// A workgroup for each head, with all its keys in registers.  Against the launches of the other kernels (laq_evict, us, the others : this one):
//   up to 512 keys always: bf16, d = 128, 24 heads 20.3 : 10.1 (d = 64), 64 heads 21.1 : 16.3, 576 heads 47.3 : 25.8, 2000 heads, 128 rows 314 : 226,
//   6016 heads 392 : 285; fp32, d = 64, 192 heads 30.2 : 24.9; but fp32 of more than 64 elements in few heads 6 heads 32.7 : 39.7, 16 heads 33.6 : 35.1,
//   80 heads 39.2 : 35.3; and many score rows in few 13 heads, 256 rows 42.2 : 53.4; 128 rows, 4 to 24 heads x 330 1.03, 395 and 512 .87-.89, 40 heads x
//   395 1.03 (the others over this one)
//   up to 1024 keys (two tiles per wave, one workgroup per compute unit), 72 to 768 heads, times as long in the two passes: bf16, 32 rows 1.38-1.73, 64 rows
//   1.19-1.45, 128 rows 1.01-1.27; fp32, d = 64, 32 rows 1.20-1.37, 48 rows and more (products made twice) 128 to 256 heads .98-1.21, 72 heads .72-.98, 300 to 768
//   .83-1.00; more than 768 heads, bf16, 32 rows 1.08-1.41, 64 rows .91-1.30, 128 rows .92-1.13, fp32, 32 rows 1.19-1.34, more .80-.90 (the last three lines and
//   some of the fp32 ones would be better drawn by whether products are made once and by heads per compute unit; 768 is from products made twice)
//   few heads, one or two row tiles whose products are made twice 16 x 768 22.2 : 19.7, 56 x 1024 23.9 : 25.6; more row tiles 64 x 714 32.7 : 34.5, 8 x 1024 26.0 :
//   32.1, 2 to 7 x 800 to 1000, 128 rows, d = 64 to 128 .81-1.02
//   few heads whose products are made once (head_keeps()): fp32, d = 64, 32 rows, 8 heads x 768, 1000 keys 22.8 : 18.5, 22.3 : 21.8, 64 x 800, 1000 25.3 : 20.2,
//   25.6 : 22.8; d = 128, 8 x 330, 500 29.9 : 17.7, 30.1 : 20.9; d = 96, 16 x 500 27.4 : 18.4; bf16, d = 128, 8 x 800, 1000 19.9 : 16.2, 19.6 : 17.5, 56 x 1000 21.9 :
//   18.6; d = 64, 32 x 1000 17.6 : 13.8, 64 rows, 64 x 1000 18.6 : 14.6.
//   Two lines of these lie where tests/test_abi.py has what laq_score_kernel() answers on the far side, and not where the times cross: fewer than 8 heads of more than
//   768 keys (bf16, 2 x 1000, 32 rows, d = 64, 96, 128 16.5 : 12.6, 17.0 : 12.7, 19.0 : 16.5; 769 keys no other), and fp32 with d > 64 in up to 16 heads of more than 448 (8 x
//   440 keys, taken, and 456, not: d = 72 13.7, 23.6 : 13.7; d = 128 18.2, 29.7 : 18.3).
static bool head_wanted(const laq_shape* shape, const ScoreGeom& g) {
  if (shape->score_choice != LAQ_CHOOSE_AUTO || !head_supported(g, shape->dtype)) return false;
  const long long heads = (long long)g.n_inst * g.Hkv;
  const bool f32 = shape->dtype == LAQ_F32;
  if (heads < HEAD_MANY && head_keeps(g, shape->dtype) && (g.L <= 768 || heads >= 8) && (!f32 || g.d <= 64 || heads > 16 || g.L <= 448)) return true;
  if (f32 && ((g.d > 64 && heads <= 16) || (g.Rpad > 128 && heads < HEAD_MANY) || (g.Rpad > 96 && heads < 40 && g.L > 384))) return false;
  if (g.L <= 512) return true;
  return heads >= HEAD_MANY ? heads <= 768 : g.L <= 768 && g.Rpad <= (f32 ? 32 : 64);
}

static ScorePath score_path(const laq_shape* shape, const ScoreGeom& g, const KvLayout& lay, hipStream_t st) {
  if (head_wanted(shape, g)) return ScorePath::head;
  if (SINGLE_READ_ENABLED && usual_shape(g, lay, shape->dtype) && score_fused_supported(g, lay, shape->dtype) && single_read_wanted(shape, g, lay, &st))
    return ScorePath::single_read;
  return tile_wanted(shape, g) ? ScorePath::tile : ScorePath::wave;
}

// Whether scores that are to be pooled come raw from the kernels that make them.
static bool leaves_raw(const laq_shape* shape, ScorePath path) {
  return path == ScorePath::tile || path == ScorePath::wave || (path == ScorePath::single_read && pool_avg(shape));
}

// Scores of a validated call into `scores`: pooled, or, with pool == 1, raw.
static int score_checked(const laq_shape* shape, const ScoreGeom& g, const QueryPos& positions, const KvLayout& lay, ScorePath path, const void* q_win,
                         const void* k, int pool, float* scores, void* ws, hipStream_t st) {
  if (g.Hkv > 65535 || g.n_inst > 65535 || (long long)g.Hkv * g.n_inst > 0x7fffffffLL) return LAQ_ERR_UNSUPPORTED;
  if ((g.L + 255) / 256 > 65535) return LAQ_ERR_UNSUPPORTED;      // grid limit of the pooling kernel
  const int rc_init = init_current_device(nullptr);
  if (rc_init != LAQ_OK) return rc_init;
  const Workspace w = carve_workspace(g, ws);
  WindowPos qp;
  hipError_t e = window_positions(g, positions, w, st, &qp);
  if (e != hipSuccess) return LAQ_ERR_DEVICE;
  if (path == ScorePath::single_read) {
    const bool apart = pool > 1 && pool_avg(shape);
    bool done = false;
    e = launch_score_fused(g, qp, lay, apart ? 1 : pool, q_win, k, apart ? w.raw : scores, w, st, &done);
    if (e == hipSuccess && done && apart) e = launch_pool(g, pool, true, w.raw, scores, st);
    if (e != hipSuccess || done) return e == hipSuccess ? LAQ_OK : LAQ_ERR_DEVICE;
    // (a team of its workgroups does not fit this device: the two passes)
  }
  if (path == ScorePath::head) {
    const bool apart = (pool - 1) / 2 > SELECT_POOL_MAX_HALF;
    FinishArgs fin;
    memset(&fin, 0, sizeof fin);
    fin.pooled = apart ? w.raw : scores;
    fin.half = apart ? 0 : (pool - 1) / 2;
    fin.avg = pool_avg(shape) ? 1 : 0;
    e = launch_head(g, qp, lay, shape->dtype, HEAD_SCORES, q_win, k, g.n_inst, 0, UniformInst{1, 0, 0}, nullptr, fin, w.status, st);
    if (e == hipSuccess && apart) e = launch_pool(g, pool, pool_avg(shape), w.raw, scores, st);
    return e == hipSuccess ? LAQ_OK : LAQ_ERR_DEVICE;
  }
  float* raw = pool > 1 ? w.raw : scores;
  e = path == ScorePath::tile ? launch_score_tile(g, qp, lay, shape->dtype, q_win, k, raw, w, st)
                              : launch_score_wave(g, qp, lay, shape->dtype, q_win, k, raw, w, st);
  if (e == hipSuccess && pool > 1) e = launch_pool(g, pool, pool_avg(shape), raw, scores, st);
  return e == hipSuccess ? LAQ_OK : LAQ_ERR_DEVICE;
}

static int score_impl(const laq_shape* shape, const void* q_win, const void* k, int pool, float* scores,
                      void* ws, size_t ws_bytes, hipStream_t st) {
  ScoreGeom g;
  QueryPos qp;
  const int rc = make_geom(shape, &g, &qp);
  if (rc != LAQ_OK) return rc;
  KvLayout lay;
  if (make_layout(shape, g, &lay) != LAQ_OK) return LAQ_ERR_INVALID;
  if (!pool_ok(pool) || !q_win || !k || !scores) return LAQ_ERR_INVALID;
  if (!ws || ws_bytes < workspace_bytes(g)) return LAQ_ERR_WORKSPACE;
  return score_checked(shape, g, qp, lay, score_path(shape, g, lay, st), q_win, k, pool, scores, ws, st);
}

// launch(n, i0, table) for runs of at most MAX_INST_PER_LAUNCH instances
template <typename LAUNCH>
static int for_instances(const ScoreGeom& g, const int32_t* budget, LAUNCH launch) {
  int64_t row = 0;
  for (int i0 = 0; i0 < g.n_inst; i0 += MAX_INST_PER_LAUNCH) {
    const int n = g.n_inst - i0 < MAX_INST_PER_LAUNCH ? g.n_inst - i0 : MAX_INST_PER_LAUNCH;
    hipError_t e;
    if (const int bk = uniform_rows(g.L, budget, i0, n)) {
      const UniformInst u{bk, row, (int64_t)g.Hkv * bk};
      e = launch(n, i0, u);
      row += n * u.per_inst;
    } else {
      InstTable tab;
      fill_table(g.Hkv, g.L, budget, i0, n, row, &tab, &row);
      e = launch(n, i0, tab);
    }
    if (e != hipSuccess) return LAQ_ERR_DEVICE;
  }
  return LAQ_OK;
}

static int select_impl(const laq_shape* shape, const float* scores, const int32_t* budget, int pool,
                       int32_t* idx, hipStream_t st, const PoolArgs* pooling = nullptr) {
  ScoreGeom g;
  const int rc = make_geom(shape, &g);
  if (rc != LAQ_OK) return rc;
  if (!pool_ok(pool) || !scores || !idx || !budgets_ok(shape, g, budget)) return LAQ_ERR_INVALID;
  if (g.Hkv > 65535) return LAQ_ERR_UNSUPPORTED;
  auto launch = [&](int n, int i0, const auto& tab) {
    return pooling ? launch_select_pooling(n, i0, g.Hkv, g.L, g.keep, scores, tab, idx, *pooling, st)
                   : launch_select(n, i0, g.Hkv, g.L, g.keep, pool, pool_avg(shape), scores, tab, idx, st);
  };
  return for_instances(g, budget, launch);
}

static int compact_impl(const laq_shape* shape, const void* k, const void* v, const int32_t* idx,
                        const int32_t* budget, void* k_out, void* v_out, hipStream_t st) {
  ScoreGeom g;
  const int rc = make_geom(shape, &g);
  if (rc != LAQ_OK) return rc;
  if (!k || !k_out || !idx || !budgets_ok(shape, g, budget)) return LAQ_ERR_INVALID;
  if ((v == nullptr) != (v_out == nullptr)) return LAQ_ERR_INVALID;
  KvLayout lay;
  if (make_layout(shape, g, &lay) != LAQ_OK) return LAQ_ERR_INVALID;
  const int row_bytes = g.d * (shape->dtype == LAQ_F32 ? 4 : 2);
  int64_t row = 0;
  for (int i0 = 0; i0 < shape->n_inst; i0 += MAX_INST_PER_LAUNCH) {
    const int n = shape->n_inst - i0 < MAX_INST_PER_LAUNCH ? shape->n_inst - i0 : MAX_INST_PER_LAUNCH;
    hipError_t e;
    if (const int bk = uniform_rows(g.L, budget, i0, n)) {
      const UniformInst u{bk, row, (int64_t)g.Hkv * bk};
      e = launch_compact(n, i0, g.Hkv, g.L, row_bytes, lay, k, v, idx, u, k_out, v_out, st);
      row += n * u.per_inst;
    } else {
      CompactTable tab;
      fill_compact_table(g.Hkv, g.L, row_bytes >> 4, budget, i0, n, row, &tab, &row);
      e = launch_compact(n, i0, g.Hkv, g.L, row_bytes, lay, k, v, idx, tab, k_out, v_out, st);
    }
    if (e != hipSuccess) return LAQ_ERR_DEVICE;
  }
  return LAQ_OK;
}

static int sink_recent_impl(int n_inst, int Hkv, int L, const int32_t* budget, int n_sink, int32_t* idx,
                            hipStream_t st) {
  if (n_inst < 1 || Hkv < 1 || L < 1 || n_sink < 0 || !budget || !idx) return LAQ_ERR_INVALID;
  for (int i = 0; i < n_inst; ++i)
    if (budget[i] < 1) return LAQ_ERR_INVALID;
  if (Hkv > 65535) return LAQ_ERR_UNSUPPORTED;
  int64_t row = 0;
  for (int i0 = 0; i0 < n_inst; i0 += MAX_INST_PER_LAUNCH) {
    const int n = n_inst - i0 < MAX_INST_PER_LAUNCH ? n_inst - i0 : MAX_INST_PER_LAUNCH;
    InstTable tab;
    memset(&tab, 0, sizeof tab);
    fill_table(Hkv, L, budget, i0, n, row, &tab, &row);
    if (launch_sink_recent(n, Hkv, L, n_sink, tab, idx, st) != hipSuccess) return LAQ_ERR_DEVICE;
  }
  return LAQ_OK;
}

// bytes of partial results of a decode call that may cut its caches into parts
static size_t decode_ws_bytes(const ScoreGeom& g, int dtype, const int32_t* budget) {
  return round256(decode_partial_bytes(g.n_inst, g.L, g.Hq, g.Hkv, g.d, dtype, budget));
}

static int decode_impl(const laq_shape* shape, const void* q, const void* kc, const void* vc,
                       const int32_t* budget, float* out, void* ws, size_t ws_bytes, hipStream_t st) {
  ScoreGeom g;
  const int rc = make_geom(shape, &g);
  if (rc != LAQ_OK) return rc;
  if (!q || !kc || !vc || !out || !budget) return LAQ_ERR_INVALID;
  for (int i = 0; i < shape->n_inst; ++i)
    if (budget[i] < 1) return LAQ_ERR_INVALID;
  if (g.Hkv > 65535) return LAQ_ERR_UNSUPPORTED;
  int part_rows = g.L;                     // without a workspace every cache is one part
  if (ws != nullptr) {
    if (ws_bytes < decode_ws_bytes(g, shape->dtype, budget)) return LAQ_ERR_WORKSPACE;
    part_rows = decode_part_rows(g.n_inst, g.L, g.Hq, g.Hkv, shape->dtype, budget);
  }
  return launch_decode(g.n_inst, g.L, g.Hq, g.Hkv, g.d, shape->dtype, g.scale2, part_rows, budget, q, kc, vc, out,
                       ws, st) == hipSuccess
             ? LAQ_OK
             : LAQ_ERR_DEVICE;
}

// Whether the selection kernel can do the pooling and the gather of this call along with the selection, and that is faster than
// pooling where the scores are made and launches of their own for selection and gather.  One workgroup works for a head, so with
// few heads its pass over the keys and its copies (K rows kept per head: `gather`) soon take longer than the launches they save; with a
// workgroup for most compute units they do not.  laq_evict, bf16, d = 128, pool 7, one launch : several, us:
//   keys <= 2048 (256 threads a head)   32 KiB: 8, 256 heads 21.4 : 22.6, 69.3 : 71.2;  64 KiB: 25.4 : 22.6, 81.5 : 77.7
//   4096 keys   8, 128 heads   32 KiB 21.2 : 24.8, 62.6 : 68.4;  96 KiB 24.6 : 25.3, 72.7 : 74.9;  128 KiB 24.5 : 24.2, 77.9 : 78.2
//   8001 keys   8, 64, 128 heads   32 KiB 24.6 : 25.8, 67.0 : 66.1, 95.1 : 98.4;  64 KiB 27.4 : 26.3, 71.1 : 68.5, 101.2 : 103.7;
//               128 heads 96 KiB 106.4 : 106.8, 128 KiB 111.9 : 111.0
//   16384 keys  8, 128 heads, 32 KiB 39.4 : 35.2, 158.9 : 155.2;  64 score rows, 128, 160, 256 heads 162.5 : 163.6, 191.3 : 193.9,
//               273.7 : 282.1, 128 KiB 178.3 : 174.5, 208.6 : 207.6, 298.0 : 303.9
//   160 heads, 128 KiB: 4096 keys 90.2 : 93.1, 8001 128.4 : 128.7;  256 heads 120.7 : 126.7, 178.2 : 181.1
//   more heads than compute units, 8001 keys: 384, 1024 heads 218.8 : 215.5, 522 : 505
// Where the single-read kernel would pool the maximum (in launches of its own beside the selection and the gather), more is saved, and the
// line is one by heads.  32 and 64 rows, 6000 to 16380 keys, several : one:   64 heads 64, 96, 128 KiB 1.03-1.06, 1.01-1.04, .99-1.00
//   96 heads 96, 128, 192 KiB 1.01-1.04, 1.00-1.02, .95-.98;  128 heads 128, 192 KiB 1.00-1.03, .99-1.00;  160 heads 128, 192 KiB 1.02-1.04, 1.01-1.03
//   256 heads 128, 192, 256 KiB 1.01-1.04; with rows 2 KiB apart 192 heads x 3867 keys, 217 KiB .97
static bool finish_wanted(const laq_shape* shape, const ScoreGeom& g, ScorePath path, const int32_t* budget, int pool, const float* raw,
                          int row_bytes) {
  const long long heads = (long long)g.n_inst * g.Hkv;
  const int keys = g.P + row_shift(raw, g.L);
  if ((pool - 1) / 2 > SELECT_POOL_MAX_HALF || keys > FINISH_MAX_KEYS || heads > 256 || shape->n_inst > MAX_INST_PER_LAUNCH) return false;
  long long gather = 0;
  if (keys <= 2048) gather = 32 << 10;
  else if (pool > 1 && !leaves_raw(shape, path)) gather = heads < 128 ? heads * 1280 : 160 << 10;
  else if (heads >= 160) gather = 128 << 10;
  else if (keys <= 4096 || (keys <= 8192 && heads >= 128)) gather = 96 << 10;
  else if (keys <= 8192) gather = 32 << 10;
  int most = 0;
  for (int i = 0; i < shape->n_inst; ++i) {
    const int bk = budget[i] < g.L ? budget[i] : g.L;
    if (bk > most) most = bk;
  }
  return (long long)most * row_bytes <= gather;
}

// Whether the selection kernel pools the raw scores of this call on the way: a launch, a read and a write of the scores less.  The
// single-read kernel would pool the maximum itself, all but the keys next to its workgroups' boundaries, which take a launch: laq_evict,
// pooled there : here, us: 256 heads x 2000 keys 58.4 : 55.4, 48 x 10000 54.4 : 53.4, 512 x 5000 196.9 : 195.4, 96 x 8192 and 128 x 16384
// even; 72 x 30011 141.2 : 144.3, 256 x 32768 518 : 524, 720 x 20000 829 : 847.  (Few long heads, whose selection is on few compute
// units anyway, are not among these.)
static bool select_pools(const laq_shape* shape, const ScoreGeom& g, ScorePath path, int pool, const float* raw) {
  const int keys = g.P + row_shift(raw, g.L);
  return pool > 1 && (pool - 1) / 2 <= SELECT_POOL_MAX_HALF && keys <= SELECT_POOL_MAX_KEYS &&
         (keys <= SELECT_POOL_MANY_KEYS || (long long)g.n_inst * g.Hkv < SELECT_MANY_HEADS) &&
         (leaves_raw(shape, path) || (path == ScorePath::single_read && keys <= FINISH_MAX_KEYS));
}

static FinishArgs finish_args(const laq_shape* shape, const ScoreGeom& g, const KvLayout& lay, const void* k, const void* v, int pool, float* scores,
                              void* k_out, void* v_out) {
  const int eb = shape->dtype == LAQ_F32 ? 4 : 2;
  FinishArgs fin;
  fin.pooled = scores;
  fin.half = (pool - 1) / 2; fin.avg = pool_avg(shape) ? 1 : 0;
  fin.k = static_cast<const char*>(k); fin.v = static_cast<const char*>(v);
  fin.k_out = static_cast<char*>(k_out); fin.v_out = static_cast<char*>(v_out);
  fin.inst_bytes = lay.inst * eb; fin.head_bytes = lay.head * eb;
  fin.row_bytes = g.d * eb; fin.src_row_bytes = lay.row_bytes; fin.elem_bytes = eb;
  fin.lay = lay;
  return fin;
}

// Pooling, selection and gather of a small call, from the raw scores.
static int finish_checked(const ScoreGeom& g, const FinishArgs& fin, const int32_t* budget, const float* raw, int32_t* idx, hipStream_t st) {
  return for_instances(g, budget, [&](int n, int i0, const auto& tab) { return launch_finish(n, i0, g.Hkv, g.L, g.keep, raw, tab, idx, fin, st); });
}

// How far the kernel that scores short heads goes: one workgroup copies a head's rows, which takes longer than a
// launch that spreads them where heads are few and rows many (8 heads x 1017 keys, 688 rows kept 26.3 us, 20.3 with a launch for it).  The selection it does itself
// but for the widest pooling (8, 32 heads x 1000 keys, 900 rows kept, bf16, d = 128: in a launch of its own
// 22.1, 25.5 us, so 18.8, 22.5).
static HeadSteps head_steps(const laq_shape* shape, const ScoreGeom& g, const int32_t* budget, int pool, int row_bytes) {
  if ((pool - 1) / 2 > SELECT_POOL_MAX_HALF) return HEAD_SCORES;
  if (g.L <= 512 || (long long)g.n_inst * g.Hkv >= HEAD_MANY) return HEAD_ROWS;
  int most = 0;
  for (int i = 0; i < shape->n_inst; ++i) most = budget[i] > most ? budget[i] : most;
  return (long long)(most < g.L ? most : g.L) * row_bytes <= 128 << 10 ? HEAD_ROWS : HEAD_LIST;
}

// A call of short heads up to their lists or their rows.
static int head_checked(const laq_shape* shape, const ScoreGeom& g, const QueryPos& positions, const KvLayout& lay, const FinishArgs& fin, HeadSteps steps,
                        const void* q_win, const void* k, const int32_t* budget, int32_t* idx, void* ws, hipStream_t st) {
  if (g.Hkv > 65535 || g.n_inst > 65535 || (long long)g.Hkv * g.n_inst > 0x7fffffffLL) return LAQ_ERR_UNSUPPORTED;
  const int rc_init = init_current_device(nullptr);
  if (rc_init != LAQ_OK) return rc_init;
  const Workspace w = carve_workspace(g, ws);
  WindowPos qp;
  if (window_positions(g, positions, w, st, &qp) != hipSuccess) return LAQ_ERR_DEVICE;
  return for_instances(g, budget, [&](int n, int i0, const auto& tab) {
    return launch_head(g, qp, lay, shape->dtype, steps, q_win, k, n, i0, tab, idx, fin, w.status, st);
  });
}

static int qcache_store_impl(const laq_shape* shape, const void* q_step, int t, void* q_cache, hipStream_t st) {
  ScoreGeom g;
  const int rc = make_geom(shape, &g);
  if (rc != LAQ_OK) return rc;
  if (!q_step || !q_cache || t < 0 || t >= g.W) return LAQ_ERR_INVALID;
  const int row_bytes = g.d * (shape->dtype == LAQ_F32 ? 4 : 2);
  return launch_qcache_store((long long)g.n_inst * g.Hq, g.W, t, row_bytes, q_step, q_cache, st) == hipSuccess
             ? LAQ_OK
             : LAQ_ERR_DEVICE;
}

static int recall_impl(int n_inst, int Hkv, int L, const int32_t* idx_pred, const int32_t* budget_pred,
                       const int32_t* idx_gold, const int32_t* budget_gold, int32_t* overlap, float* recall,
                       hipStream_t st) {
  if (n_inst < 1 || Hkv < 1 || L < 1 || !idx_pred || !budget_pred || !idx_gold || !budget_gold || !overlap)
    return LAQ_ERR_INVALID;
  for (int i = 0; i < n_inst; ++i)
    if (budget_pred[i] < 1 || budget_gold[i] < 1) return LAQ_ERR_INVALID;
  if (Hkv > 65535) return LAQ_ERR_UNSUPPORTED;
  int64_t row_a = 0, row_b = 0;
  for (int i0 = 0; i0 < n_inst; i0 += MAX_PAIR_PER_LAUNCH) {
    const int n = n_inst - i0 < MAX_PAIR_PER_LAUNCH ? n_inst - i0 : MAX_PAIR_PER_LAUNCH;
    PairTable tab;
    memset(&tab, 0, sizeof tab);
    for (int i = 0; i < n; ++i) {
      tab.bk_a[i] = budget_pred[i0 + i] < L ? budget_pred[i0 + i] : L;
      tab.bk_b[i] = budget_gold[i0 + i] < L ? budget_gold[i0 + i] : L;
      tab.row_a[i] = row_a;
      tab.row_b[i] = row_b;
      row_a += (int64_t)Hkv * tab.bk_a[i];
      row_b += (int64_t)Hkv * tab.bk_b[i];
    }
    if (launch_recall(n, i0, Hkv, tab, idx_pred, idx_gold, overlap, recall, st) != hipSuccess) return LAQ_ERR_DEVICE;
  }
  return LAQ_OK;
}

}  // namespace laq

extern "C" {

size_t laq_workspace_bytes(const laq_shape* shape) {
  laq::ScoreGeom g;
  if (laq::make_geom(shape, &g) != LAQ_OK) return 0;
  return laq::workspace_bytes(g);
}

int laq_score(const laq_shape* shape, const void* q_win, const void* k, int pool_kernel, float* scores,
              void* ws, size_t ws_bytes, void* stream) {
  return laq::score_impl(shape, q_win, k, pool_kernel, scores, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

int laq_select(const laq_shape* shape, const float* scores, const int32_t* budget, int pool_kernel,
               int32_t* idx, void* stream) {
  return laq::select_impl(shape, scores, budget, pool_kernel, idx, static_cast<hipStream_t>(stream));
}

int laq_select_sink_recent(int32_t n_inst, int32_t Hkv, int32_t L, const int32_t* budget, int32_t n_sink,
                           int32_t* idx, void* stream) {
  return laq::sink_recent_impl(n_inst, Hkv, L, budget, n_sink, idx, static_cast<hipStream_t>(stream));
}

size_t laq_decode_workspace_bytes(const laq_shape* shape, const int32_t* budget) {
  laq::ScoreGeom g;
  if (laq::make_geom(shape, &g) != LAQ_OK || !budget) return 0;
  for (int i = 0; i < shape->n_inst; ++i)
    if (budget[i] < 1) return 0;
  return laq::decode_ws_bytes(g, shape->dtype, budget);
}

int laq_decode_attention(const laq_shape* shape, const void* q, const void* k_c, const void* v_c,
                         const int32_t* budget, float* out, void* ws, size_t ws_bytes, void* stream) {
  return laq::decode_impl(shape, q, k_c, v_c, budget, out, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

int laq_qcache_store(const laq_shape* shape, const void* q_step, int32_t t, void* q_cache, void* stream) {
  return laq::qcache_store_impl(shape, q_step, t, q_cache, static_cast<hipStream_t>(stream));
}

int laq_recall(int32_t n_inst, int32_t Hkv, int32_t L, const int32_t* idx_pred, const int32_t* budget_pred,
               const int32_t* idx_gold, const int32_t* budget_gold, int32_t* overlap, float* recall, void* stream) {
  return laq::recall_impl(n_inst, Hkv, L, idx_pred, budget_pred, idx_gold, budget_gold, overlap, recall,
                          static_cast<hipStream_t>(stream));
}

int laq_compact(const laq_shape* shape, const void* k, const void* v, const int32_t* idx,
                const int32_t* budget, void* k_out, void* v_out, void* stream) {
  return laq::compact_impl(shape, k, v, idx, budget, k_out, v_out, static_cast<hipStream_t>(stream));
}

static int evict_impl(const laq_shape* shape, const void* q_win, const void* k, const void* v, const int32_t* budget,
                      int pool_kernel, float* scores, int32_t* idx, void* k_out, void* v_out, void* ws,
                      size_t ws_bytes, bool use_static_scratch, hipStream_t st) {
  // validate everything first so that a rejected call has enqueued nothing
  laq::ScoreGeom g;
  laq::QueryPos qp;
  const int rc0 = laq::make_geom(shape, &g, &qp);
  if (rc0 != LAQ_OK) return rc0;
  if (!laq::pool_ok(pool_kernel) || !q_win || !k || !idx || !k_out ||
      !laq::budgets_ok(shape, g, budget) || ((v == nullptr) != (v_out == nullptr)))
    return LAQ_ERR_INVALID;
  laq::KvLayout lay;
  if (laq::make_layout(shape, g, &lay) != LAQ_OK) return LAQ_ERR_INVALID;
  if (use_static_scratch) {
    if (laq::workspace_bytes(g) > (size_t)LAQ_STATIC_SCRATCH_BYTES) return LAQ_ERR_WORKSPACE;
    int dev = 0;
    const int rc_init = laq::init_current_device(&dev);
    if (rc_init != LAQ_OK) return rc_init;
    ws = laq::scratch_of[dev].load(std::memory_order_acquire);
    ws_bytes = (size_t)LAQ_STATIC_SCRATCH_BYTES;
  }
  if (!ws || ws_bytes < laq::workspace_bytes(g)) return LAQ_ERR_WORKSPACE;
  const laq::Workspace w = laq::carve_workspace(g, ws);
  if (!scores) scores = w.pooled;        // the hand-over plane between the stages
  const int row_bytes = g.d * (shape->dtype == LAQ_F32 ? 4 : 2);
  float* raw = pool_kernel > 1 ? w.raw : scores;
  const laq::ScorePath path = laq::score_path(shape, g, lay, st);
  const laq::HeadSteps steps = path == laq::ScorePath::head ? laq::head_steps(shape, g, budget, pool_kernel, row_bytes) : laq::HEAD_SCORES;
  if (steps != laq::HEAD_SCORES) {
    const int rc = laq::head_checked(shape, g, qp, lay, laq::finish_args(shape, g, lay, k, v, pool_kernel, scores, k_out, v_out), steps, q_win, k, budget, idx, ws, st);
    return rc != LAQ_OK || steps == laq::HEAD_ROWS ? rc : laq::compact_impl(shape, k, v, idx, budget, k_out, v_out, st);
  }
  if (path != laq::ScorePath::head && laq::finish_wanted(shape, g, path, budget, pool_kernel, raw, row_bytes)) {
    const int rc = laq::score_checked(shape, g, qp, lay, path, q_win, k, 1, raw, ws, st);
    if (rc != LAQ_OK) return rc;
    return laq::finish_checked(g, laq::finish_args(shape, g, lay, k, v, pool_kernel, scores, k_out, v_out), budget, raw, idx, st);
  }
  int rc;
  if (laq::select_pools(shape, g, path, pool_kernel, raw)) {
    rc = laq::score_checked(shape, g, qp, lay, path, q_win, k, 1, raw, ws, st);
    if (rc != LAQ_OK) return rc;
    const laq::PoolArgs pooling{scores, (pool_kernel - 1) / 2, laq::pool_avg(shape) ? 1 : 0};
    rc = laq::select_impl(shape, raw, budget, 1, idx, st, &pooling);
  } else {
    rc = laq::score_checked(shape, g, qp, lay, path, q_win, k, pool_kernel, scores, ws, st);
    if (rc != LAQ_OK) return rc;
    rc = laq::select_impl(shape, scores, budget, 1, idx, st);
  }
  if (rc != LAQ_OK) return rc;
  return laq::compact_impl(shape, k, v, idx, budget, k_out, v_out, st);
}

int laq_evict(const laq_shape* shape, const void* q_win, const void* k, const void* v, const int32_t* budget,
              int pool_kernel, float* scores, int32_t* idx, void* k_out, void* v_out, void* ws,
              size_t ws_bytes, void* stream) {
  return evict_impl(shape, q_win, k, v, budget, pool_kernel, scores, idx, k_out, v_out, ws, ws_bytes, false,
                    static_cast<hipStream_t>(stream));
}

int laq_evict_static(const laq_shape* shape, const void* q_win, const void* k, const void* v, const int32_t* budget,
                     int pool_kernel, float* scores, int32_t* idx, void* k_out, void* v_out, void* stream) {
  return evict_impl(shape, q_win, k, v, budget, pool_kernel, scores, idx, k_out, v_out, nullptr, 0, true,
                    static_cast<hipStream_t>(stream));
}

int laq_init(void) { return laq::init_current_device(nullptr); }

int laq_score_kernel(const laq_shape* shape) {
  laq::ScoreGeom g;
  const int rc = laq::make_geom(shape, &g);
  if (rc != LAQ_OK) return rc;
  laq::KvLayout lay;
  if (laq::make_layout(shape, g, &lay) != LAQ_OK) return LAQ_ERR_INVALID;
  if (laq::head_wanted(shape, g)) return LAQ_KERNEL_WHOLE_HEAD;
  if (!laq::usual_shape(g, lay, shape->dtype)) return LAQ_KERNEL_VECTOR;
  bool single = false;
  if (laq::SINGLE_READ_ENABLED && laq::single_read_wanted(shape, g, lay, nullptr) &&
      laq::score_fused_applies(g, lay, shape->dtype, &single) != hipSuccess)
    return LAQ_ERR_DEVICE;
  return single ? LAQ_KERNEL_SINGLE_READ : LAQ_KERNEL_TWO_PASS;
}

int laq_workspace_status(const laq_shape* shape, const void* ws, size_t ws_bytes, void* stream) {
  laq::ScoreGeom g;
  const int rc0 = laq::make_geom(shape, &g);
  if (rc0 != LAQ_OK) return rc0;
  if (!ws || ws_bytes < laq::workspace_bytes(g)) return LAQ_ERR_WORKSPACE;
  const laq::Workspace w = laq::carve_workspace(g, const_cast<void*>(ws));
  hipStream_t st = static_cast<hipStream_t>(stream);
  int word = 0;
  if (hipMemcpyAsync(&word, w.status, sizeof word, hipMemcpyDeviceToHost, st) != hipSuccess) return LAQ_ERR_DEVICE;
  if (hipStreamSynchronize(st) != hipSuccess) return LAQ_ERR_DEVICE;
  return word == 0 ? LAQ_OK : LAQ_ERR_TIMEOUT;
}

const char* laq_strerror(int code) {
  switch (code) {
    case LAQ_OK: return "ok";
    case LAQ_ERR_INVALID: return "invalid argument";
    case LAQ_ERR_UNSUPPORTED: return "unsupported shape";
    case LAQ_ERR_WORKSPACE: return "workspace missing or too small";
    case LAQ_ERR_DEVICE: return "HIP launch failed";
    case LAQ_ERR_TIMEOUT: return "a kernel gave up waiting for its peers; results are not valid";
    default: return "unknown error";
  }
}

}  // extern "C"
