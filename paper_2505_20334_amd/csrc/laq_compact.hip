// Cache compaction: gather the retained key / value rows into the compacted cache the
// decoder continues on (Sec. 4.3, the re-eviction that follows the ranking of Eq. 4).
// Pure data movement: each 16-byte piece of an output row is copied by one lane, so a
// 256-byte bf16 row (d = 128) is one coalesced 16-lane read and one coalesced write.  The source
// rows are addressed through byte strides (instance, head, row), or through the block table of a
// paged cache; the output is packed.
#include "laq_internal.h"

namespace laq {

namespace {

constexpr int CP_THREADS = COMPACT_THREADS;

// the instance of a workgroup and the workgroup's number among its instance's
__device__ __forceinline__ int instance_of(const CompactTable& tab, int n_inst, int blk, int* local) {
  // the last one whose first workgroup is not beyond it (uniform bisection over the table in the
  // kernel arguments)
  int lo = 0, hi = n_inst;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (tab.blk0[mid] <= blk) lo = mid; else hi = mid;
  }
  *local = blk - tab.blk0[lo];
  return lo;
}
struct UniformCompact {
  UniformInst u;
  int32_t blocks_per_inst;
};
__device__ __forceinline__ int instance_of(const UniformCompact& tab, int, int blk, int* local) {
  const int i = blk / tab.blocks_per_inst;
  *local = blk - i * tab.blocks_per_inst;
  return i;
}
__device__ __forceinline__ int rows_of(const CompactTable& tab, int i) { return tab.bk[i]; }
__device__ __forceinline__ int rows_of(const UniformCompact& tab, int i) { return tab.u.rows(i); }
__device__ __forceinline__ int64_t first_of(const CompactTable& tab, int i) { return tab.row0[i]; }
__device__ __forceinline__ int64_t first_of(const UniformCompact& tab, int i) { return tab.u.first(i); }

template <typename TAB>
__global__ __launch_bounds__(CP_THREADS) void compact_kernel(int n_inst, int Hkv, int L, int row_bytes, size_t inst_bytes,
                                                             size_t head_bytes, size_t src_row_bytes, KvLayout lay,
                                                             TAB tab,
                                                             int inst0, const char* __restrict__ k,
                                                             const char* __restrict__ v,
                                                             const int32_t* __restrict__ idx,
                                                             char* __restrict__ k_out, char* __restrict__ v_out) {
  int local;
  const int li = instance_of(tab, n_inst, (int)blockIdx.x, &local);
  const int bk = rows_of(tab, li);
  const int ppr = row_bytes >> 4;                              // 16-byte pieces per row
  const int64_t piece = (int64_t)local * CP_THREADS + threadIdx.x;
  const int64_t row = piece / ppr;
  const int col = (int)(piece - row * ppr);
  if (row >= (int64_t)Hkv * bk) return;
  const int head = (int)(row / bk);
  const int64_t orow = first_of(tab, li) + row;
  const int j = idx[orow];
  if (j < 0 || j >= L) return;
  const char* src = (blockIdx.y == 0) ? k : v;
  char* dst = (blockIdx.y == 0) ? k_out : v_out;
  size_t so = (size_t)(inst0 + li) * inst_bytes + (size_t)j * src_row_bytes;
  if (lay.table) {                       // paged cache: the row's block, and its row in there
    int r;
    const size_t eb = src_row_bytes / (size_t)lay.row;
    so = (size_t)paged_block_offset(lay, inst0 + li, j, &r) * eb;
    so += (size_t)r * src_row_bytes;
  }
  so += (size_t)head * head_bytes + (size_t)col * 16;
  const size_t dof = (size_t)orow * row_bytes + (size_t)col * 16;
  *reinterpret_cast<uint4*>(dst + dof) = *reinterpret_cast<const uint4*>(src + so);
}

template <typename TAB>
hipError_t launch(int blocks, int n_inst, int inst0, int Hkv, int L, int row_bytes, const KvLayout& lay, const void* k, const void* v,
                  const int32_t* idx, const TAB& tab, void* k_out, void* v_out, hipStream_t st) {
  if (blocks == 0) return hipSuccess;
  dim3 grid((unsigned)blocks, v ? 2 : 1);
  const size_t eb = (size_t)lay.row_bytes / (size_t)lay.row;        // element size of the source rows
  hipLaunchKernelGGL(compact_kernel<TAB>, grid, dim3(CP_THREADS), 0, st, n_inst, Hkv, L, row_bytes, (size_t)lay.inst * eb,
                     (size_t)lay.head * eb, (size_t)lay.row_bytes, lay, tab, inst0,
                     static_cast<const char*>(k), static_cast<const char*>(v), idx, static_cast<char*>(k_out),
                     static_cast<char*>(v_out));
  return hipGetLastError();
}

}  // namespace

hipError_t launch_compact(int n_inst, int inst0, int Hkv, int L, int row_bytes, const KvLayout& lay,
                          const void* k, const void* v, const int32_t* idx, const CompactTable& tab, void* k_out,
                          void* v_out, hipStream_t st) {
  return launch(tab.blk0[n_inst], n_inst, inst0, Hkv, L, row_bytes, lay, k, v, idx, tab, k_out, v_out, st);
}

hipError_t launch_compact(int n_inst, int inst0, int Hkv, int L, int row_bytes, const KvLayout& lay,
                          const void* k, const void* v, const int32_t* idx, const UniformInst& tab, void* k_out,
                          void* v_out, hipStream_t st) {
  UniformCompact u;
  u.u = tab;
  u.blocks_per_inst = (int)(((int64_t)Hkv * tab.bk * (row_bytes >> 4) + CP_THREADS - 1) / CP_THREADS);
  return launch(u.blocks_per_inst * n_inst, n_inst, inst0, Hkv, L, row_bytes, lay, k, v, idx, u, k_out, v_out, st);
}

}  // namespace laq
