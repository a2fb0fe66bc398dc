// What the selecting kernels share: the order of scores as keys, ranking of one key per thread, the gather of listed rows.
#pragma once

#include "laq_internal.h"

namespace laq {

__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);   // larger float <=> larger key
}

__device__ __forceinline__ int lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// inclusive sum over the lanes of a wave
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or(int none, int x) { return __builtin_amdgcn_update_dpp(none, x, CTRL, ROWS, 0xf, false); }
__device__ __forceinline__ int wave_scan(int x) {
  x += dpp_or<0x111, 0xf>(0, x);           // row_shr 1, 2, 4, 8 within 16 lanes
  x += dpp_or<0x112, 0xf>(0, x);
  x += dpp_or<0x114, 0xf>(0, x);
  x += dpp_or<0x118, 0xf>(0, x);
  x += dpp_or<0x142, 0xa>(0, x);           // lane 15 of a row to the next row
  x += dpp_or<0x143, 0xc>(0, x);           // lane 31 to the upper half
  return x;
}
// the largest of a wave's lanes, in lane 63
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  x = max(x, (uint32_t)dpp_or<0x111, 0xf>(0, (int)x));
  x = max(x, (uint32_t)dpp_or<0x112, 0xf>(0, (int)x));
  x = max(x, (uint32_t)dpp_or<0x114, 0xf>(0, (int)x));
  x = max(x, (uint32_t)dpp_or<0x118, 0xf>(0, (int)x));
  x = max(x, (uint32_t)dpp_or<0x142, 0xa>(0, (int)x));
  x = max(x, (uint32_t)dpp_or<0x143, 0xc>(0, (int)x));
  return x;
}

// ---- one key per thread ----
constexpr int RANK_FEW = 64;               // keys that are ranked by comparing all pairs
template <int WAVES> struct RankScratch {
  int bins[WAVES * 64];                    // (cleared by the caller, a barrier before the call)
  alignas(16) uint32_t few[RANK_FEW];
  uint32_t high[WAVES], low[WAVES];        // by wave: the largest key, and the largest complement of one
  int total[WAVES], above[WAVES], equal[WAVES];
  int n_few, bin, before, count;
};

// The place of this thread's key among the `want` largest of the workgroup's, these in the order of the threads; -1: not among
// them.  Equal keys: the lower threads' first.  0 is no key; there are more than `want` keys.  The keys (of floats: a logarithmic scale) are counted in as
// many bins as threads between the smallest and the largest, the bin of the want-th largest again if it holds more than RANK_FEW,
// else all pairs of it are compared.  What bounds it: seven barriers of 16 waves.  (512 keys: about 1 us; bit by bit with ballots 2.4 to
// 5.2 us in one wave, 3 to 7 us with sixteen waves and a barrier per four bits.)
template <int WAVES>
__device__ __forceinline__ int rank_position(RankScratch<WAVES>& sh, uint32_t key, int want, int lane, int wave) {
  constexpr int THREADS = WAVES * 64, BITS = WAVES == 16 ? 10 : 9;
  static_assert(1 << BITS == THREADS, "one bin per thread");
  const int tid = threadIdx.x;
  {
    const uint32_t hi = wave_max(key), lo = wave_max(key ? ~key : 0u);
    if (lane == 63) {
      sh.high[wave] = hi;
      sh.low[wave] = lo;
    }
    if (tid == 0) sh.n_few = 0;
  }
  __syncthreads();
  uint32_t high = 0, low = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    high = max(high, sh.high[w]);
    low = max(low, sh.low[w]);
  }
  uint32_t base = ~low, range = high - base;
  uint32_t t;
  int equal_wanted = 0;
#pragma unroll 1
  for (;;) {
    const int shift = max(32 - __clz((int)range) - BITS, 0);               // (range 0: clz is 32)
    const bool in = key >= base && key - base <= range && key != 0;
    if (in) atomicAdd(&sh.bins[(key - base) >> shift], 1);
    __syncthreads();
    const int b = THREADS - 1 - tid, n = sh.bins[b];
    const int upto = wave_scan(n);
    if (lane == 63) sh.total[wave] = upto;
    __syncthreads();
    int incl = upto;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) incl += w < wave ? sh.total[w] : 0;
    if (incl - n < want && want <= incl) {
      sh.bin = b;
      sh.before = incl - n;
      sh.count = n;
    }
    __syncthreads();
    const int bin = sh.bin, count = sh.count;
    want -= sh.before;
    base += (uint32_t)bin << shift;
    range = (1u << shift) - 1;
    if (count == want || shift == 0) {
      t = count == want ? base - 1 : base;
      equal_wanted = count == want ? 0 : want;
      break;
    }
    if (count <= RANK_FEW) {
      if (key >= base && key - base <= range && key != 0) sh.few[atomicAdd(&sh.n_few, 1)] = key;
      __syncthreads();
      const uint32_t mine = lane < count ? sh.few[lane] : 0u;
      int gt = 0, eq = 0;
      for (int j = 0; j < count; j += 4) {
        const uint4 c = *reinterpret_cast<const uint4*>(sh.few + j);       // (beyond count: whatever was there before)
        gt += (c.x > mine) + (j + 1 < count && c.y > mine) + (j + 2 < count && c.z > mine) + (j + 3 < count && c.w > mine);
        eq += (c.x == mine) + (j + 1 < count && c.y == mine) + (j + 2 < count && c.z == mine) + (j + 3 < count && c.w == mine);
      }
      const int l = __ffsll((long long)__ballot(lane < count && gt < want && want <= gt + eq)) - 1;
      t = (uint32_t)__builtin_amdgcn_readlane((int)mine, l);
      equal_wanted = want - __builtin_amdgcn_readlane(gt, l);
      break;
    }
    sh.bins[tid] = 0;                      // (every thread has read its own, and the result, by now)
    __syncthreads();
  }
  const bool gt = key > t, eq = key == t;
  const uint64_t mg = __ballot(gt), me = __ballot(eq);
  if (lane == 0) {
    sh.above[wave] = __popcll(mg);
    sh.equal[wave] = __popcll(me);
  }
  __syncthreads();
  int g_before = lanes_below(mg), e_before = lanes_below(me);
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    g_before += w < wave ? sh.above[w] : 0;
    e_before += w < wave ? sh.equal[w] : 0;
  }
  return gt || (eq && e_before < equal_wanted) ? g_before + min(e_before, equal_wanted) : -1;
}

// ---- K and V rows of a head's list to the packed outputs ----
// row_of(r): position of list entry r; row0: the list's first output row.  Several pieces per thread and turn, so that their list
// entries and then their rows are on the way together.
template <int THREADS, typename ROW>
__device__ __forceinline__ void gather_rows(const FinishArgs& fin, int inst, int head, int bk, int64_t row0, ROW row_of) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));           // (a native vector: arrays of it stay in registers)
  constexpr int TURN = 4;
  const int tid = threadIdx.x, ppr = fin.row_bytes >> 4, total = bk * ppr;
  const char *ks = fin.k + (size_t)head * fin.head_bytes, *vs = fin.v + (fin.v ? (size_t)head * fin.head_bytes : 0);
  const int drow = THREADS / ppr, dcol = THREADS - drow * ppr;
  int row = tid / ppr, col = tid - row * ppr;
  for (int p = tid; p < total; p += THREADS * TURN) {
    int j[TURN];
    size_t from[TURN], to[TURN];
#pragma unroll
    for (int u = 0; u < TURN; ++u) {
      const bool in = p + u * THREADS < total;
      j[u] = row_of(in ? row : 0);
      from[u] = (size_t)col * 16;
      to[u] = (size_t)(row0 + row) * fin.row_bytes + (size_t)col * 16;
      row += drow;
      col += dcol;
      if (col >= ppr) {
        col -= ppr;
        ++row;
      }
    }
    u32x4 x[TURN], y[TURN];
#pragma unroll
    for (int u = 0; u < TURN; ++u) {
      if (fin.lay.table) {
        int r;
        from[u] += (size_t)paged_block_offset(fin.lay, inst, j[u], &r) * fin.elem_bytes + (size_t)r * fin.src_row_bytes;
      } else {
        from[u] += (size_t)inst * fin.inst_bytes + (size_t)j[u] * fin.src_row_bytes;
      }
      x[u] = *reinterpret_cast<const u32x4*>(ks + from[u]);
      if (fin.v) y[u] = *reinterpret_cast<const u32x4*>(vs + from[u]);
    }
#pragma unroll
    for (int u = 0; u < TURN; ++u) {
      if (p + u * THREADS < total) {
        *reinterpret_cast<u32x4*>(fin.k_out + to[u]) = x[u];
        if (fin.v) *reinterpret_cast<u32x4*>(fin.v_out + to[u]) = y[u];
      }
    }
  }
}

}  // namespace laq
