// The steps around the re-eviction (Sec. 4.2 / 4.3): storing the queries of a lookahead step into
// the Q-cache, and the attention of one new token over the compacted cache that decoding
// continues on.
//
// Decode attention reads K' and V' once.  One workgroup serves up to eight query heads that share a KV head
// (they share every key and value row it reads) over one part of a cache: caches are cut into parts (laq_parts.h)
// where there would be too few workgroups otherwise (a compute unit alone reads some 25 KB per
// microsecond), and the workgroup that finds all parts of its cache finished folds them (merge_parts).
// A row is read by a group of PP adjacent lanes, 8 elements each, so a wave's loads cover whole rows contiguously;
// the lane groups of the workgroup take the rows round-robin, ROWS rows per turn.
//
// What bounds it next to memory is the vector ALU (it was busy 62 % of the time when every lane of a group held
// every logit of its rows).  So the sum over a group's lanes leaves each logit in one lane (halving exchange),
// one exponential then serves 16 (row, head) pairs, and the weighted sum of the value rows takes its weights from
// those lanes through the operand's lane selection.  2048 caches x 256 rows x 4 heads, bf16, 275 MB: 56 us before, 45
// now (6.1 TB/s); 256 caches of 128 to 2048 rows, 143 MB: 43 us in two launches before, 35 now; 8 caches of 512
// rows: 13 us before, 7 now.
//
// Each group keeps its own running (max, sum, weighted value sum) per query head; the groups of a wave are merged
// in registers, the waves through LDS, in a fixed order (the results do not depend on timing).
#include <atomic>
#include <chrono>
#include <type_traits>

#include "laq_internal.h"
#include "laq_lanegroup.h"
#include "laq_parts.h"

namespace laq {

namespace {

constexpr float DEC_NEG_BIG = -1.0e30f;
constexpr int DEC_THREADS = 256, DEC_WAVES = DEC_THREADS / 64;

template <int FROM, int TO, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (FROM < TO) {
    f(std::integral_constant<int, FROM>{});
    static_for<FROM + 1, TO>(f);
  }
}

// Eight elements of a row that the launch reads once (ONCE: the caches need not keep it, 45 us instead of 50 for 275 MB) or
// that several workgroups read (then that took 54 us instead of 50).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool ONCE>
__device__ __forceinline__ uint4 load16(const void* p) {
  if constexpr (ONCE) {
    const u32x4 r = __builtin_nontemporal_load(static_cast<const u32x4*>(p));
    return make_uint4(r[0], r[1], r[2], r[3]);
  } else {
    return *static_cast<const uint4*>(p);
  }
}
template <bool ONCE>
__device__ __forceinline__ void fetch_row(const uint16_t* p, Piece8BF16& x) { x.r = load16<ONCE>(p); }
template <bool ONCE>
__device__ __forceinline__ void fetch_row(const float* p, Piece8F32& x) {
  x.a = __builtin_bit_cast(float4, load16<ONCE>(p));
  x.b = __builtin_bit_cast(float4, load16<ONCE>(p + 4));
}

// Where the parts of a launch lie: part i of the launch belongs to instance inst_of(i) and is number
// i - part0(inst) of its cache.
struct DecodeTable {
  int32_t part_before[MAX_INST_PER_LAUNCH + 1];
  int32_t bk[MAX_INST_PER_LAUNCH];
  int64_t row0[MAX_INST_PER_LAUNCH];
  int32_t n;
  __device__ int inst_of(int i) const {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (part_before[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
  }
  __device__ int part0(int li) const { return part_before[li]; }
  __device__ int parts(int li) const { return part_before[li + 1] - part_before[li]; }
  __device__ int part_rows(int li) const { return even_rows(bk[li], parts(li)); }
  __device__ int rows(int li) const { return bk[li]; }
  __device__ int64_t first(int li) const { return row0[li]; }
};
struct DecodeUniform {
  UniformInst u;
  int32_t n_parts, rows_per_part;      // of every cache
  __device__ int inst_of(int i) const { return i / n_parts; }
  __device__ int part0(int li) const { return li * n_parts; }
  __device__ int parts(int) const { return n_parts; }
  __device__ int part_rows(int) const { return rows_per_part; }
  __device__ int rows(int li) const { return u.rows(li); }
  __device__ int64_t first(int li) const { return u.first(li); }
};

// A value and its sum over lanes that differ in BIT (16 or 32): the two halves of a register pair change places
// so that one addition serves both registers (sum2), or both copies of one (sum1, max1).
template <int BIT>
__device__ __forceinline__ void swap_halves(float& x, float& y) {
  if constexpr (BIT == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
  } else if constexpr (BIT == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
  }
}
// `BIT` 8 is a rotation within 16 lanes.
template <int BIT>
__device__ __forceinline__ float sum1(float x) {
  if constexpr (BIT == 8) return x + lane_select<0x128>(x);
  float y = x;
  swap_halves<BIT>(x, y);
  return x + y;
}
template <int BIT>
__device__ __forceinline__ float max1(float x) {
  if constexpr (BIT == 8) return fmaxf(x, lane_select<0x128>(x));
  float y = x;
  swap_halves<BIT>(x, y);
  return fmaxf(x, y);
}
// The first N values summed over the lanes that differ in BIT: lanes without it keep the first half, lanes with it the second.
template <int BIT, int N, int NV>
__device__ __forceinline__ void sum_halves(float (&x)[NV], int lane) {
  if constexpr (BIT == 8) {
    reduce_step<0x128, 8, N>(x, lane);
  } else {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      float y = x[i + N / 2];
      swap_halves<BIT>(x[i], y);
      x[i] += y;
    }
  }
}

// The parts of a split cache: part p of column x of a launch has sums[p][x][GB][d] and, per query head, the two
// words marks[p][x][GB][2]: the launch's nonce with M, and with Z.
struct PartArea {
  unsigned long long* marks;
  float* sums;
  uint32_t nonce;                    // a number that no other recent launch of the process has
};

// Written through to the device's memory, and read from there: whole caches need not be written back or dropped for it.
__device__ __forceinline__ void store_pair(void* p, uint32_t a, uint32_t b) {
  __hip_atomic_store(static_cast<unsigned long long*>(p), (unsigned long long)b << 32 | a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint2 load_pair(const void* p) {
  const unsigned long long v = __hip_atomic_load(static_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Folds the S parts of column blockIdx.x of a cache, in part order, if all of them are finished.  Every part says
// so with its marks after its sums have been written, and then looks at the marks of all: the last to do so
// finds them all (should two find that, both write the same values).  Whoever finds all of them set clears
// them, so that a captured launch, which has the same nonce every time, never finds its own old marks; whatever else
// lies in the workspace is taken for an unfinished part.  It takes four trips to memory, 3 to 4 us (a launch of its own
// took 4 to 6 and what it takes to enqueue it; fences instead of write-through took 7, and 700 us in a call of
// 4500 parts).
template <int GB>
__device__ void merge_parts(const PartArea& pa, int p0, int S, int d, float* sm, float* out, int heads) {
  const int tid = threadIdx.x, columns = gridDim.x;
  float* sm_m = sm;                        // [S][GB]
  float* sm_z = sm + S * GB;               // [S][GB]
  bool all = true;
  for (int i = tid; i < S * GB; i += DEC_THREADS) {
    const unsigned long long* mark = pa.marks + (((size_t)(p0 + i / GB) * columns + blockIdx.x) * GB + i % GB) * 2;
    const uint2 m = load_pair(mark), z = load_pair(mark + 1);
    all = all && m.x == pa.nonce && z.x == pa.nonce;
    sm_m[i] = __uint_as_float(m.y);
    sm_z[i] = __uint_as_float(z.y);
  }
  if (!__syncthreads_and(all)) return;
  for (int i = tid; i < S * GB; i += DEC_THREADS) {
    unsigned long long* mark = pa.marks + (((size_t)(p0 + i / GB) * columns + blockIdx.x) * GB + i % GB) * 2;
    store_pair(mark, 0, 0);
    store_pair(mark + 1, 0, 0);
  }
  const size_t part_floats = (size_t)columns * GB * d;
  const float* sums = pa.sums + ((size_t)p0 * columns + blockIdx.x) * GB * d;
  const int pairs = d / 2;
  for (int e = tid; e < GB * pairs; e += DEC_THREADS) {
    const int g = e / pairs, c = (e - g * pairs) * 2;
    if (g >= heads) break;
    float M = DEC_NEG_BIG;
    for (int s = 0; s < S; ++s) M = fmaxf(M, sm_m[s * GB + g]);
    float Z = 0.f, O0 = 0.f, O1 = 0.f;
#pragma unroll 8
    for (int s = 0; s < S; ++s) {
      const float w = __builtin_amdgcn_exp2f(sm_m[s * GB + g] - M);
      const uint2 o = load_pair(sums + s * part_floats + (size_t)g * d + c);
      Z = fmaf(sm_z[s * GB + g], w, Z);
      O0 = fmaf(__uint_as_float(o.x), w, O0);
      O1 = fmaf(__uint_as_float(o.y), w, O1);
    }
    out[(size_t)g * d + c] = O0 / Z;
    out[(size_t)g * d + c + 1] = O1 / Z;
  }
}

// A workgroup works on part blockIdx.y for the query-head batch blockIdx.x: a cache in one part writes `out`;
// one of several parts leaves its unnormalised sums, maxima and sums of weights to merge_parts.
template <int GB, bool SHARED, typename T, int PP, typename TAB>
__global__ __launch_bounds__(DEC_THREADS) void decode_kernel(int Hq, int Hkv, int d, float scale2, int inst0,
                                                             TAB tab, const T* __restrict__ q,
                                                             const T* __restrict__ kc, const T* __restrict__ vc,
                                                             float* __restrict__ out, PartArea pa) {
  using Piece = typename PieceOf<T>::type;
  constexpr int RP = PP < 16 ? PP : 16;    // lanes among which the logits are left
  constexpr int ROWS = sizeof(T) == 4 || GB >= 4 ? 4 : 8;         // rows per lane group and turn
  constexpr int SETS = ROWS * GB > RP ? ROWS * GB / RP : 1;        // logits per lane
  constexpr int NV = ROWS * GB / SETS;     // values per set: index u * GB + g for rows u of the set
  constexpr int PER = RP / NV;             // lanes that hold the same value
  constexpr int RSET = ROWS / SETS;        // rows per set
  constexpr int GROUPS = DEC_THREADS / PP, WAVES = DEC_WAVES;
  static_assert(RSET * GB == NV, "");
  extern __shared__ __align__(16) float sm[];
  float* sm_acc = sm;                      // [WAVES][GB][d]
  float* sm_m = sm + (size_t)WAVES * GB * d;       // [WAVES][GB]
  float* sm_z = sm_m + WAVES * GB;         // [WAVES][GB]
  const int G = Hq / Hkv, nbatch = (G + GB - 1) / GB;
  const int head = blockIdx.x / nbatch, g0 = (blockIdx.x % nbatch) * GB;
  const int li = tab.inst_of(blockIdx.y), part = blockIdx.y - tab.part0(li), inst = inst0 + li;
  const int cache_rows = tab.rows(li), rows_per_part = tab.part_rows(li), start = part * rows_per_part;
  const int bk = min(rows_per_part, cache_rows - start);          // rows of this part
  const int tid = threadIdx.x, lane = tid & 63;
  const int dc = tid % PP, ks = tid / PP;
  const bool active = dc * 8 < d;
  const int64_t first_row = tab.first(li) + (int64_t)head * cache_rows + start;
  const T* K = kc + first_row * d + dc * 8;
  const T* V = vc + first_row * d + dc * 8;

  Piece qv[GB];                            // this lane's 8 elements of every query of the batch
  float acc[GB * 8];
#pragma unroll
  for (int i = 0; i < GB * 8; ++i) acc[i] = 0.f;
#pragma unroll
  for (int g = 0; g < GB; ++g) {
    clear8(qv[g]);
    if (active && g0 + g < G) fetch8(q + ((size_t)inst * Hq + (size_t)head * G + g0 + g) * d + dc * 8, qv[g]);
  }
  // a value from lane N of the group, for every lane of it
  auto from = [&](float y, auto N) {
    constexpr int n = decltype(N)::value;
    if constexpr (RP == 16) return lane_select<0x150 + n>(y);
    else return lane & 8 ? lane_select<0x150 + 8 + n>(y) : lane_select<0x150 + n>(y);
  };
  const int my_u = (lane & (RP - 1)) / PER / GB;                  // the row within a set whose logit this lane holds
  float m = DEC_NEG_BIG, z = 0.f;          // of this lane's head: running maximum of the group's rows; sum over the rows whose logits it held

  for (int t0 = 0; t0 < bk; t0 += GROUPS * ROWS) {
    Piece kp[ROWS], vp[ROWS];              // rows t0 + ks + GROUPS * u; beyond the part: zeros
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int j = t0 + ks + GROUPS * u;
      clear8(kp[u]);
      clear8(vp[u]);
      if (active && j < bk) {
        fetch_row<!SHARED>(K + (size_t)j * d, kp[u]);
        fetch_row<!SHARED>(V + (size_t)j * d, vp[u]);
      }
    }
    float x[SETS], m_new = m;
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
      float v[NV];
#pragma unroll
      for (int u = 0; u < RSET; ++u)
#pragma unroll
        for (int g = 0; g < GB; ++g) {
          v[u * GB + g] = dot8(qv[g], kp[s * RSET + u]);
          if (PP == 32) v[u * GB + g] += __shfl_xor(v[u * GB + g], 16);
        }
      x[s] = group_reduce<RP, NV>(v, lane) * scale2;
      if (t0 + ks + GROUPS * (s * RSET + my_u) >= bk) x[s] = -INFINITY;
      m_new = fmaxf(m_new, x[s]);
    }
    // the maximum over the lanes that hold the same head's logits
    if constexpr (RP == 16) {
      if constexpr (GB * PER <= 2) m_new = fmaxf(m_new, lane_select<0x122>(m_new));   // rotate by 2
      if constexpr (GB * PER <= 4) m_new = fmaxf(m_new, lane_select<0x124>(m_new));   // by 4
      if constexpr (GB * PER <= 8) m_new = fmaxf(m_new, lane_select<0x128>(m_new));   // by 8
    } else {
      if constexpr (GB * PER == 1) m_new = fmaxf(m_new, lane_select<0xB1>(m_new));    // lane ^ 1
      if constexpr (GB * PER <= 2) m_new = fmaxf(m_new, lane_select<0x4E>(m_new));    // lane ^ 2
      if constexpr (GB * PER <= 4) m_new = fmaxf(m_new, lane_select<0x141>(lane_select<0x1B>(m_new)));   // lane ^ 3, ^ 7
    }
    const bool moved = m_new > m;
    const float a = __builtin_amdgcn_exp2f(m - m_new);
    float p[SETS];
    z *= a;
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
      p[s] = __builtin_amdgcn_exp2f(x[s] - m_new);
      z += p[s];
    }
    m = m_new;
    if (__any(moved))
      static_for<0, GB>([&](auto GI) {
        constexpr int g = decltype(GI)::value;
        const float ag = from(a, std::integral_constant<int, g * PER>{});
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[g * 8 + c] *= ag;
      });
    static_for<0, ROWS>([&](auto U) {
      constexpr int u = decltype(U)::value, s = u / RSET;
      float vf[8];
      widen8(vp[u], vf);
      static_for<0, GB>([&](auto GI) {
        constexpr int g = decltype(GI)::value;
        const float w = from(p[s], std::integral_constant<int, ((u % RSET) * GB + g) * PER>{});
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[g * 8 + c] = fmaf(w, vf[c], acc[g * 8 + c]);
      });
    });
  }
  // the head's sum over the lanes that held its logits
  if constexpr (RP == 16) {
    if constexpr (GB * PER <= 2) z += lane_select<0x122>(z);
    if constexpr (GB * PER <= 4) z += lane_select<0x124>(z);
    if constexpr (GB * PER <= 8) z += lane_select<0x128>(z);
  } else {
    if constexpr (GB * PER == 1) z += lane_select<0xB1>(z);
    if constexpr (GB * PER <= 2) z += lane_select<0x4E>(z);
    if constexpr (GB * PER <= 4) z += lane_select<0x141>(lane_select<0x1B>(z));
  }
  // merge the groups of the wave; a lane ends with values i0 .. i0+KEPT-1 of acc[g * 8 + c]
  float m_wave = max1<32>(m);
  if constexpr (PP <= 16) m_wave = max1<16>(m_wave);
  if constexpr (PP <= 8) m_wave = max1<8>(m_wave);
  const float a = __builtin_amdgcn_exp2f(m - m_wave);
  z = sum1<32>(z * a);
  if constexpr (PP <= 16) z = sum1<16>(z);
  if constexpr (PP <= 8) z = sum1<8>(z);
  static_for<0, GB>([&](auto GI) {
    constexpr int g = decltype(GI)::value;
    const float ag = from(a, std::integral_constant<int, g * PER>{});
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[g * 8 + c] *= ag;
  });
  constexpr int NA = GB * 8, KEPT = NA * PP / 64;
  sum_halves<32, NA>(acc, lane);
  if constexpr (PP <= 16) sum_halves<16, NA / 2>(acc, lane);
  if constexpr (PP <= 8) sum_halves<8, NA / 4>(acc, lane);
  const int i0 = (lane & 32 ? NA / 2 : 0) + (PP <= 16 && lane & 16 ? NA / 4 : 0) + (PP <= 8 && lane & 8 ? NA / 8 : 0);
  const int wave = tid >> 6;
  if (lane < GB * PER && lane % PER == 0) {
    sm_m[wave * GB + lane / PER] = m_wave;
    sm_z[wave * GB + lane / PER] = z;
  }
  if (active) {
#pragma unroll
    for (int i = 0; i < KEPT; ++i) sm_acc[((size_t)wave * GB + (i0 + i) / 8) * d + dc * 8 + (i0 + i) % 8] = acc[i];
  }
  __syncthreads();
  // merge the waves
  const bool whole = cache_rows <= rows_per_part;
  const int pairs = d / 2;
  float* out0 = out + ((size_t)inst * Hq + (size_t)head * G + g0) * d;
  const size_t part_slot = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * GB;
  for (int e = tid; e < GB * pairs; e += DEC_THREADS) {
    const int g = e / pairs, c = (e - g * pairs) * 2;
    float M = DEC_NEG_BIG;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) M = fmaxf(M, sm_m[w * GB + g]);
    float Z = 0.f, O0 = 0.f, O1 = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float wgt = __builtin_amdgcn_exp2f(sm_m[w * GB + g] - M);
      const float2 o = *reinterpret_cast<const float2*>(sm_acc + ((size_t)w * GB + g) * d + c);
      Z = fmaf(sm_z[w * GB + g], wgt, Z);
      O0 = fmaf(o.x, wgt, O0);
      O1 = fmaf(o.y, wgt, O1);
    }
    if (!whole) {
      store_pair(pa.sums + (part_slot + g) * d + c, __float_as_uint(O0), __float_as_uint(O1));
    } else if (g0 + g < G) {
      out0[(size_t)g * d + c] = O0 / Z;
      out0[(size_t)g * d + c + 1] = O1 / Z;
    }
  }
  if (whole) return;
  stores_done();
  __syncthreads();
  if (tid < GB) {
    float M = DEC_NEG_BIG, Z = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) M = fmaxf(M, sm_m[w * GB + tid]);
#pragma unroll
    for (int w = 0; w < WAVES; ++w) Z = fmaf(sm_z[w * GB + tid], __builtin_amdgcn_exp2f(sm_m[w * GB + tid] - M), Z);
    store_pair(pa.marks + (part_slot + tid) * 2, pa.nonce, __float_as_uint(M));
    store_pair(pa.marks + (part_slot + tid) * 2 + 1, pa.nonce, __float_as_uint(Z));
    stores_done();
  }
  __syncthreads();
  merge_parts<GB>(pa, tab.part0(li), tab.parts(li), d, sm, out0, G - g0);
}

// q_cache[inst][h][t][:] = q_step[inst][h][:], 16 bytes per thread
__global__ __launch_bounds__(256) void qcache_store_kernel(long long rows, int W, int t, int pieces,
                                                           const uint4* __restrict__ q_step,
                                                           uint4* __restrict__ q_cache) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= rows * pieces) return;
  const long long row = i / pieces;
  const int piece = (int)(i - row * pieces);
  q_cache[(row * W + t) * pieces + piece] = q_step[i];
}

struct DecodeCall {
  int Hq, Hkv, d, columns, head_batch;
  float scale2;
  const void *q, *kc, *vc;
  float* out;
  PartArea parts;
  hipStream_t st;
};

template <int GB, bool SHARED, typename T, int PP, typename TAB>
hipError_t launch_pp(const DecodeCall& c, int n_parts, int inst0, const TAB& tab) {
  const int merge = DEC_MOST_PARTS * GB * 2, sums = DEC_WAVES * GB * (c.d + 2);   // floats of the two uses of the LDS
  hipLaunchKernelGGL((decode_kernel<GB, SHARED, T, PP, TAB>), dim3(c.columns, n_parts), dim3(DEC_THREADS),
                     (c.parts.marks && merge > sums ? merge : sums) * sizeof(float), c.st, c.Hq, c.Hkv, c.d, c.scale2, inst0,
                     tab, static_cast<const T*>(c.q), static_cast<const T*>(c.kc), static_cast<const T*>(c.vc), c.out, c.parts);
  return hipGetLastError();
}

// lanes per row: the power of two (at least 8) that covers the row's d / 8 pieces
template <int GB, bool SHARED, typename T, typename TAB>
hipError_t launch_gb(const DecodeCall& c, int n_parts, int inst0, const TAB& tab) {
  if (c.d <= 64) return launch_pp<GB, SHARED, T, 8>(c, n_parts, inst0, tab);
  if (c.d <= 128) return launch_pp<GB, SHARED, T, 16>(c, n_parts, inst0, tab);
  return launch_pp<GB, SHARED, T, 32>(c, n_parts, inst0, tab);
}

// SHARED: several workgroups read the same rows (more query heads per KV head than one serves).
template <typename T, typename TAB>
hipError_t launch_for(const DecodeCall& c, int n_parts, int inst0, const TAB& tab) {
  if (c.head_batch == 1) return launch_gb<1, false, T>(c, n_parts, inst0, tab);
  if (c.head_batch == 2) return launch_gb<2, false, T>(c, n_parts, inst0, tab);
  if constexpr (sizeof(T) == 2) {
    if (c.head_batch == 4) return launch_gb<4, false, T>(c, n_parts, inst0, tab);
    return c.columns == c.Hkv ? launch_gb<8, false, T>(c, n_parts, inst0, tab) : launch_gb<8, true, T>(c, n_parts, inst0, tab);
  } else {
    return c.columns == c.Hkv ? launch_gb<4, false, T>(c, n_parts, inst0, tab) : launch_gb<4, true, T>(c, n_parts, inst0, tab);
  }
}

}  // namespace

// Query heads of a KV head that one workgroup serves: all of them up to 8 (fp32: 4, for the registers' sake), so that
// the rows are read once.  (8 heads over 2048 rows, 128 caches: two batches of 4
// took 50 us, one of 8 takes 41.)
int decode_head_batch(int Hq, int Hkv, int dtype) {
  const int G = Hq / Hkv, most = dtype == LAQ_BF16 ? 8 : 4;
  int gb = 1;
  while (gb < G && gb < most) gb *= 2;
  return gb;
}

static int decode_columns(int Hq, int Hkv, int dtype) {
  const int gb = decode_head_batch(Hq, Hkv, dtype);
  return Hkv * ((Hq / Hkv + gb - 1) / gb);
}
int decode_part_rows(int n, int L, int Hq, int Hkv, int dtype, const int32_t* budget) {
  return limit_of_parts(n, L, decode_columns(Hq, Hkv, dtype), budget);
}

// The area of the parts of a launch, in a workspace of any alignment: marks, then sums.
static size_t part_slots(long long parts, int Hq, int Hkv, int dtype) { return (size_t)parts * decode_columns(Hq, Hkv, dtype) * decode_head_batch(Hq, Hkv, dtype); }

// Bytes that hold the parts of any launch of a call (launches reuse the area; they are ordered on the stream), and of any
// other call of this shape whose caches are no longer: one workspace serves layers of different budgets.  A cache has at most a
// part for every DEC_PART_STEP rows and at most DEC_MOST_PARTS; and as evening parts out adds none, the caches of a call have no more than
// parts of the limit would be, one each and DEC_WORKGROUPS / columns in all beside those.  Each of the three bounds grows with every
// budget.  (The number itself does not: the length of a part goes in steps, so that 2048 rows can have fewer parts than 1535.)
size_t decode_partial_bytes(int n, int L, int Hq, int Hkv, int d, int dtype, const int32_t* budget) {
  const long long columns = decode_columns(Hq, Hkv, dtype);
  if (n * columns >= DEC_WHOLE_FROM || longest_cache(n, L, budget) <= DEC_PART_STEP) return 0;
  long long parts = 0, most = 0;
  for (int i = 0; i < n; ++i) {
    if (i % MAX_INST_PER_LAUNCH == 0) parts = 0;
    const int s = parts_of(budget[i] < L ? budget[i] : L, DEC_PART_STEP);
    parts += s < DEC_MOST_PARTS ? s : DEC_MOST_PARTS;
    if (parts > most) most = parts;
  }
  const long long by_rows = (n < MAX_INST_PER_LAUNCH ? n : MAX_INST_PER_LAUNCH) + DEC_WORKGROUPS / columns;
  return 8 + part_slots(most < by_rows ? most : by_rows, Hq, Hkv, dtype) * (2 * sizeof(unsigned long long) + d * sizeof(float));
}

hipError_t launch_decode(int n_inst, int L, int Hq, int Hkv, int d, int dtype, float scale2, int rows_per_part, const int32_t* budget,
                         const void* q, const void* kc, const void* vc, float* out, void* ws, hipStream_t st) {
  static std::atomic<uint32_t> launches{(uint32_t)(std::chrono::steady_clock::now().time_since_epoch().count() * 0x9E3779B97F4A7C15ull >> 32)};
  DecodeCall c{Hq, Hkv, d, decode_columns(Hq, Hkv, dtype), decode_head_batch(Hq, Hkv, dtype), scale2, q, kc, vc, out, {}, st};
  const auto launch = [&](int n_parts, int inst0, const auto& tab) {
    if (ws) {
      c.parts.marks = reinterpret_cast<unsigned long long*>((reinterpret_cast<uintptr_t>(ws) + 7) & ~(uintptr_t)7);
      c.parts.sums = reinterpret_cast<float*>(c.parts.marks + 2 * part_slots(n_parts, Hq, Hkv, dtype));
      do c.parts.nonce = launches.fetch_add(1); while (c.parts.nonce == 0);          // 0 is the cleared mark
    }
    return dtype == LAQ_BF16 ? launch_for<uint16_t>(c, n_parts, inst0, tab) : launch_for<float>(c, n_parts, inst0, tab);
  };
  int64_t row = 0;
  for (int i0 = 0; i0 < n_inst; i0 += MAX_INST_PER_LAUNCH) {
    const int n = n_inst - i0 < MAX_INST_PER_LAUNCH ? n_inst - i0 : MAX_INST_PER_LAUNCH;
    hipError_t e;
    if (const int bk = uniform_rows(L, budget, i0, n)) {
      const int parts = parts_of(bk, rows_per_part);
      const DecodeUniform tab{UniformInst{bk, row, (int64_t)Hkv * bk}, parts, even_rows(bk, parts)};
      row += n * tab.u.per_inst;
      e = launch(n * parts, i0, tab);
    } else {
      DecodeTable tab;
      tab.n = n;
      tab.part_before[0] = 0;
      for (int i = 0; i < n; ++i) {
        tab.bk[i] = budget[i0 + i] < L ? budget[i0 + i] : L;
        tab.row0[i] = row;
        tab.part_before[i + 1] = tab.part_before[i] + parts_of(tab.bk[i], rows_per_part);
        row += (int64_t)Hkv * tab.bk[i];
      }
      e = launch(tab.part_before[n], i0, tab);
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_qcache_store(long long rows, int W, int t, int row_bytes, const void* q_step, void* q_cache,
                               hipStream_t st) {
  const int pieces = row_bytes / 16;
  const long long total = rows * pieces;
  hipLaunchKernelGGL(qcache_store_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, rows, W, t, pieces,
                     static_cast<const uint4*>(q_step), static_cast<uint4*>(q_cache));
  return hipGetLastError();
}

}  // namespace laq
