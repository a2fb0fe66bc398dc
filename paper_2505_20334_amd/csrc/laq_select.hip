// Per-KV-head selection: the "ArgSort(...)[:B]" of Eq. 4 done as a radix select (no sort).
//
// One workgroup of 4, 8 or 16 waves ranks the prefix scores of one (instance, KV head).  Scores are mapped to
// order-preserving 32-bit keys, which live in registers for prefixes up to 32768 (longer ones re-read the
// scores from memory in every sweep).
//   1. A lower bound of the k-th largest key: the keys are cut into at least k groups (a thread's, or halves
//      or quarters of them); the k-th largest of the groups' maxima is such a bound, and only one key per
//      group is counted for it (by its 9, 10 or 11 leading bits -- two bins per thread; the bound is the lower edge of a bin).  Few more
//      than k keys are left above it.  (Short prefixes with many keys wanted: every key is a group.)
//   2. Long prefixes (more than 16 keys a thread): the quads of neighbouring keys that hold one above the bound go, in order, into a list
//      per wave, so that the sweeps that follow are over few keys.  Where a wave has more of them than its list holds, and for short
//      prefixes, these sweeps are over the registers.
//   3. The keys above the bound are counted by their distance from it, in as many bins up to the largest key, and the bin of
//      the k-th one is refined, as many bits at a time, until its keys are all wanted or so few (CANDIDATES)
//      that comparing all pairs tells the key T of the k-th largest and how many keys equal to T still
//      fit (ties go to the lower position).
//   4. A last sweep emits, in ascending position order, every key above T plus the first `want` keys equal to
//      T, then the `keep` window positions.
// What bounds it: latency -- loads, LDS adds and barriers of one workgroup per head -- and, for long prefixes, the instructions of one
// compute unit, most of which run once and are fetched cold.  The scores of a head
// crowd into few values of the leading bits, and LDS adds of many lanes to one word go one after the other
// (counting every key of a 32768-key head by its leading byte took 9 us of 25); so few keys are counted
// there, into COPIES histograms side by side, one per lane number modulo COPIES.
// With the lists, a test per wave instead of per element for the ends of the row, and the pooling in one piece of code per width: 8 heads x
// 30011 keys, 1024 of them, laq_evict 52.6 -> 46.6 us; 2048 heads x 32752 keys 4.12 -> 4.07 ms.  (Lists for 16 keys a thread and fewer
// cost 0.5 to 1 us: writing and reading them back takes longer than the sweeps they save.)
#include <type_traits>

#include "laq_internal.h"
#include "laq_pool.h"
#include "laq_rank.h"

namespace laq {

namespace {

constexpr int COPIES = 8;                  // histograms of the first pass
constexpr int CANDIDATES = 128;            // keys that are ranked by comparing all pairs

__device__ __forceinline__ float4 quad_of_lane(float4 x, int l) {
  return make_float4(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(x.x), l)), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x.y), l)),
                     __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x.z), l)), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x.w), l)));
}

// Sizes that follow from the threads of a workgroup: two bins per thread.
template <int THREADS> struct Sel {
  static constexpr int WAVES = THREADS / 64, BINS = 2 * THREADS;
  static constexpr int BITS = THREADS == 1024 ? 11 : THREADS == 512 ? 10 : 9;
  static_assert(BINS == 1 << BITS && WAVES <= 16, "");
  int first[BINS * COPIES];                // first pass: [bin][copy]; then the quads that hold keys above the bound, by wave
  static constexpr int QUADS_LISTED = BINS * COPIES / WAVES / 5 / 4 * 4;                 // per wave: uint4[], int[] (their first positions)
  int later[BINS];                         // the other passes
  uint32_t cand[CANDIDATES];
  int n_cand, over;                        // over: a wave has more quads than its list
  int wave_total[2][WAVES];
  int bin, above, count, top;              // result of a pass; top: the highest bin that is not empty
  uint32_t threshold;
  int equal_wanted;
};

// The bin (from the top) in which the `want`-th key lies, the number of keys above it and in it.  Ends
// behind a barrier.
template <int C, int THREADS>
__device__ __forceinline__ void find_bin(Sel<THREADS>& sh, const int* hist, int want, int tid) {
  const int lane = tid & 63, wave = tid >> 6, b = Sel<THREADS>::BINS - 2 - 2 * tid;   // this thread: bins b + 1, then b
  int h0, h1;
  if constexpr (C == 1) {
    const int2 v = *reinterpret_cast<const int2*>(hist + b);
    h0 = v.y;
    h1 = v.x;
  } else {
    h0 = h1 = 0;
#pragma unroll
    for (int c = 0; c < C; c += 4) {
      const int4 lo = *reinterpret_cast<const int4*>(hist + b * C + c), hi = *reinterpret_cast<const int4*>(hist + (b + 1) * C + c);
      h1 += lo.x + lo.y + lo.z + lo.w;
      h0 += hi.x + hi.y + hi.z + hi.w;
    }
  }
  const int upto = wave_scan(h0 + h1);
  if (lane == 63) sh.wave_total[0][wave] = upto;
  __syncthreads();
  int before = lane < wave ? sh.wave_total[0][lane] : 0;                // (at most 16 waves)
  before = __builtin_amdgcn_readlane(wave_scan(before), 15);
  const int incl = before + upto, excl = incl - h0 - h1;
  if (excl == 0 && incl > 0) sh.top = h0 > 0 ? b + 1 : b;
  if (excl < want && want <= incl) {
    const bool second = excl + h0 < want;
    sh.bin = second ? b : b + 1;
    sh.above = second ? excl + h0 : excl;
    sh.count = second ? h1 : h0;
  }
  __syncthreads();
}

// ITEMS > 0: keys of the wave's segment are held in ITEMS registers per lane.
// ITEMS == 0: keys are recomputed from memory on every sweep (any prefix length).
// QUADS (scores that are final: no pooling here): register 4q + c of a lane holds position
// seg0 + 256 q + 4 lane + c - shift, where shift (0 .. 3) is how far the row starts behind a 16-byte boundary,
// fetched with one load per q.  Otherwise register i holds position seg0 + 64 i + lane.
// FIN = PoolArgs, FinishArgs: the scores are raw ones, see there; NoFinish: nothing of that.
struct NoFinish {};
template <int THREADS, int ITEMS, bool QUADS, typename TAB, typename FIN>
__global__ __launch_bounds__(THREADS, 4) void select_kernel(int Hkv, int L, int keep, int pool, bool avg,
                                                             const float* __restrict__ scores, TAB tab,
                                                             int inst0, int32_t* __restrict__ idx, FIN fin) {
  constexpr bool FINISH = std::is_same<FIN, FinishArgs>::value, POOLS = std::is_base_of<PoolArgs, FIN>::value;
  static_assert(!POOLS || QUADS, "four neighbours per lane");
  __shared__ __align__(16) Sel<THREADS> sh;
  constexpr int BINS = Sel<THREADS>::BINS, BITS = Sel<THREADS>::BITS, TOP = 32 - BITS;

  const int head = blockIdx.x, li = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int P = L - keep, half = (pool - 1) / 2;
  const int bk = tab.rows(li);
  const int ksel = bk - keep;
  const float* s = scores + ((size_t)(inst0 + li) * Hkv + head) * L;
  int32_t* out = idx + (tab.first(li) + (int64_t)head * bk);

  for (int w = tid; w < keep; w += THREADS) out[ksel + w] = P + w;
  const bool all = ksel >= P, ranked = ksel > 0 && !all;
  if (all)
    for (int j = tid; j < P; j += THREADS) out[j] = j;
  if constexpr (!POOLS) {
    if (!ranked) return;
  } else if (fin.pooled != scores) {
    float* pooled = fin.pooled + ((size_t)(inst0 + li) * Hkv + head) * L;
    for (int w = tid; w < keep; w += THREADS) pooled[P + w] = s[P + w];
  }

  constexpr int UNROLL = ITEMS > 0 ? ITEMS : 1;     // register-resident keys: full unrolling; memory path: none
  const int items = (ITEMS > 0) ? ITEMS : (P + THREADS - 1) / THREADS;
  const int shift = QUADS ? (int)((reinterpret_cast<uintptr_t>(s) >> 2) & 3) : 0;
  const int seg0 = wave * items * 64 - shift;       // first position of this wave's segment

  static_assert(!QUADS || (ITEMS > 0 && ITEMS % 4 == 0), "four registers per load");
  uint32_t key[ITEMS > 0 ? ITEMS : 1];
  if constexpr (QUADS) {
    constexpr int NQ = ITEMS / 4;
    float4 v[NQ];
    // positions pos .. pos + 3 of the prefix, 0 for those that are not in it
    auto quad_at = [&](int pos) {
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
      if (pos >= 0 && pos + 3 < P) {
        x = *reinterpret_cast<const float4*>(s + pos);
      } else {
        if (pos >= 0 && pos < P) x.x = s[pos];
        if (pos + 1 >= 0 && pos + 1 < P) x.y = s[pos + 1];
        if (pos + 2 >= 0 && pos + 2 < P) x.z = s[pos + 2];
        if (pos + 3 >= 0 && pos + 3 < P) x.w = s[pos + 3];
      }
      return x;
    };
    // The quad lies inside the prefix.  Most of a row's do: with several per lane, one test for a wave's 64.
    auto inside = [&](int q4) {
      const int first = seg0 + q4 * 256 + (NQ == 1 ? lane * 4 : 0);
      return first >= 0 && first + (NQ == 1 ? 4 : 256) <= P;
    };
#pragma unroll
    for (int q4 = 0; q4 < NQ; ++q4) {
      if (inside(q4)) v[q4] = *reinterpret_cast<const float4*>(s + (seg0 + q4 * 256 + lane * 4));
      else v[q4] = quad_at(seg0 + q4 * 256 + lane * 4);
    }
    if constexpr (POOLS) {
      if (fin.half > 0) {
        float* pooled = fin.pooled + ((size_t)(inst0 + li) * Hkv + head) * L;
        // The quads around a lane's own come from its neighbours' registers; around the first and the last of the wave's
        // from memory.
        const float4 none = make_float4(0.f, 0.f, 0.f, 0.f);
        const bool wide = fin.half > 4;
        float4 before1 = none, before2 = none, after1 = none, after2 = none;
        if (lane == 0 || lane == 63) {
          const int end = seg0 + NQ * 256;
          before1 = quad_at(lane == 0 ? seg0 - 4 : end);
          if (wide) before2 = quad_at(lane == 0 ? seg0 - 8 : end + 4);
          after1 = before1;
          after2 = before2;
        }
        for_half(fin.half, [&](auto h) {
          constexpr int H = decltype(h)::value;
#pragma unroll
          for (int q4 = 0; q4 < NQ; ++q4) {
            const int pos = seg0 + q4 * 256 + lane * 4;
            const float4 own = v[q4], next = v[q4 + 1 < NQ ? q4 + 1 : 0];
            const float4 n1 = q4 + 1 < NQ ? quad_of_lane(next, 0) : after1, n2 = q4 + 1 < NQ ? quad_of_lane(next, 1) : after2;
            const float4 r = pool_quad_of<H>(own, before1, before2, n1, n2, fin.avg != 0);
            before1 = quad_of_lane(own, 63);
            if (H > 4) before2 = quad_of_lane(own, 62);
            if (inside(q4)) {
              *reinterpret_cast<float4*>(pooled + pos) = r;
              v[q4] = r;
            } else {
              float* e = &v[q4].x;
              const float* x = &r.x;
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if (pos + c >= 0 && pos + c < P) {
                  pooled[pos + c] = x[c];
                  e[c] = x[c];
                }
            }
          }
        });
      }
    }
#pragma unroll
    for (int i = tid * 4; i < BINS * COPIES; i += THREADS * 4) *reinterpret_cast<int4*>(sh.first + i) = make_int4(0, 0, 0, 0);
#pragma unroll
    for (int q4 = 0; q4 < NQ; ++q4) {
      const int pos = seg0 + q4 * 256 + lane * 4;
      key[4 * q4] = max(order_key(v[q4].x), 1u);
      key[4 * q4 + 1] = max(order_key(v[q4].y), 1u);
      key[4 * q4 + 2] = max(order_key(v[q4].z), 1u);
      key[4 * q4 + 3] = max(order_key(v[q4].w), 1u);
      if (!inside(q4)) {                   // positions outside the prefix rank below every score, -inf too:
#pragma unroll
        for (int c = 0; c < 4; ++c)        // those before it would come first among equals
          if (pos + c < 0 || pos + c >= P) key[4 * q4 + c] = 0u;
      }
    }
  } else {
    for (int i = tid * 4; i < BINS * COPIES; i += THREADS * 4) *reinterpret_cast<int4*>(sh.first + i) = make_int4(0, 0, 0, 0);
    if (ITEMS > 0) {
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int pos = seg0 + i * 64 + lane;
        key[i] = (pos < P) ? order_key(pool_window(s, pos, P, half, avg)) : 0u;
      }
    }
  }
  if (POOLS ? ranked : true) {
  auto key_of = [&](int i) -> uint32_t {
    if (ITEMS > 0) return key[i];
    const int pos = seg0 + i * 64 + lane;
    return (pos < P) ? order_key(pool_window(s, pos, P, half, avg)) : 0u;
  };
  *reinterpret_cast<int2*>(sh.later + 2 * tid) = make_int2(0, 0);
  if (tid < CANDIDATES) sh.cand[tid] = 0;
  if (tid == 0) sh.n_cand = sh.over = 0;
  __syncthreads();

  // ---- 1. a lower bound of the ksel-th largest key ----
  {
    int* hist = sh.first + (lane & (COPIES - 1));
    // (groups of ITEMS, ITEMS / 2 or ITEMS / 4 keys: at least P / ITEMS, twice, four times as many of them hold keys)
    const int groups = ITEMS > 0 ? P / ITEMS : 0;
    if (ITEMS >= 4 && ksel <= 4 * groups) {
      constexpr int Q = ITEMS >= 4 ? ITEMS / 4 : 1;
      uint32_t m[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        m[q] = key_of(q * Q);
#pragma unroll
        for (int i = 1; i < Q; ++i) m[q] = max(m[q], key_of(q * Q + i));
      }
      m[0] = ksel > 2 * groups ? m[0] : max(m[0], m[1]);
      m[2] = ksel > 2 * groups ? m[2] : max(m[2], m[3]);
      if (ksel <= groups) {
        atomicAdd(&hist[(max(m[0], m[2]) >> TOP) * COPIES], 1);
      } else {
        atomicAdd(&hist[(m[0] >> TOP) * COPIES], 1);
        atomicAdd(&hist[(m[2] >> TOP) * COPIES], 1);
        if (ksel > 2 * groups) {
          atomicAdd(&hist[(m[1] >> TOP) * COPIES], 1);
          atomicAdd(&hist[(m[3] >> TOP) * COPIES], 1);
        }
      }
    } else {
#pragma unroll UNROLL
      for (int i = 0; i < items; ++i) atomicAdd(&hist[(key_of(i) >> TOP) * COPIES], 1);
    }
    __syncthreads();
  }
  find_bin<COPIES, THREADS>(sh, sh.first, ksel, tid);
  // ---- 2. the quads with a key from the bound on, in ascending order, into the wave's list ----
  const uint32_t bound = (uint32_t)sh.bin << TOP;
  constexpr int LIST = Sel<THREADS>::QUADS_LISTED;
  constexpr bool LISTS = QUADS && ITEMS > 16;
  uint4* const quads = reinterpret_cast<uint4*>(sh.first + wave * (BINS * COPIES / Sel<THREADS>::WAVES));   // (the counts there are read)
  int* const quad_pos = reinterpret_cast<int*>(quads + LIST);
  int listed = 0;
  bool fits = false;
  if constexpr (LISTS) {
#pragma unroll
    for (int q4 = 0; q4 < ITEMS / 4; ++q4) {
      const uint32_t *k = key + 4 * q4;
      const bool in = max(max(k[0], k[1]), max(k[2], k[3])) >= bound;
      const uint64_t some = __ballot(in);
      const int slot = listed + lanes_below(some);
      if (in && slot < LIST) {
        quads[slot] = make_uint4(k[0], k[1], k[2], k[3]);
        quad_pos[slot] = seg0 + q4 * 256 + lane * 4;
      }
      listed += __popcll(some);
    }
    if (listed > LIST && lane == 0) sh.over = 1;
    __syncthreads();
    fits = sh.over == 0;                   // (else the best keys of a row crowd in one wave's part: the registers are swept again)
  }
  // f(key) for all keys from the bound on (and others): of the list, or of the registers / of memory
  auto sweep_list = [&](auto f) {
    for (int e = lane; e < listed; e += 64) {
      const uint4 k = quads[e];
      f(k.x);
      f(k.y);
      f(k.z);
      f(k.w);
    }
  };
  auto sweep_all = [&](auto f) {
    constexpr int EACH = ITEMS > 0 ? ITEMS : 1;
#pragma unroll EACH
    for (int i = 0; i < items; ++i) f(key_of(i));
  };
  // ---- 3. the key T of the ksel-th largest score and how many keys equal to it are taken ----
  uint32_t T;
  int want;
  auto find_threshold = [&](auto sweep) {
    // keys base .. base + width - 1 (width <= BINS << low): `want` of them are taken, and all above
    uint32_t base = bound;
    uint64_t width = (uint64_t)(sh.top - sh.bin + 1) << TOP;
    int low = TOP - BITS + (32 - __clz(sh.top - sh.bin)), count;
    want = ksel;
#pragma unroll 1
    for (int pass = 0;; ++pass) {
      int* hist = sh.later;
      if (pass > 0) {
        *reinterpret_cast<int2*>(hist + 2 * tid) = make_int2(0, 0);
        __syncthreads();
      }
      sweep([&](uint32_t kv) {
        const uint32_t d = kv - base;
        if (kv >= base && d < width) atomicAdd(&hist[d >> low], 1);
      });
      __syncthreads();
      find_bin<1, THREADS>(sh, hist, want, tid);
      base += (uint32_t)sh.bin << low;
      width = 1ull << low;
      count = sh.count;
      want -= sh.above;
      if (count == want || count <= CANDIDATES || low == 0) break;
      low = max(low - BITS, 0);
    }
    T = base;                              // width 1: the key itself
    if (count == want) {                   // all of them: everything from T on
      T -= 1;
      want = 0;
    } else if (width > 1) {
      sweep([&](uint32_t kv) {
        if (kv >= base && kv - base < width) sh.cand[atomicAdd(&sh.n_cand, 1)] = kv;
      });
      __syncthreads();
      if (tid < count) {
        const uint32_t mine = sh.cand[tid];
        int gt = 0, eq = 0;
        for (int j = 0; j < count; j += 4) {
          const uint4 c = *reinterpret_cast<const uint4*>(sh.cand + j);   // (zeros beyond count)
          gt += (c.x > mine) + (c.y > mine) + (c.z > mine) + (c.w > mine);
          eq += (c.x == mine) + (c.y == mine) + (c.z == mine) + (c.w == mine);
        }
        if (gt < want && want <= gt + eq) {  // (equal candidates write the same values)
          sh.threshold = mine;
          sh.equal_wanted = want - gt;
        }
      }
      __syncthreads();
      T = sh.threshold;
      want = sh.equal_wanted;
    }
  };

  // ---- 4. emission in ascending position order ----
  // the wave's numbers of keys above T and equal to it -> those of the waves before
  int run_gt, run_eq;
  auto before_wave = [&](int wg, int we) {
    if (lane == 0) { sh.wave_total[0][wave] = wg; sh.wave_total[1][wave] = we; }
    __syncthreads();
    run_gt = lane < wave ? sh.wave_total[0][lane] : 0, run_eq = lane < wave ? sh.wave_total[1][lane] : 0;
    run_gt = __builtin_amdgcn_readlane(wave_scan(run_gt), 15);
    run_eq = __builtin_amdgcn_readlane(wave_scan(run_eq), 15);
  };
  // four consecutive positions per lane: ascending = (lane, c): before a lane's four come those of the lower lanes
  auto emit_quads = [&](const uint32_t (&k)[4], int pos) {
    uint64_t mg[4], me[4], some = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      mg[c] = __ballot(k[c] > T);
      me[c] = __ballot(k[c] == T);
      some |= mg[c] | me[c];
    }
    if (some == 0) return;                 // (the same in every lane)
    int g_before = run_gt, e_before = run_eq;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      g_before += lanes_below(mg[c]);
      e_before += lanes_below(me[c]);
      run_gt += __popcll(mg[c]);
      run_eq += __popcll(me[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const bool gt = k[c] > T, eq = k[c] == T;
      if (gt || (eq && e_before < want)) out[g_before + min(e_before, want)] = pos + c;
      g_before += gt;
      e_before += eq;
    }
  };
  if constexpr (LISTS) {
    if (fits) {
      find_threshold(sweep_list);
      int wg = 0, we = 0;
      for (int e0 = 0; e0 < listed; e0 += 64) {
        const bool have = e0 + lane < listed;
        const uint4 k = quads[have ? e0 + lane : 0];
        wg += __popcll(__ballot(have && k.x > T)) + __popcll(__ballot(have && k.y > T)) + __popcll(__ballot(have && k.z > T)) +
              __popcll(__ballot(have && k.w > T));
        we += __popcll(__ballot(have && k.x == T)) + __popcll(__ballot(have && k.y == T)) + __popcll(__ballot(have && k.z == T)) +
              __popcll(__ballot(have && k.w == T));
      }
      before_wave(wg, we);
      for (int e0 = 0; e0 < listed; e0 += 64) {
        const bool have = e0 + lane < listed;
        const uint4 q = quads[have ? e0 + lane : 0];
        const uint32_t k[4] = {have ? q.x : 0u, have ? q.y : 0u, have ? q.z : 0u, have ? q.w : 0u};   // (T > 0 or no equal is wanted)
        emit_quads(k, quad_pos[have ? e0 + lane : 0]);
      }
    }
  }
  if (!fits) {
    find_threshold(sweep_all);
    int wg = 0, we = 0;
#pragma unroll UNROLL
    for (int i = 0; i < items; ++i) {
      const uint32_t kv = key_of(i);
      wg += __popcll(__ballot(kv > T));
      we += __popcll(__ballot(kv == T));
    }
    before_wave(wg, we);
    if constexpr (ITEMS > 16) asm volatile("" : "+v"(T));                // (else the comparisons above are kept, in 4 * ITEMS registers)
    if constexpr (QUADS) {
#pragma unroll
      for (int q4 = 0; q4 < ITEMS / 4; ++q4) {
        const uint32_t k[4] = {key[4 * q4], key[4 * q4 + 1], key[4 * q4 + 2], key[4 * q4 + 3]};
        emit_quads(k, seg0 + q4 * 256 + lane * 4);
      }
    } else {
#pragma unroll UNROLL
      for (int i = 0; i < items; ++i) {
        const uint32_t kv = key_of(i);
        const bool gt = kv > T, eq = kv == T;
        const uint64_t mg = __ballot(gt), me = __ballot(eq);
        if ((mg | me) == 0) continue;
        const int g_before = run_gt + lanes_below(mg);
        const int e_before = run_eq + lanes_below(me);
        if (gt || (eq && e_before < want)) out[g_before + min(e_before, want)] = seg0 + i * 64 + lane;
        run_gt += __popcll(mg);
        run_eq += __popcll(me);
      }
    }
  }
  }
  if constexpr (FINISH) {
    // ---- gather: this workgroup's own list, complete behind the barrier ----
    __syncthreads();
    gather_rows<THREADS>(fin, inst0 + li, head, bk, tab.first(li) + (int64_t)head * bk, [&](int r) { return out[r]; });
  }
}

template <int THREADS, int ITEMS, bool QUADS, typename TAB, typename FIN>
hipError_t launch_one(int n_inst, int inst0, int Hkv, int L, int keep, int pool, bool avg, const float* scores,
                      const TAB& tab, int32_t* idx, const FIN& fin, hipStream_t st) {
  hipLaunchKernelGGL((select_kernel<THREADS, ITEMS, QUADS, TAB, FIN>), dim3(Hkv, n_inst), dim3(THREADS), 0, st, Hkv, L, keep, pool,
                     avg, scores, tab, inst0, idx, fin);
  return hipGetLastError();
}

// Score-free list (Sec. 2.1, StreamingLLM form): row = 0 .. s-1, then the Bk - s most recent
// positions, s = min(n_sink, Bk).  One workgroup per (KV head, instance).
__global__ __launch_bounds__(256) void sink_recent_kernel(int Hkv, int L, int n_sink, InstTable tab,
                                                          int32_t* __restrict__ idx) {
  const int head = blockIdx.x, li = blockIdx.y;
  const int bk = tab.bk[li];
  const int s = min(n_sink, bk);
  const int shift = L - bk;                 // recent entry at list slot t sits at position t + (L - Bk)
  int32_t* out = idx + (tab.row0[li] + (int64_t)head * bk);
  for (int t = threadIdx.x; t < bk; t += 256) out[t] = t < s ? t : t + shift;
}

template <typename TAB, typename FIN>
hipError_t launch_for(int n_inst, int inst0, int Hkv, int L, int keep, int pool, bool avg, const float* scores, const TAB& tab,
                      int32_t* idx, const FIN& fin, hipStream_t st) {
  // The fewest registers that hold the prefix.
  // With many heads in the launch, small workgroups of which several share a compute unit: while one
  // waits at a barrier or for its scores, another one works.
  const int most = L - keep + (pool == 1 ? row_shift(scores, L) : 0);
  auto at = [&](auto launch) { return launch(n_inst, inst0, Hkv, L, keep, pool, avg, scores, tab, idx, fin, st); };
  if (pool == 1) {
    if ((long long)Hkv * n_inst >= SELECT_MANY_HEADS) {
      if (most <= 256 * 8) return at(launch_one<256, 8, true, TAB, FIN>);
      if (most <= 256 * 32) return at(launch_one<256, 32, true, TAB, FIN>);
      if constexpr (std::is_same<FIN, NoFinish>::value)
        if (most <= 512 * 64) return at(launch_one<512, 64, true, TAB, FIN>);
    }
    if (most <= 1024 * 4) return at(launch_one<1024, 4, true, TAB, FIN>);
    if (most <= 1024 * 8) return at(launch_one<1024, 8, true, TAB, FIN>);
    if (most <= 1024 * 16) return at(launch_one<1024, 16, true, TAB, FIN>);
    if (most <= 1024 * 32) return at(launch_one<1024, 32, true, TAB, FIN>);
  }
  if constexpr (std::is_same<FIN, NoFinish>::value) {
    if (pool == 1) return at(launch_one<1024, 0, false, TAB, FIN>);
    if (most <= 1024 * 2) return at(launch_one<1024, 2, false, TAB, FIN>);
    if (most <= 1024 * 8) return at(launch_one<1024, 8, false, TAB, FIN>);
    if (most <= 1024 * 32) return at(launch_one<1024, 32, false, TAB, FIN>);
    return at(launch_one<1024, 0, false, TAB, FIN>);
  }
  return hipErrorInvalidValue;             // (the callers pool longer prefixes before)
}
static_assert(SELECT_POOL_MAX_KEYS == 1024 * 32, "");

template <typename TAB>
hipError_t finish_for(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const TAB& tab, int32_t* idx,
                      const FinishArgs& fin, hipStream_t st) {
  const int most = L - keep + row_shift(raw, L);
  auto at = [&](auto launch) { return launch(n_inst, inst0, Hkv, L, keep, 1, false, raw, tab, idx, fin, st); };
  if (most <= 256 * 8) return at(launch_one<256, 8, true, TAB, FinishArgs>);
  if (most <= 1024 * 4) return at(launch_one<1024, 4, true, TAB, FinishArgs>);
  if (most <= 1024 * 8) return at(launch_one<1024, 8, true, TAB, FinishArgs>);
  return at(launch_one<1024, 16, true, TAB, FinishArgs>);
}
static_assert(FINISH_MAX_KEYS == 1024 * 16, "the largest variant above; finish_wanted() counts the shift of the rows too");

}  // namespace

hipError_t launch_sink_recent(int n_inst, int Hkv, int L, int n_sink, const InstTable& tab, int32_t* idx,
                              hipStream_t st) {
  hipLaunchKernelGGL(sink_recent_kernel, dim3(Hkv, n_inst), dim3(256), 0, st, Hkv, L, n_sink, tab, idx);
  return hipGetLastError();
}

hipError_t launch_select(int n_inst, int inst0, int Hkv, int L, int keep, int pool, bool avg, const float* scores,
                         const InstTable& tab, int32_t* idx, hipStream_t st) {
  return launch_for(n_inst, inst0, Hkv, L, keep, pool, avg, scores, tab, idx, NoFinish{}, st);
}
hipError_t launch_select(int n_inst, int inst0, int Hkv, int L, int keep, int pool, bool avg, const float* scores,
                         const UniformInst& tab, int32_t* idx, hipStream_t st) {
  return launch_for(n_inst, inst0, Hkv, L, keep, pool, avg, scores, tab, idx, NoFinish{}, st);
}
hipError_t launch_select_pooling(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const InstTable& tab, int32_t* idx,
                                 const PoolArgs& pool, hipStream_t st) {
  return launch_for(n_inst, inst0, Hkv, L, keep, 1, false, raw, tab, idx, pool, st);
}
hipError_t launch_select_pooling(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const UniformInst& tab, int32_t* idx,
                                 const PoolArgs& pool, hipStream_t st) {
  return launch_for(n_inst, inst0, Hkv, L, keep, 1, false, raw, tab, idx, pool, st);
}
hipError_t launch_finish(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const InstTable& tab, int32_t* idx,
                         const FinishArgs& fin, hipStream_t st) {
  return finish_for(n_inst, inst0, Hkv, L, keep, raw, tab, idx, fin, st);
}
hipError_t launch_finish(int n_inst, int inst0, int Hkv, int L, int keep, const float* raw, const UniformInst& tab, int32_t* idx,
                         const FinishArgs& fin, hipStream_t st) {
  return finish_for(n_inst, inst0, Hkv, L, keep, raw, tab, idx, fin, st);
}

}  // namespace laq
