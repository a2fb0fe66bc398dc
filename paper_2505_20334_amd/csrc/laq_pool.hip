// Sequence pooling in launches of its own: of raw scores, for the paths that do not pool where they score or select; and
// of the keys next to the boundaries between the workgroups of the single-read scoring kernel.
#include "laq_internal.h"
#include "laq_pool.h"

namespace laq {

namespace {

// pooled[j] = max (or mean) of raw[i], |i - j| <= half, 0 <= i < P, for prefix keys; the kept trailing columns are
// copied.  A wave takes WAVE_QUADS quads of four scores a turn, the lanes at its ends two more on either side, so
// that every lane finds the scores around its own in its neighbours' registers: no LDS, no barrier.  Rows may start at any
// address: a quad is a 16-byte piece of memory, `shift` scores of the first one belong to the row before.
constexpr int WAVE_QUADS = 60, TURNS = 4, THREADS = 256;
constexpr int WORKGROUP_KEYS = THREADS / 64 * TURNS * WAVE_QUADS * 4;

__device__ __forceinline__ float4 quad_at(const float* __restrict__ r, int pos, int end) {
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  if (pos >= 0 && pos + 3 < end) {
    x = *reinterpret_cast<const float4*>(r + pos);
  } else {
    if (pos >= 0 && pos < end) x.x = r[pos];
    if (pos + 1 >= 0 && pos + 1 < end) x.y = r[pos + 1];
    if (pos + 2 >= 0 && pos + 2 < end) x.z = r[pos + 2];
    if (pos + 3 >= 0 && pos + 3 < end) x.w = r[pos + 3];
  }
  return x;
}

__global__ __launch_bounds__(THREADS) void pool_quads_kernel(int L, int P, int half, bool avg, const float* __restrict__ raw,
                                                             float* __restrict__ pooled) {
  const float* r = raw + (size_t)blockIdx.x * L;
  float* out = pooled + (size_t)blockIdx.x * L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int shift = (int)((reinterpret_cast<uintptr_t>(r) >> 2) & 3), out_shift = (int)((reinterpret_cast<uintptr_t>(out) >> 2) & 3);
  const int first = ((int)blockIdx.y * (THREADS / 64) + wave) * (TURNS * WAVE_QUADS) + lane - 2;
  float4 x[TURNS];
#pragma unroll
  for (int t = 0; t < TURNS; ++t) x[t] = quad_at(r, (first + t * WAVE_QUADS) * 4 - shift, L);
#pragma unroll
  for (int t = 0; t < TURNS; ++t) {
    const int pos = (first + t * WAVE_QUADS) * 4 - shift;
    float4 own = x[t];
    if (pos + 3 >= P) {                    // what lies behind the prefix is in no window
      if (pos >= P) own.x = 0.f;
      if (pos + 1 >= P) own.y = 0.f;
      if (pos + 2 >= P) own.z = 0.f;
      own.w = 0.f;
    }
    float4 p;
    for_half(half, [&](auto h) { p = pool_quad_of<decltype(h)::value>(own, own, own, own, own, avg); });
    if (lane < 2 || lane >= 62) continue;
    const float v[4] = {pos < P ? p.x : x[t].x, pos + 1 < P ? p.y : x[t].y, pos + 2 < P ? p.z : x[t].z, pos + 3 < P ? p.w : x[t].w};
    if (out_shift == shift && pos >= 0 && pos + 3 < L) {
      *reinterpret_cast<float4*>(out + pos) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (pos + c >= 0 && pos + c < L) out[pos + c] = v[c];
    }
  }
}

// The same for wider windows.  A workgroup stages POOL_TILE scores plus the window margins in
// LDS, with zeros for positions outside the prefix: the scores are sums of probabilities, never
// negative, so a zero leaves a maximum alone, and it leaves the ascending fp32 sum of the average
// bit-identical to pool_window()'s sum over the clipped window.  grid.x walks the (instance, KV
// head) pairs.
constexpr int POOL_TILE = 1024;
__global__ __launch_bounds__(256) void pool_kernel(int L, int P, int half, bool avg, const float* __restrict__ raw,
                                                   float* __restrict__ pooled) {
  __shared__ float tile[POOL_TILE + MAX_POOL - 1];
  const float* r = raw + (size_t)blockIdx.x * L;
  float* out = pooled + (size_t)blockIdx.x * L;
  const int j0 = blockIdx.y * POOL_TILE;
  for (int t = threadIdx.x; t < POOL_TILE + 2 * half; t += 256) {
    const int i = j0 - half + t;
    tile[t] = (i >= 0 && i < P) ? r[i] : 0.f;
  }
  __syncthreads();
  const float kernel_size = (float)(2 * half + 1);
  for (int t = threadIdx.x; t < POOL_TILE && j0 + t < L; t += 256) {
    const int j = j0 + t;
    float v;
    if (j >= P) {
      v = r[j];
    } else if (avg) {
      float acc = 0.f;
      for (int o = 0; o <= 2 * half; ++o) acc += tile[t + o];
      v = acc / kernel_size;
    } else {
      v = tile[t + half];
      for (int o = 0; o <= 2 * half; ++o) v = fmaxf(v, tile[t + o]);
    }
    out[j] = v;
  }
}

// Pooled scores of the prefix keys whose pooling window crosses a boundary between two workgroups (`chunks` of chunk_rows keys) of
// the single-read scoring kernel, from the edge records (per chunk: raw scores of its first 2*half rows, then of its last
// 2*half rows).  The boundary before chunk c lies at key b = c * chunk_rows and the keys
// b-half .. b+half-1 are pooled here, one per thread; blockIdx.x is the head.
__global__ __launch_bounds__(256) void pool_boundaries_kernel(int L, int P, int half, int nchunk, int chunk_rows,
                                                               const float* __restrict__ edge,
                                                               float* __restrict__ scores) {
  const int hg = blockIdx.x;
  const int rec = 4 * half, per = 2 * half;
  const int it = blockIdx.y * 256 + threadIdx.x;
  if (it >= (nchunk - 1) * per) return;
  const int c = it / per + 1;
  const int b = c * chunk_rows;
  const int j = b - half + it % per;
  if (j >= P) return;
  // raw score of key i, b - 2*half <= i < b + 2*half, is e[i]: the tail of chunk c-1's record is
  // followed in memory by the head of chunk c's
  const float* e = edge + ((size_t)hg * nchunk + c - 1) * rec + per - (b - per);
  const int hi = min(j + half, P - 1);
  float v = 0.f;
  for (int i = j - half; i <= hi; ++i) v = fmaxf(v, e[i]);
  scores[(size_t)hg * L + j] = v;
}

}  // namespace

hipError_t launch_pool_boundaries(const ScoreGeom& g, int half, int nchunk, int chunk_rows, const float* edge,
                                  float* scores, hipStream_t st) {
  const long long n_heads = (long long)g.n_inst * g.Hkv;
  const int items = (nchunk - 1) * 2 * half;
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(pool_boundaries_kernel, dim3((unsigned)n_heads, (items + 255) / 256), dim3(256), 0, st, g.L, g.P,
                     half, nchunk, chunk_rows, edge, scores);
  return hipGetLastError();
}

hipError_t launch_pool(const ScoreGeom& g, int pool, bool avg, const float* raw, float* pooled, hipStream_t st) {
  const int half = (pool - 1) / 2;
  const unsigned heads = (unsigned)(g.n_inst * g.Hkv);
  if (half <= SELECT_POOL_MAX_HALF) {
    hipLaunchKernelGGL(pool_quads_kernel, dim3(heads, (g.L + 3 + WORKGROUP_KEYS - 1) / WORKGROUP_KEYS), dim3(THREADS), 0, st, g.L, g.P, half, avg,
                       raw, pooled);
  } else {
    hipLaunchKernelGGL(pool_kernel, dim3(heads, (g.L + POOL_TILE - 1) / POOL_TILE), dim3(256), 0, st, g.L, g.P, half, avg, raw, pooled);
  }
  return hipGetLastError();
}

}  // namespace laq
