// Fixed-order sums of weight-gradient partials as a workgroup's work, for kernels
// that run them alone or beside something else.
#pragma once

#include <hip/hip_runtime.h>

namespace ckpt {

// from this many float4 columns on sixteen slices are added, below 64 (as
// sum_partials does for E >= 32,768)
constexpr int SUM_SLICES16_E4 = 16 * 2048 / 4;

// Workgroups are dispatched to the eight XCDs (each with its own L2) in
// turn; consecutive column groups are mapped to one XCD so that the cache
// lines they share are fetched from HBM once, not once per XCD.
__device__ __forceinline__ int xcd_grouped(int id, int G) {
  const int q = G / 8, r = G % 8, x = id % 8, k = id / 8;
  return x * q + (x < r ? x : r) + k;
}

__device__ __forceinline__ void add4(float4 &s, const float4 &v) {
  s.x += v.x;
  s.y += v.y;
  s.z += v.z;
  s.w += v.w;
}

// k_sum_partials<16>'s sum for any nb, four consecutive e per thread: column
// group blk of 64 threads' columns, each wavefront four of the sixteen slices
// (slice k adds part[k], part[k + 16], ...; sixteen 16-byte loads in flight),
// then the slices are added in order.  red holds [16][64].
__device__ __forceinline__ void sum_slices16(const float4 *__restrict__ part, int nb, int E4,
                                             float4 *__restrict__ out, int blk, float4 *red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blk * 64 + lane;
  const float4 *p = part + min(i, E4 - 1);
  float4 s[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) s[k] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int b = 4 * wave; b < nb; b += 64) {
    float4 v[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) v[u][k] = p[size_t(min(b + 16 * u + k, nb - 1)) * E4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (b + 16 * u + k < nb) add4(s[k], v[u][k]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) red[(4 * wave + k) * 64 + lane] = s[k];
  __syncthreads();
  if (wave == 0 && i < E4) {
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < 16; ++k) add4(t, red[k * 64 + lane]);
    out[i] = t;
  }
}

// k_sum_partials<64>'s sum, four consecutive e per thread: column group blk is
// four threads' columns, so a workgroup reads 64 consecutive bytes of a partial
// (16 with one e per thread) with eight loads in flight.  red holds [64][4].
__device__ __forceinline__ void sum_slices64(const float4 *__restrict__ part, int nb, int E4,
                                             float4 *__restrict__ out, int blk, float4 *red) {
  const int ex = threadIdx.x % 4, sl = threadIdx.x / 4;
  const int i = blk * 4 + ex;
  const float4 *p = part + min(i, E4 - 1);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int b = sl; b < nb; b += 8 * 64) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[size_t(min(b + 64 * u, nb - 1)) * E4];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (b + 64 * u < nb) add4(s, v[u]);
  }
  red[sl * 4 + ex] = s;
  __syncthreads();
  if (sl == 0 && i < E4) {
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 16
    for (int k = 0; k < 64; ++k) add4(t, red[k * 4 + ex]);
    out[i] = t;
  }
}

}  // namespace ckpt
