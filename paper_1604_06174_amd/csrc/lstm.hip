// Row kernels of the LSTM's softmax head, weight copies and reductions (the
// recurrence itself is in lstm_step.hip).
//   head   softmax cross-entropy of a [B, V] row block; the gradient
//          (p - onehot) * scale is kept in fp32
// Every sum runs in an order fixed by
// the shapes alone, so a step is bit-reproducible whatever the schedule.
#include <hip/hip_runtime.h>

#include "common.h"
#include "kernels.h"

namespace ckpt {
namespace {

// dst[c][r] = bf16(src[r][c]) for src [R][C] fp32, through 32x32 LDS tiles.
__global__ __launch_bounds__(256) void k_transpose_bf16(int R, int C, const float *__restrict__ src,
                                                        __bf16 *__restrict__ dst, int ld) {
  __shared__ float t[32][33];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = ty; k < 32; k += 8) {
    const int r = r0 + k, c = c0 + tx;
    t[k][tx] = (r < R && c < C) ? src[size_t(r) * C + c] : 0.f;
  }
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int c = c0 + k, r = r0 + tx;
    if (c < C && r < R) dst[size_t(c) * ld + r] = (__bf16)t[tx][k];
  }
}

__global__ __launch_bounds__(256) void k_cvt_bf16(int64_t n, const float *__restrict__ src,
                                                  __bf16 *__restrict__ dst) {
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256)
    dst[e] = (__bf16)src[e];
}

// the same conversion, eight elements per thread and iteration (two 16-byte
// loads, one 16-byte store) for n a multiple of 8 with src 16-byte and dst
// 16-byte aligned
__global__ __launch_bounds__(256) void k_cvt_bf16x8(int64_t n8, const float4 *__restrict__ src,
                                                    uint4 *__restrict__ dst) {
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n8; e += int64_t(gridDim.x) * 256) {
    const float4 a = src[2 * e], b = src[2 * e + 1];
    const float f[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    unsigned w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const __bf16 lo = (__bf16)f[2 * k], hi = (__bf16)f[2 * k + 1];
      w[k] = unsigned(__builtin_bit_cast(unsigned short, lo)) |
             (unsigned(__builtin_bit_cast(unsigned short, hi)) << 16);
    }
    dst[e] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// dst[r * ld + c] = bf16(src[r * C + c]) for src [R][C] fp32
__global__ __launch_bounds__(256) void k_cvt_bf16_rows(int R, int C, const float *__restrict__ src,
                                                       __bf16 *__restrict__ dst, int ld) {
  const int64_t n = int64_t(R) * C;
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256)
    dst[(e / C) * ld + e % C] = (__bf16)src[e];
}

// (m, s) <- the pair for the union of two column sets: m the larger maximum,
// s both sums rescaled to it (0 while both sets are empty)
__device__ __forceinline__ void lse_combine(float &m, float &s, float om, float os) {
  const float mx = fmaxf(m, om);
  s = mx == -INFINITY ? 0.f : s * expf(m - mx) + os * expf(om - mx);
  m = mx;
}

// Softmax cross-entropy: loss_row = log sum exp(l - max) + max - l[label],
// dlog = (softmax - onehot) * scale (a label outside [0, V) gives a NaN loss
// for the row and no one-hot term), from the logits l (bias included) and
// each row's (max, sum of exp) pairs per column tile of the product that
// wrote them.  Every
// wavefront combines its row's pairs itself (lane j takes tiles j, j + 64,
// ... in order, then a butterfly, whose pairwise combinations are symmetric),
// so all workgroups of a row use the same maximum and sum with no exchange
// between them.  Workgroup = 1024 columns of one row, four per thread;
// blockIdx.z = the unit of a batch (its logits, dlog and statistics ul, ul
// and ur floats after the previous unit's, its labels and loss rows `rows`
// after).  The row's loss is formed by the thread that holds the label's
// logit, from its register, so dlog may overwrite the logits in place.
__global__ __launch_bounds__(256) void k_softmax_ce_tiles(int V, const float *logits, int nt,
                                                          const float *__restrict__ rstat,
                                                          const int *__restrict__ labels, float scale,
                                                          float *dlog, float *__restrict__ loss_rows,
                                                          int rows, int64_t ul, int64_t ur) {
  const int row = blockIdx.y, lane = threadIdx.x & 63;
  const int64_t u = blockIdx.z;
  logits += u * ul;
  dlog += u * ul;
  labels += u * rows;
  loss_rows += u * rows;
  const float *rs = rstat + u * ur + size_t(row) * nt * 2;
  float m = -INFINITY, se = 0.f;
  for (int j = lane; j < nt; j += 64) lse_combine(m, se, rs[2 * j], rs[2 * j + 1]);
  for (int o = 32; o > 0; o >>= 1) {
    const float om = __shfl_xor(m, o, 64), os = __shfl_xor(se, o, 64);
    lse_combine(m, se, om, os);
  }
  const int lab = labels[row];
  const float inv = 1.0f / se;
  const int v0 = (blockIdx.x * 256 + threadIdx.x) * 4;
  const float *x = logits + size_t(row) * V;
  if (v0 < V) {
    const float4 xv = *reinterpret_cast<const float4 *>(x + v0);
    const float xs[4] = {xv.x, xv.y, xv.z, xv.w};
    float d[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      d[k] = (expf(xs[k] - m) * inv - (v0 + k == lab ? 1.f : 0.f)) * scale;
      if (v0 + k == lab) loss_rows[row] = (logf(se) + m) - xs[k];
    }
    *reinterpret_cast<float4 *>(dlog + size_t(row) * V + v0) = make_float4(d[0], d[1], d[2], d[3]);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && !(lab >= 0 && lab < V)) loss_rows[row] = NAN;
}

// db[n] (+)= the nrec records rec[r][n] (record stride N), r = 0 .. nrec-1:
// workgroup = 64 columns x 4 groups of consecutive records; each group adds
// its records in order, the groups combine as ((g0 + g1) + g2) + g3.
__global__ __launch_bounds__(256) void k_db_chunk(int N, int nrec, const float *__restrict__ rec,
                                                  float *__restrict__ db, int first) {
  __shared__ float part[4][64];
  const int cx = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int n = blockIdx.x * 64 + cx;
  const int per = (nrec + 3) / 4, r0 = min(nrec, g * per), r1 = min(nrec, r0 + per);
  float s = 0.f;
  if (n < N) {
    int r = r0;
    for (; r + 8 <= r1; r += 8) {
      float t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = rec[size_t(r + u) * N + n];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += t[u];
    }
    for (; r < r1; ++r) s += rec[size_t(r) * N + n];
  }
  part[g][cx] = s;
  __syncthreads();
  if (g == 0 && n < N) {
    const float t = ((part[0][cx] + part[1][cx]) + part[2][cx]) + part[3][cx];
    db[n] = first ? t : db[n] + t;
  }
}

// loss = scale * sum of rows (fixed order: thread t takes rows t, t+1024, ...)
__global__ __launch_bounds__(1024) void k_loss_reduce(int64_t rows, const float *__restrict__ v,
                                                      float scale, float *__restrict__ loss) {
  __shared__ float red[1024];
  float s = 0.f;
  for (int64_t r = threadIdx.x; r < rows; r += 1024) s += v[r];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = red[0] * scale;
}

__global__ __launch_bounds__(256) void k_fill_f32(int64_t n, float *__restrict__ p, float v) {
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256) p[e] = v;
}

inline int grid_for(int64_t n) {
  int64_t g = (n + 255) / 256;
  return int(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

}  // namespace

void transpose_bf16(hipStream_t s, int R, int C, const float *src, void *dst, int ld) {
  hipLaunchKernelGGL(k_transpose_bf16, dim3((C + 31) / 32, (R + 31) / 32), dim3(256), 0, s, R, C,
                     src, static_cast<__bf16 *>(dst), ld > 0 ? ld : R);
}

void cvt_bf16_rows(hipStream_t s, int R, int C, const float *src, void *dst, int ld) {
  hipLaunchKernelGGL(k_cvt_bf16_rows, dim3(grid_for(int64_t(R) * C)), dim3(256), 0, s, R, C, src,
                     static_cast<__bf16 *>(dst), ld);
}

void cvt_bf16(hipStream_t s, int64_t n, const float *src, void *dst) {
  if (n % 8 == 0 && uintptr_t(src) % 16 == 0 && uintptr_t(dst) % 16 == 0) {
    hipLaunchKernelGGL(k_cvt_bf16x8, dim3(grid_for(n / 8)), dim3(256), 0, s, n / 8,
                       reinterpret_cast<const float4 *>(src), static_cast<uint4 *>(dst));
    return;
  }
  hipLaunchKernelGGL(k_cvt_bf16, dim3(grid_for(n)), dim3(256), 0, s, n, src, static_cast<__bf16 *>(dst));
}

void softmax_ce_tiles_batched(hipStream_t s, int nunits, int rows, int V, float *logits, int64_t ul, int nt,
                              const float *rstat, int64_t ur, const int *labels, float scale,
                              float *loss_rows) {
  if (nunits <= 0) return;
  if (V % 4 != 0 || ul % 4 != 0 || reinterpret_cast<uintptr_t>(logits) % 16 != 0)
    fail(CKPT_E_INVALID, "softmax_ce_tiles_batched: V and the unit stride multiples of 4, rows 16-byte aligned");
  hipLaunchKernelGGL(k_softmax_ce_tiles, dim3((V + 1023) / 1024, rows, nunits), dim3(256), 0, s, V, logits,
                     nt, rstat, labels, scale, logits, loss_rows, rows, ul, ur);
}

void db_chunk(hipStream_t s, int N, int nrec, const float *rec, float *db, bool first) {
  hipLaunchKernelGGL(k_db_chunk, dim3((N + 63) / 64), dim3(256), 0, s, N, nrec, rec, db, first ? 1 : 0);
}

void loss_reduce(hipStream_t s, int64_t rows, const float *v, float scale, float *loss) {
  hipLaunchKernelGGL(k_loss_reduce, dim3(1), dim3(1024), 0, s, rows, v, scale, loss);
}

void fill_f32(hipStream_t s, int64_t n, float *p, float v) {
  hipLaunchKernelGGL(k_fill_f32, dim3(grid_for(n)), dim3(256), 0, s, n, p, v);
}

}  // namespace ckpt
