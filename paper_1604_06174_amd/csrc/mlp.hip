// Elementwise and reduction kernels of the residual-MLP unit and the MSE head.
// Reductions are fixed-order trees (no atomics), so every result is
// reproducible bit for bit.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace ckpt {
namespace {

// Workgroup = 64 columns x 4 row groups over a block of 16 rows (blockIdx.y)
// of g (of g where z > 0 when z is given, stored to dr when that is): the
// workgroup's column sums over its rows, ((s0 + s1) + s2) + s3 with s_j = rows
// j, j+4, .. in order, go to pdb[blockIdx.y][cols].
__global__ __launch_bounds__(256) void k_colsum_part(int rows, int cols, const float *__restrict__ g,
                                                     const float *__restrict__ z, float *__restrict__ dr,
                                                     float *__restrict__ pdb) {
  __shared__ float part[4][64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int n = blockIdx.x * 64 + tx, r0 = blockIdx.y * 16 + ty;
  float s = 0.f;
  if (n < cols) {
    float gv[4], zv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = r0 + 4 * i;
      const size_t e = size_t(m < rows ? m : 0) * cols + n;
      gv[i] = g[e];
      zv[i] = z ? z[e] : 1.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (r0 + 4 * i < rows) {
        const float v = zv[i] > 0.f ? gv[i] : 0.f;
        if (dr) dr[size_t(r0 + 4 * i) * cols + n] = v;
        s += v;
      }
  }
  part[ty][tx] = s;
  __syncthreads();
  if (ty == 0 && n < cols)
    pdb[size_t(blockIdx.y) * cols + n] = ((part[0][tx] + part[1][tx]) + part[2][tx]) + part[3][tx];
}

// db[n] = sum over r < R of pdb[r][n], in order of r
__global__ __launch_bounds__(256) void k_colsum_rows(int R, int cols, const float *__restrict__ pdb,
                                                     float *__restrict__ db) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= cols) return;
  float s = 0.f;
  int r = 0;
  for (; r + 8 <= R; r += 8) {
    float t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = pdb[size_t(r + u) * cols + n];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += t[u];
  }
  for (; r < R; ++r) s += pdb[size_t(r) * cols + n];
  db[n] = s;
}

// Sum of 256 values by a fixed binary tree in LDS, in thread 0.
__device__ __forceinline__ float tree256(float v, float *red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  return red[0];
}

// Each workgroup sums elements 256 b + t, then 256 gridDim.x further, ...;
// its sum times scale goes to part[b] (2,048 elements per workgroup and up to
// 256 workgroups: one workgroup alone took 120 us over 262,144 elements, bound
// by its own loads).
__global__ __launch_bounds__(256) void k_mse_part(int64_t count, const float *__restrict__ y,
                                                  const float *__restrict__ t, float *__restrict__ g, float scale,
                                                  float *__restrict__ part) {
  __shared__ float red[256];
  const float inv = 1.0f / float(count);
  float s = 0.f;
  const int64_t step = int64_t(gridDim.x) * 256;
  for (int64_t i0 = blockIdx.x * int64_t(256) + threadIdx.x; i0 < count; i0 += 4 * step) {
    float yv[4], tv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + u * step < count ? i0 + u * step : i0;
      yv[u] = y[i];
      tv[u] = t[i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i0 + u * step < count) {
        const float d = yv[u] - tv[u];
        g[i0 + u * step] = 2.0f * d * inv;
        s += d * d;
      }
  }
  const float v = tree256(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = v * scale;
}

// out = scale * the sum of n <= 256 values
__global__ __launch_bounds__(256) void k_sum256(int n, const float *__restrict__ v, float scale,
                                                float *__restrict__ out) {
  __shared__ float red[256];
  const float s = tree256(int(threadIdx.x) < n ? v[threadIdx.x] : 0.f, red);
  if (threadIdx.x == 0) out[0] = s * scale;
}

__global__ void k_copy_scalar(const float *src, float *dst) { dst[0] = src[0]; }

// Elementwise operators of the node-level graph (any of the pointers may
// alias the output: every thread reads its element before writing it).
enum { EW_RELU = 0, EW_ADD = 1, EW_RELU_BWD = 2, EW_COPY = 3 };
template <int OP>
__global__ __launch_bounds__(256) void k_elementwise(int64_t n, const float *a, const float *b, float *y) {
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256) {
    const float x = a[e];
    float v;
    if (OP == EW_RELU) v = fmaxf(x, 0.f);
    else if (OP == EW_ADD) v = x + b[e];
    else if (OP == EW_RELU_BWD) v = b[e] > 0.f ? x : 0.f;
    else v = x;
    y[e] = v;
  }
}

int ew_blocks(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return int(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

}  // namespace

int mlp_row_blocks(int rows) { return (rows + 15) / 16; }

void mlp_colsum_long(hipStream_t s, int rows, int cols, const float *g, const float *z, float *db, float *pdb,
                     float *dr) {
  const int R = mlp_row_blocks(rows);
  hipLaunchKernelGGL(k_colsum_part, dim3((cols + 63) / 64, R), dim3(256), 0, s, rows, cols, g, z, dr, pdb);
  hipLaunchKernelGGL(k_colsum_rows, dim3((cols + 255) / 256), dim3(256), 0, s, R, cols, pdb, db);
}

void ew_relu(hipStream_t s, int64_t n, const float *x, float *y) {
  hipLaunchKernelGGL(k_elementwise<EW_RELU>, dim3(ew_blocks(n)), dim3(256), 0, s, n, x, nullptr, y);
}
void ew_add(hipStream_t s, int64_t n, const float *a, const float *b, float *y) {
  hipLaunchKernelGGL(k_elementwise<EW_ADD>, dim3(ew_blocks(n)), dim3(256), 0, s, n, a, b, y);
}
void ew_relu_bwd(hipStream_t s, int64_t n, const float *dy, const float *y, float *dx) {
  hipLaunchKernelGGL(k_elementwise<EW_RELU_BWD>, dim3(ew_blocks(n)), dim3(256), 0, s, n, dy, y, dx);
}
void ew_copy(hipStream_t s, int64_t n, const float *x, float *y) {
  hipLaunchKernelGGL(k_elementwise<EW_COPY>, dim3(ew_blocks(n)), dim3(256), 0, s, n, x, nullptr, y);
}

int mse_blocks(int64_t count) {
  const int64_t b = (count + 2047) / 2048;
  return int(b < 256 ? b : 256);
}

int mse_head(hipStream_t s, int64_t count, const float *y, const float *t, float *g, float *part,
             float *loss_out) {
  const int nb = mse_blocks(count);
  const float inv = 1.0f / float(count);
  if (nb == 1) {
    hipLaunchKernelGGL(k_mse_part, dim3(1), dim3(256), 0, s, count, y, t, g, inv, loss_out);
    return 1;
  }
  hipLaunchKernelGGL(k_mse_part, dim3(nb), dim3(256), 0, s, count, y, t, g, 1.f, part);
  hipLaunchKernelGGL(k_sum256, dim3(1), dim3(256), 0, s, nb, part, inv, loss_out);
  return 2;
}

void copy_scalar(hipStream_t s, const float *src, float *dst) {
  hipLaunchKernelGGL(k_copy_scalar, dim3(1), dim3(1), 0, s, src, dst);
}

}  // namespace ckpt
