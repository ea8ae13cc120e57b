// The LSTM recurrence's two serial kernels: one time step's product and its
// pointwise work in one launch each (and the pointwise work alone, for the
// shapes that are faster with a split-K product: lstm_step_fwd_wins, lstm_step_bwd_wins).
//   forward   z = [x_t | h_{t-1}] [W_x; W_h] + b, gates, c_t, h_t
//   backward  dh = dl_t W_o^T (slices formed ahead) + dz_{t+1} W_h^T, the gate
//             backward: dz_t, dc_{t-1}, bias-gradient column sums
//
// What bounds them: a step has few rows (the batch), a long k (1024 - 4096)
// and cannot start before the previous one ends, so its time is one kernel's
// latency plus the operand bytes each compute unit must load: the products
// are 0.5 - 1 GFLOP against 16 or 8 MB of weights.  Hence one workgroup per
// small tile of the result with the whole k range inside it, split over its
// wavefronts: 32 rows x 8 hidden units of all four gates (256 workgroups of
// 256 KB of operands at batch 64, 1024 hidden; a 16-row tile for batches of
// at most 16) forward, 16 x 16 backward (256 workgroups, 256 KB).  Every
// wavefront issues the loads of its share at once, straight into registers in
// the MFMA operand layout, the wavefronts' partial sums meet in LDS and are
// added in wavefront order, and the same workgroup then holds the complete
// sums it needs for the pointwise work: no split-K slices go through memory
// and no second launch waits for them.
//
// Every sum's order depends on the shape alone (k steps of 32 in blocks per
// wavefront, wavefronts in order, then the head slices in order), so a step's
// bits do not depend on the plan that runs it.
#include <hip/hip_runtime.h>

#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace ckpt {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 global_u32x4;

// an operand chunk outside its matrix is loaded from here (16 bytes per lane)
static __device__ __align__(16) const unsigned g_zero_chunks[256] = {};

__device__ __forceinline__ float sigm(float x) { return 1.0f / (1.0f + expf(-x)); }

// one element's gate backward: dh and the incoming dc to the gates' z gradients
// and dc_{t-1} (none where null)
__device__ __forceinline__ void gate_backward(float dh, float dc, float ig, float fg, float gg, float og, float c,
                                              float c_prev, float (&dz)[4], float *dc_prev) {
  const float tc = tanhf(c);
  const float dct = dc + dh * og * (1.f - tc * tc);
  dz[0] = dct * gg * ig * (1.f - ig);
  dz[1] = dct * c_prev * fg * (1.f - fg);
  dz[2] = dct * ig * (1.f - gg * gg);
  dz[3] = dh * tc * og * (1.f - og);
  if (dc_prev) *dc_prev = dct * fg;
}

typedef __attribute__((address_space(3))) void lds_void_t;

// NV sums v[k] = part[k d] + part[slice + k d] + ... over the ns slices in that
// order; U slices are loaded for all of them before any is added, so a round's
// loads are in flight together
template <int NV, int U>
__device__ __forceinline__ void slices_sum(const float *__restrict__ part, int64_t d, int ns, int64_t slice,
                                           float (&v)[NV]) {
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = part[k * d];
  int z = 1;
  for (; z + U <= ns; z += U) {
    float t[U][NV];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < NV; ++k) t[u][k] = part[(z + u) * slice + k * d];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < NV; ++k) v[k] += t[u][k];
  }
  for (; z < ns; ++z)
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += part[z * slice + k * d];
}
template <int U>
__device__ __forceinline__ float slices_sum(const float *__restrict__ part, int ns, int64_t slice) {
  float v[1];
  slices_sum<1, U>(part, 0, ns, slice, v);
  return v[0];
}

// acc[r][c] (16 x 16 tiles) += the product over the k chunks of eight
// [g, g + G) (G / 4 MFMA steps of 32), or over [g, q1) with q1 - g < 4 (TAIL).
// a(row, q) is the address of row `row`'s chunk q, b(q) that of column lane %
// 16's chunk q in the first column tile, bt the distance to the next tile's.
// The rows go straight from global memory into the wavefront's own part of
// LDS, in runs of G chunks per row (consecutive lanes read consecutive
// chunks), slot p of row r holding chunk p ^ (r mod G) so that the operand
// reads of sixteen rows spread over the banks; the columns are stored in
// operand order and go straight to registers.  Every load is issued before any
// is waited for.
template <int RT, int CT, int G, bool TAIL, class FA, class FB>
__device__ __forceinline__ void wave_group(int g, int q1, FA a, FB b, size_t bt, unsigned char *lds,
                                           floatx4 (&acc)[RT][CT]) {
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4;
  const void *zero = g_zero_chunks + 4 * lane;
  constexpr int RPI = 64 / G;  // rows per load instruction
  bf16x8 bv[G / 4][CT];
#pragma unroll
  for (int i = 0; i < 16 * RT / RPI; ++i) {
    const int row = i * RPI + lane / G, q = g + ((lane % G) ^ (row % G));
    const void *src = !TAIL || q < q1 ? a(row, q) : zero;
    __builtin_amdgcn_global_load_lds(src, (lds_void_t *)(lds + i * 1024), 16, 0, 0);
  }
  const __bf16 *bp = b(g + kq);
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int u = 0; u < G / 4; ++u) {
      const void *p = bp + c * bt + b.step(4 * u);
      if (TAIL && g + kq >= q1) p = zero;
      bv[u][c] = __builtin_bit_cast(bf16x8, *(global_u32x4 *)p);
    }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // every load above has landed
#pragma unroll
  for (int u = 0; u < G / 4; ++u) {
    bf16x8 av[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int row = r * 16 + i16, slot = (4 * u + kq) ^ (row % G);
      av[r] = *reinterpret_cast<const bf16x8 *>(lds + (row * G + slot) * 16);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < CT; ++c)
        acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[r], bv[u][c], acc[r][c], 0, 0, 0);
  }
  __builtin_amdgcn_s_waitcnt(0xC07F);  // the reads have returned before the next group's loads
}

// the product over this wavefront's chunks [q0, q1), G at once while they
// last, then in halves
template <int RT, int CT, int G, class FA, class FB>
__device__ __forceinline__ void wave_product(int q0, int q1, FA a, FB b, size_t bt, unsigned char *lds,
                                             floatx4 (&acc)[RT][CT]) {
  for (; q0 + G <= q1; q0 += G) wave_group<RT, CT, G, false>(q0, q1, a, b, bt, lds, acc);
  if constexpr (G > 4)
    wave_product<RT, CT, G / 2>(q0, q1, a, b, bt, lds, acc);
  else if (q0 < q1)
    wave_group<RT, CT, 4, true>(q0, q1, a, b, bt, lds, acc);
}

// The wavefronts' partial tiles, added in wavefront order into sum[row][col]
// (LDS, pitch COLS): wavefront w's partial goes to red + w * pitch (its own
// staging part, which only it has read).  Ends with a barrier.
template <int RT, int CT, int NW>
__device__ __forceinline__ void wave_sum(const floatx4 (&acc)[RT][CT], float *red, int pitch, float *sum) {
  constexpr int ROWS = 16 * RT, COLS = 16 * CT, E = ROWS * COLS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        red[wave * pitch + (r * 16 + 4 * (lane >> 4) + i) * COLS + c * 16 + (lane & 15)] = acc[r][c][i];
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += 64 * NW) {
    float t[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) t[w] = red[w * pitch + e];
    float v = t[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += t[w];
    sum[e] = v;
  }
  __syncthreads();
}

// Column chunk addresses in the packed operand orders: chunk q of the lane's
// column at p + q * pitch (values)
struct Packed {
  const __bf16 *p;
  int pitch;
  __device__ __forceinline__ const __bf16 *operator()(int q) const { return p + size_t(q) * pitch; }
  __device__ __forceinline__ size_t step(int n) const { return size_t(n) * pitch; }
};

// Workgroup tile of the linear id: the row blocks of one column block have ids
// that differ by multiples of 8, i.e. they run on one XCD and read its weights
// through one L2.
__device__ __forceinline__ void tile_of_id(int nr, int nc, int &row, int &col) {
  const int id = blockIdx.x, full = nc / 8 * 8 * nr;
  if (id < full) {
    const int g = id / (8 * nr), o = id % (8 * nr);
    col = g * 8 + o % 8;
    row = o / 8;
  } else {
    const int o = id - full, rest = nc % 8;
    col = nc / 8 * 8 + o % rest;
    row = o / rest;
  }
}

// Forward step: tile of 16 RT rows x 8 hidden units (columns gate * 8 + unit).
// x [B, K1] and h [B, K2] bf16 (K2 = 0: no recurrent part), w = the packed
// [W_x; W_h] (see k_pack_gates).
template <int RT, int NW>
__global__ __launch_bounds__(64 * NW) void k_lstm_step_fwd(int B, int H, int K1, int K2,
                                                           const __bf16 *__restrict__ x,
                                                           const __bf16 *__restrict__ h,
                                                           const __bf16 *__restrict__ w,
                                                           const float *__restrict__ bias,
                                                           const float *__restrict__ c_prev,
                                                           float *__restrict__ gates,
                                                           __bf16 *__restrict__ h_out,
                                                           float *__restrict__ c_out) {
  constexpr int CT = 2, ROWS = 16 * RT, COLS = 32, G = 16, PART = ROWS * G * 16;
  __shared__ __align__(1024) unsigned char lds[NW * PART];
  __shared__ float z[ROWS * COLS];
  static_assert(PART >= ROWS * COLS * 4, "a wavefront's partial tile fits its staging part");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15;
  int tr, tc;
  tile_of_id((B + ROWS - 1) / ROWS, H / 8, tr, tc);
  const int b0 = tr * ROWS, j0 = tc * 8;
  // the pointwise part's operands, loaded ahead of the product
  const int pr = threadIdx.x >> 3, pu = threadIdx.x & 7;
  const int pb = b0 + pr, pj = j0 + pu;
  const bool point = pr < ROWS && pb < B;
  float bi[4] = {0.f, 0.f, 0.f, 0.f}, cp = 0.f;
  if (point) {
#pragma unroll
    for (int g = 0; g < 4; ++g) bi[g] = bias[g * H + pj];
    if (c_prev) cp = c_prev[size_t(pb) * H + pj];
  }
  // k chunks of eight, per wavefront a multiple of four (one MFMA step); the
  // split is that of the whole [x | h] whether or not there is an h
  const int nq = (K1 + K2) / 8, nqh = (K1 + H) / 8, per = (nqh + 4 * NW - 1) / (4 * NW) * 4;
  floatx4 acc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[r][c] = floatx4{0.f, 0.f, 0.f, 0.f};
  const __bf16 *wt = w + size_t(tc) * 4 * nqh * 64;  // this column block: two tiles of 16 nqh chunks
  wave_product<RT, CT, G>(
      min(wave * per, nq), min(wave * per + per, nq),
      [&](int row, int q) -> const void * {
        // a row past the batch re-reads the last one (its results are dropped)
        const int b = min(b0 + row, B - 1), k = 8 * q;
        const __bf16 *p = k < K1 ? x + size_t(b) * K1 : h + (ptrdiff_t(b) * K2 - K1);
        return p + k;
      },
      Packed{wt + i16 * 8, 128}, size_t(nqh) * 128, lds + wave * PART, acc);
  wave_sum<RT, CT, NW>(acc, reinterpret_cast<float *>(lds), PART / 4, z);
  if (point) {
    const float *zr = z + pr * COLS + pu;
    const float ig = sigm(zr[0] + bi[0]);
    const float fg = sigm(zr[8] + bi[1]);
    const float gg = tanhf(zr[16] + bi[2]);
    const float og = sigm(zr[24] + bi[3]);
    const float c = fg * cp + ig * gg;
    float *gr = gates + size_t(pb) * 4 * H + pj;
    gr[0] = ig;
    gr[H] = fg;
    gr[2 * H] = gg;
    gr[3 * H] = og;
    c_out[size_t(pb) * H + pj] = c;
    h_out[size_t(pb) * H + pj] = (__bf16)(og * tanhf(c));
  }
}

// The pointwise part of the forward after a split-K product, one thread per (b,
// j): z = the ns partial slices [B, 4H] in order + bias.
__global__ __launch_bounds__(256) void k_lstm_fwd_point(int B, int H, const float *__restrict__ zpart, int ns,
                                                        const float *__restrict__ bias,
                                                        const float *__restrict__ c_prev,
                                                        float *__restrict__ gates, __bf16 *__restrict__ h_out,
                                                        float *__restrict__ c_out) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= B * H) return;
  const int b = e / H, j = e % H;
  const size_t r = size_t(b) * 4 * H + j;
  float z[4];
  slices_sum<4, 4>(zpart + r, H, ns, int64_t(B) * 4 * H, z);
  const float ig = sigm(z[0] + bias[j]);
  const float fg = sigm(z[1] + bias[H + j]);
  const float gg = tanhf(z[2] + bias[2 * H + j]);
  const float og = sigm(z[3] + bias[3 * H + j]);
  const float cp = c_prev ? c_prev[e] : 0.f;
  const float c = fg * cp + ig * gg;
  gates[r] = ig;
  gates[r + H] = fg;
  gates[r + 2 * size_t(H)] = gg;
  gates[r + 3 * size_t(H)] = og;
  c_out[e] = c;
  h_out[e] = (__bf16)(og * tanhf(c));
}

// Backward step: tile of 16 rows x 16 hidden units.  dh = sum over z < ns of
// hpart[z][b][j] (slices `slice` floats apart) + the product of dzn [B, 4H]
// (null, at the last step: none) and the packed W_h (see k_pack_rows) over k = 4H.  Records of 16 rows' bias-gradient
// column sums go to dbp[row block][4H], rows added in order.
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_lstm_step_bwd(
    int B, int H, const __bf16 *dzn, const __bf16 *__restrict__ w,
    const float *__restrict__ hpart, int ns, int64_t slice, const float *__restrict__ dc_in,
    const float *__restrict__ gates, const float *__restrict__ c_t, const float *__restrict__ c_prev,
    const __bf16 *__restrict__ h_prev, const __bf16 *__restrict__ h_t, __bf16 *dz,
    float *__restrict__ dc_prev, __bf16 *__restrict__ hp_copy, __bf16 *__restrict__ hc_copy,
    float *__restrict__ dbp) {
  constexpr int G = 32, PART = 16 * G * 16;
  __shared__ __align__(1024) unsigned char lds[NW * PART];
  __shared__ float sum[256];
  __shared__ float zs[4][16][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15;
  int tr, tc;
  tile_of_id((B + 15) / 16, (H + 15) / 16, tr, tc);
  const int b0 = tr * 16, j0 = tc * 16;
  const int pr = (threadIdx.x >> 4) & 15, pu = threadIdx.x & 15;
  const int b = b0 + pr, j = j0 + pu;
  const bool point = threadIdx.x < 256 && b < B && j < H;
  const size_t e = size_t(b) * H + j;
  // the pointwise part's operands, loaded ahead of the product
  float gv[4] = {0.f, 0.f, 0.f, 0.f}, ct = 0.f, cp = 0.f, dci = 0.f, hd = 0.f;
  __bf16 hp = (__bf16)0.f, ht = (__bf16)0.f;
  if (point) {
#pragma unroll
    for (int g = 0; g < 4; ++g) gv[g] = gates[size_t(b) * 4 * H + g * H + j];
    ct = c_t[e];
    dci = dc_in[e];
    if (c_prev) cp = c_prev[e];
    if (h_prev) hp = h_prev[e];
    ht = h_t[e];
    hd = slices_sum<8>(hpart + e, ns, slice);
  }
  if (dzn) {
    const int nq = H / 2, per = (nq + 4 * NW - 1) / (4 * NW) * 4;  // chunks of eight of 4H
    floatx4 acc[1][1] = {{floatx4{0.f, 0.f, 0.f, 0.f}}};
    const int nc = min(16, H - j0);
    const __bf16 *wt = w + size_t(j0) * 4 * H;
    wave_product<1, 1, G>(
        min(wave * per, nq), min(wave * per + per, nq),
        [&](int row, int q) -> const void * {
          return dzn + size_t(min(b0 + row, B - 1)) * 4 * H + 8 * q;
        },
        // a column past the last tile's re-reads its last one
        Packed{wt + min(i16, nc - 1) * 8, nc * 8}, 0, lds + wave * PART, acc);
    wave_sum<1, 1, NW>(acc, reinterpret_cast<float *>(lds), PART / 4, sum);
  }
  if (threadIdx.x < 256) {
    float zv[4] = {0.f, 0.f, 0.f, 0.f};
    if (point) {
      const float dhv = dzn ? hd + sum[threadIdx.x] : hd;
      gate_backward(dhv, dci, gv[0], gv[1], gv[2], gv[3], ct, cp, zv, dc_prev ? dc_prev + e : nullptr);
      __bf16 *dr = dz + size_t(b) * 4 * H + j;
#pragma unroll
      for (int k = 0; k < 4; ++k) dr[k * H] = (__bf16)zv[k];
      hp_copy[e] = hp;
      hc_copy[e] = ht;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) zs[k][pr][pu] = zv[k];
  }
  __syncthreads();
  if (threadIdx.x < 64 && j0 + i16 < H) {
    const int k = threadIdx.x >> 4;
    float t[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r] = zs[k][r][i16];
    float v = t[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) v += t[r];
    dbp[size_t(tr) * 4 * H + size_t(k) * H + j0 + i16] = v;
  }
}

// The gate backward after a split-K product, one thread per (b, j): workgroup =
// 64 hidden units x 4 batch rows (blockIdx.y = row block).  dh = the ns partial
// slices [B, H] in order.  The workgroup's bias-gradient column sums over its 4
// rows, ((r0 + r1) + r2) + r3, go to dbp[blockIdx.y][4H].
__global__ __launch_bounds__(256) void k_lstm_bwd_point(
    int B, int H, const float *__restrict__ dhpart, int ns, const float *__restrict__ dc_in,
    const float *__restrict__ gates, const float *__restrict__ c_t, const float *__restrict__ c_prev,
    const __bf16 *__restrict__ h_prev, const __bf16 *__restrict__ h_t, __bf16 *__restrict__ dz,
    float *__restrict__ dc_prev, __bf16 *__restrict__ hp_copy, __bf16 *__restrict__ hc_copy,
    float *__restrict__ dbp) {
  __shared__ float part[4][4][64];
  const int cx = threadIdx.x & 63, rg = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + cx, b = blockIdx.y * 4 + rg;
  float zv[4] = {0.f, 0.f, 0.f, 0.f};
  if (j < H && b < B) {
    const size_t e = size_t(b) * H + j;
    const float dhv = slices_sum<8>(dhpart + e, ns, int64_t(B) * H);
    const float *gr = gates + size_t(b) * 4 * H;
    const float ig = gr[j], fg = gr[H + j], gg = gr[2 * H + j], og = gr[3 * H + j];
    gate_backward(dhv, dc_in[e], ig, fg, gg, og, c_t[e], c_prev ? c_prev[e] : 0.f, zv, dc_prev ? dc_prev + e : nullptr);
    __bf16 *dr = dz + size_t(b) * 4 * H;
#pragma unroll
    for (int k = 0; k < 4; ++k) dr[k * H + j] = (__bf16)zv[k];
    hp_copy[e] = h_prev ? h_prev[e] : (__bf16)0.f;
    hc_copy[e] = h_t[e];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) part[k][rg][cx] = zv[k];
  __syncthreads();
  if (j < H) {
    const int k = rg;  // row group rg writes gate k's column sum
    const float t = ((part[k][0][cx] + part[k][1][cx]) + part[k][2][cx]) + part[k][3][cx];
    dbp[size_t(blockIdx.y) * 4 * H + size_t(k) * H + j] = t;
  }
}

// Column sums of the softmax gradients of steps t, t - 1, ... (blockIdx.y = 0,
// 1, ...) with their bf16 copies: step u's gradient at dlog - u sd, its copy
// at dl - u B V.  Workgroup = 32 columns x 16 row groups of one step; group rg
// takes rows rg, rg + 16, ..., issuing four row loads before it uses any, and
// the groups combine as a fixed pairwise tree.  cs[u][v] = the step's sum, which
// a launch of a single step adds to db itself (when given).
__global__ __launch_bounds__(512) void k_head_prep(int B, int V, const float *__restrict__ dlog, int64_t sd,
                                                   __bf16 *__restrict__ dl, float *__restrict__ cs,
                                                   float *__restrict__ db, int first) {
  __shared__ float part[16][32];
  const int cx = threadIdx.x & 31, rg = threadIdx.x >> 5;
  const int v = blockIdx.x * 32 + cx;
  const int64_t u = blockIdx.y;
  dlog -= u * sd;
  dl -= u * B * V;
  float s = 0.f;
  if (v < V)
    for (int b0 = rg; b0 < B; b0 += 64) {
      float d[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int b = b0 + 16 * q;
        d[q] = b < B ? dlog[size_t(b) * V + v] : 0.f;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int b = b0 + 16 * q;
        if (b < B) {
          dl[size_t(b) * V + v] = (__bf16)d[q];
          s += d[q];
        }
      }
    }
  part[rg][cx] = s;
  __syncthreads();
  if (rg == 0 && v < V) {
    float q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = part[2 * i][cx] + part[2 * i + 1][cx];
    const float t = (((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7])));
    if (db) db[v] = first ? t : db[v] + t;
    else cs[u * V + v] = t;
  }
}

// db[v] (+)= cs[0][v], cs[1][v], ... in order
__global__ __launch_bounds__(256) void k_head_db(int V, int nu, const float *__restrict__ cs,
                                                 float *__restrict__ db, int first) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= V) return;
  float s = first ? 0.f : db[v];
  for (int u0 = 0; u0 < nu; u0 += 8) {
    float t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = u0 + u < nu ? cs[size_t(u0 + u) * V + v] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u0 + u < nu) s = first && u0 + u == 0 ? t[u] : s + t[u];
  }
  db[v] = s;
}

// dst = [W_x; W_h] in the forward step's operand order: per block of 8 hidden
// units two tiles of 16 columns (gate * 8 + unit), per tile the k chunks in
// order, per chunk 16 columns of 8 k.  This launch packs src [8 nq][4H] as
// chunks [qoff, qoff + nq) of nqt.  Thread = one column of a chunk.
__global__ __launch_bounds__(256) void k_pack_gates(int H, int nq, int qoff, int nqt,
                                                    const float *__restrict__ src, __bf16 *__restrict__ dst) {
  const int64_t e = blockIdx.x * int64_t(256) + threadIdx.x;
  if (e >= int64_t(nq) * 4 * H) return;
  const int q = int(e / (4 * H)), n = int(e % (4 * H)), gate = n / H, j = n % H;
  bf16x8 v;
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = (__bf16)src[(size_t(q) * 8 + k) * 4 * H + n];
  const size_t tile = size_t(j / 8) * 2 + (gate >> 1);
  const int col = (gate & 1) * 8 + j % 8;
  *reinterpret_cast<bf16x8 *>(dst + ((tile * nqt + qoff + q) * 16 + col) * 8) = v;
}

// dst = W_h [H][4H] in the backward step's operand order: per tile of 16 rows
// (the last one may have 8) the k chunks in order, per chunk the tile's rows
// of 8 k.  Thread = one row of a chunk.
__global__ __launch_bounds__(256) void k_pack_rows(int H, const float *__restrict__ src, __bf16 *__restrict__ dst) {
  const int64_t e = blockIdx.x * int64_t(256) + threadIdx.x;  // the chunk's place in dst
  const int nq = H / 2;
  if (e >= int64_t(H) * nq) return;
  const int tile = int(e / (16 * nq)), nc = min(16, H - tile * 16);
  const int o = int(e - int64_t(tile) * 16 * nq), q = o / nc, j = tile * 16 + o % nc;
  const float *p = src + size_t(j) * 4 * H + size_t(q) * 8;
  bf16x8 v;
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = (__bf16)p[k];
  *reinterpret_cast<bf16x8 *>(dst + e * 8) = v;
}

}  // namespace

// The step kernels' time is that of the rounds of one workgroup per compute unit
// (sixteen wavefronts, 128 KB of LDS) that their tiles make, each round the
// operand loads of its tiles; a split-K product shares loads over larger tiles
// and needs a second launch.  One round: always the step kernels.  More: while
// the operands of all rounds are short enough.  48 steps under the sqrt /
// recursive plan (vocabulary 10,000, and 1000 at hidden 512), us, products in
// both directions and step kernels in those that the rules give:
//   32 x 2048 (1 round) 3856 / 5999 and 3149 / 5522;  128 x 1024 (2) 3361 / 5090
//   and 3171 / 5081;  256 x 512 (2) 1932 / 3573 and 1906 / 3372;  256 x 520 with
//   an input of 136 (3 forward, the backward as a product) 2438 / 4487 and 2102 /
//   3771
// Past the rules, products in both directions and step kernels forward: 64 x
// 1536 (2) 3467 / 5427 and 3556 / 5617, 64 x 2048 (2) 4398 / 6749 and 4423 /
// 7334, 192 x 1024 (3) 4586 / 6642 and 4677 / 6759; and per backward step,
// product and step kernel: 256 x 520 (3) 21.7 / 23.2, 512 x 512 (4) 25.4 / 28.8,
// 1024 x 256 (4) 27.2 / 29.9, 256 x 1024 (4) 35.7 / 42.0.
// With four wavefronts (k of at most 512) several workgroups share a compute
// unit and the step kernels stay ahead: 2048 x 256 forward 22.9 / 17.2, 4096 x 128
// 21.5 / 14.8, backward 54.7 / 46.0.
static int rounds(int64_t workgroups) { return int((workgroups + 255) / 256); }

bool lstm_step_fwd_wins(int B, int H, int E) {
  const int rows = B <= 16 ? 16 : 32;
  const int r = rounds(int64_t((B + rows - 1) / rows) * (H / 8));
  return E + H <= 512 || r == 1 || int64_t(r) * (E + H) <= 4096;
}

bool lstm_step_bwd_wins(int B, int H) {
  const int r = rounds(int64_t(lstm_step_row_blocks(B)) * ((H + 15) / 16));
  return 4 * H <= 512 || r == 1 || (r == 2 && H <= 1024);
}

void lstm_fwd_point(hipStream_t s, int B, int H, const float *zpart, int ns, const float *bias,
                    const float *c_prev, float *gates, void *h_out, float *c_out) {
  hipLaunchKernelGGL(k_lstm_fwd_point, dim3((B * H + 255) / 256), dim3(256), 0, s, B, H, zpart, ns, bias, c_prev,
                     gates, static_cast<__bf16 *>(h_out), c_out);
}

void lstm_step_fwd(hipStream_t s, int B, int H, int E, const void *x, const void *h, const void *w,
                   const float *bias, const float *c_prev, float *gates, void *h_out,
                   float *c_out) {
  const int K2 = h ? H : 0;
  const auto *xp = static_cast<const __bf16 *>(x), *hp = static_cast<const __bf16 *>(h),
             *wp = static_cast<const __bf16 *>(w);
  auto *ho = static_cast<__bf16 *>(h_out);
  // batches of at most 16 rows take 16-row tiles; a short k (at most 16 steps
  // of 32) four wavefronts instead of sixteen
#define CKPT_STEP_FWD(RT, NW)                                                                          \
  launch_timed(k_lstm_step_fwd<RT, NW>, dim3((B + 16 * RT - 1) / (16 * RT) * (H / 8)), dim3(64 * NW), 0, \
                     s, B, H, E, K2, xp, hp, wp, bias, c_prev, gates, ho, c_out)
  const bool few = E + H <= 512;  // of the shape, not of the step: the same order with and without h
  if (B <= 16) {
    if (few) CKPT_STEP_FWD(1, 4);
    else CKPT_STEP_FWD(1, 16);
  } else {
    if (few) CKPT_STEP_FWD(2, 4);
    else CKPT_STEP_FWD(2, 16);
  }
#undef CKPT_STEP_FWD
}

int lstm_step_row_blocks(int B) { return (B + 15) / 16; }
int lstm_point_row_blocks(int B) { return (B + 3) / 4; }

void lstm_bwd_point(hipStream_t s, int B, int H, const float *dhpart, int ns, const float *dc_in,
                    const float *gates, const float *c_t, const float *c_prev, const void *h_prev,
                    const void *h_t, void *dz, float *dc_prev, void *hp_copy, void *hc_copy, float *dbp) {
  hipLaunchKernelGGL(k_lstm_bwd_point, dim3((H + 63) / 64, lstm_point_row_blocks(B)), dim3(256), 0, s, B, H, dhpart,
                     ns, dc_in, gates, c_t, c_prev, static_cast<const __bf16 *>(h_prev),
                     static_cast<const __bf16 *>(h_t), static_cast<__bf16 *>(dz), dc_prev,
                     static_cast<__bf16 *>(hp_copy), static_cast<__bf16 *>(hc_copy), dbp);
}

void lstm_step_bwd(hipStream_t s, int B, int H, const void *dzn, const void *w,
                   const float *hpart, int ns, int64_t slice, const float *dc_in, const float *gates,
                   const float *c_t, const float *c_prev, const void *h_prev, const void *h_t, void *dz,
                   float *dc_prev, void *hp_copy, void *hc_copy, float *dbp) {
  const dim3 grid(lstm_step_row_blocks(B) * ((H + 15) / 16));
#define CKPT_STEP_BWD(NW)                                                                             \
  launch_timed(k_lstm_step_bwd<NW>, grid, dim3(64 * NW), 0, s, B, H, static_cast<const __bf16 *>(dzn), \
                     static_cast<const __bf16 *>(w), hpart, ns, slice, dc_in, gates, c_t, c_prev, \
                     static_cast<const __bf16 *>(h_prev), static_cast<const __bf16 *>(h_t),           \
                     static_cast<__bf16 *>(dz), dc_prev, static_cast<__bf16 *>(hp_copy),              \
                     static_cast<__bf16 *>(hc_copy), dbp)
  if (4 * H <= 512) CKPT_STEP_BWD(4);
  else CKPT_STEP_BWD(16);
#undef CKPT_STEP_BWD
}

void lstm_pack_gates(hipStream_t s, int E, int H, const float *wx, const float *wh, void *dst) {
  const auto run = [&](int rows, int qoff, const float *src) {
    hipLaunchKernelGGL(k_pack_gates, dim3(unsigned((int64_t(rows) / 2 * H + 255) / 256)), dim3(256), 0, s, H, rows / 8,
                       qoff, (E + H) / 8, src, static_cast<__bf16 *>(dst));
  };
  run(E, 0, wx);
  run(H, E / 8, wh);
}

void lstm_pack_rows(hipStream_t s, int H, const float *wh, void *dst) {
  hipLaunchKernelGGL(k_pack_rows, dim3(unsigned((int64_t(H) * H / 2 + 255) / 256)), dim3(256), 0, s, H, wh,
                     static_cast<__bf16 *>(dst));
}

int head_prep(hipStream_t s, int nu, int B, int V, const float *dlog, int64_t sd, void *dl, float *cs,
              float *db, bool first) {
  hipLaunchKernelGGL(k_head_prep, dim3((V + 31) / 32, nu), dim3(512), 0, s, B, V, dlog, sd,
                     static_cast<__bf16 *>(dl), cs, nu == 1 ? db : nullptr, first ? 1 : 0);
  if (nu == 1) return 1;
  hipLaunchKernelGGL(k_head_db, dim3((V + 255) / 256), dim3(256), 0, s, V, nu, cs, db, first ? 1 : 0);
  return 2;
}

}  // namespace ckpt
