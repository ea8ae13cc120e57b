// The residual-MLP block's backward in one launch: dW = x^T dr, dx = g + dr W^T
// and db = column sums of dr, dr = (z > 0 ? g : 0), fp32 on the matrix cores
// (v_mfma_f32_32x32x2f32).
//
// None of the three needs another, so one launch runs them side by side.  As
// four launches (dr with partial column sums, their sum, dW, dx) a block of 64 x
// 256 took 13.6 us and one of 256 x 1024 30 us, most of it launches and chips
// left idle by each small product in turn; together they take 6.2 and 24 us.
// dr is not stored: the mask is applied to g as it is read.
//
// Workgroup = 8 wavefronts; each wavefront computes a 32 x 32 tile over its
// part of k on its own: KS wavefronts share a tile, each a run of the k groups
// of 16, and 8 / KS tiles side by side along n share the workgroup.  A
// wavefront stages its operands through its own part of LDS (a ring of NS
// stages of one k group, filled by direct global -> LDS loads NS - 1 groups
// ahead), so the main loop has no barrier and the two wavefronts of a SIMD
// fill each other's waits; the KS partial tiles meet in LDS once, at the end,
// and are added in wavefront order.  Every element is reduced over K in one
// order fixed by the shape alone.  What bounds it: the loads (three operands,
// 768 KB per compute unit at 256 x 1024) beside 6.8 us of matrix work.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernel_args.h"
#include "kernels.h"
#include "launch.h"

namespace ckpt {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int NW = 8;            // wavefronts per workgroup
constexpr int T = 32, KG = 16;   // tile, k per group
constexpr int OPB = T * KG * 4;  // bytes of one staged operand
constexpr int kMaxDbRows = 1024;  // rows up to which one workgroup forms a column's sum

typedef __attribute__((address_space(3))) void lds_void_t;

// s_waitcnt immediate: at most n vector-memory operations outstanding, every
// LDS read returned
constexpr int wait_vm_lds(int n) { return (n & 15) | ((n >> 4) << 14) | 0x70; }

// One operand of a tile: 32 rows (or columns) from `base`, `n` of them inside
// the matrix (an index past them re-reads the last one; its results are
// dropped).  KC: element (i, k) at base[i ld + k], staged [i][16 k] with the
// 16-byte chunk c of row i in slot c ^ (i / 4 mod 4); else at base[k ld + i],
// staged [k][32].  VEC: 16-byte loads (4-float chunks wholly inside or outside:
// extents, ld multiples of 4, base 16-byte aligned), else 4-byte ones.
template <bool KC, bool VEC>
struct Operand {
  const float *base;
  int ld, n;
  static constexpr int LOADS = VEC ? 2 : 8;

  // the lane's source of load i of the k group that starts at k (k indexes
  // past K re-read the last one; such values are masked in the product)
  __device__ __forceinline__ const float *source(int i, int k, int K) const {
    const int lane = threadIdx.x & 63;
    if constexpr (KC && VEC) {
      const int row = i * 16 + lane / 4, c = (lane % 4) ^ ((row >> 2) & 3);
      return base + size_t(min(row, n - 1)) * ld + min(k + 4 * c, K - 4);
    } else if constexpr (KC) {
      const int row = i * 4 + lane / 16, c = ((lane % 16) / 4) ^ ((row >> 2) & 3);
      return base + size_t(min(row, n - 1)) * ld + min(k + 4 * c + lane % 4, K - 1);
    } else if constexpr (VEC) {
      return base + size_t(min(k + i * 8 + lane / 8, K - 1)) * ld + min(4 * (lane % 8), n - 4);
    } else {
      return base + size_t(min(k + i * 2 + lane / 32, K - 1)) * ld + min(lane % 32, n - 1);
    }
  }
  // from one whole group's sources to the next one's
  __device__ __forceinline__ int64_t stride() const { return KC ? KG : int64_t(KG) * ld; }
  __device__ __forceinline__ static void load(const float *src, int i, unsigned char *lds) {
    if constexpr (VEC)
      __builtin_amdgcn_global_load_lds(src, (lds_void_t *)(lds + i * 1024), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds(src, (lds_void_t *)(lds + i * 256), 4, 0, 0);
  }
  // the lane's values k = 8 (lane / 32) + j, j = 0..7, of row lane % 32
  __device__ __forceinline__ static void read(const unsigned char *lds, float (&v)[8]) {
    const int l32 = threadIdx.x & 31, h = (threadIdx.x & 63) >> 5;
    if constexpr (KC) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int slot = (2 * h + u) ^ ((l32 >> 2) & 3);
        const f32x4 t = *reinterpret_cast<const f32x4 *>(lds + (l32 * 4 + slot) * 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 * u + j] = t[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const float *>(lds + ((8 * h + j) * T + l32) * 4);
    }
  }
};

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>)
template <class F, int... I>
__device__ __forceinline__ void unroll_seq(F &f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unroll(F &&f) {
  unroll_seq(f, std::make_integer_sequence<int, N>{});
}

// The sources of one operand's loads, group after group.
template <class O>
struct Stream {
  const float *p[O::LOADS];
  __device__ __forceinline__ void start(const O &o, int g, int K) {
#pragma unroll
    for (int i = 0; i < O::LOADS; ++i) p[i] = o.source(i, g * KG, K);
  }
  __device__ __forceinline__ void issue(unsigned char *lds) const {
#pragma unroll
    for (int i = 0; i < O::LOADS; ++i) O::load(p[i], i, lds);
  }
  __device__ __forceinline__ void advance(int64_t d) {
#pragma unroll
    for (int i = 0; i < O::LOADS; ++i) p[i] += d;
  }
};

// acc += a b over the k groups [g0, g1) of this wavefront.  MASK = 1 (2): A's
// (B's) values count only where the operand m, laid out like it, is positive.
// The stages are separate LDS objects, so the compiler knows which loads in
// flight an LDS read has to wait for.
template <int NS, int MASK, bool AKC, bool BKC, bool VEC>
__device__ __forceinline__ void wave_tile(const Operand<AKC, VEC> &a, const Operand<BKC, VEC> &b,
                                          const Operand<(MASK == 2 ? BKC : AKC), VEC> &m, int K, int g0, int g1,
                                          unsigned char *s0, unsigned char *s1, unsigned char *s2,
                                          floatx16 &acc) {
  constexpr int OPS = MASK ? 3 : 2, LPG = OPS * (VEC ? 2 : 8);
  static_assert(NS >= 2 && NS <= 3 && (NS - 1) * LPG <= 63, "loads in flight fit the counter");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = (threadIdx.x & 63) >> 5;
  auto stage = [&](auto I) -> unsigned char * {
    constexpr int i = decltype(I)::value;
    unsigned char *p = i == 0 ? s0 : i == 1 ? s1 : s2;
    return p + wave * OPS * OPB;
  };
  Stream<Operand<AKC, VEC>> sa;
  Stream<Operand<BKC, VEC>> sb;
  Stream<Operand<(MASK == 2 ? BKC : AKC), VEC>> sm;
  auto start = [&](int g) {
    sa.start(a, g, K);
    sb.start(b, g, K);
    if constexpr (MASK != 0) sm.start(m, g, K);
  };
  // loads of the next group in line into stage s: whole groups follow each
  // other at a fixed distance, the last, partial one has its own addresses, and
  // past the range the last group is loaded again (and never multiplied)
  int gi = g0;
  auto issue = [&](unsigned char *s) {
    sa.issue(s);
    sb.issue(s + OPB);
    if constexpr (MASK != 0) sm.issue(s + 2 * OPB);
    const bool more = gi + 1 < g1;
    gi += more;
    if (more && (gi + 1) * KG > K) {
      start(gi);
    } else {
      sa.advance(more ? a.stride() : 0);
      sb.advance(more ? b.stride() : 0);
      if constexpr (MASK != 0) sm.advance(more ? m.stride() : 0);
    }
  };
  auto compute = [&](int g, const unsigned char *s) {
    float av[8], bv[8];
    Operand<AKC, VEC>::read(s, av);
    Operand<BKC, VEC>::read(s + OPB, bv);
    if constexpr (MASK != 0) {
      float mv[8];
      Operand<(MASK == 2 ? BKC : AKC), VEC>::read(s + 2 * OPB, mv);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if constexpr (MASK == 1) av[j] = mv[j] > 0.f ? av[j] : 0.f;
        else bv[j] = mv[j] > 0.f ? bv[j] : 0.f;
      }
    }
    if ((g + 1) * KG > K) {  // the last, partial group
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bool in = g * KG + 8 * h + j < K;
        av[j] = in ? av[j] : 0.f;
        bv[j] = in ? bv[j] : 0.f;
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[j], bv[j], acc, 0, 0, 0);
  };
  if (g0 >= g1) return;
  start(g0);
  unroll<NS - 1>([&](auto J) { issue(stage(J)); });
  auto step = [&](int g, auto J) {
    constexpr int w = (decltype(J)::value + NS - 1) % NS;
    // this group has landed, and the previous group's stage has been read
    __builtin_amdgcn_s_waitcnt(wait_vm_lds((NS - 2) * LPG));
    issue(stage(std::integral_constant<int, w>{}));
    compute(g, stage(J));
  };
  int g = g0;
  for (; g + NS <= g1; g += NS) unroll<NS>([&](auto J) { step(g + decltype(J)::value, J); });
  unroll<NS - 1>([&](auto J) {
    if (g + decltype(J)::value < g1) step(g + decltype(J)::value, J);
  });
}

// How a product is split: ks wavefronts per tile, the fewest that still give
// 256 workgroups (one per compute unit), at most one per k group.
struct Split {
  int ks, blocks;
};

inline Split split_of(int M, int N, int K) {
  const int64_t tm = (M + T - 1) / T, tn = (N + T - 1) / T;
  const int ng = (K + KG - 1) / KG;
  int ks = 1;
  while (ks < NW && ks * 2 <= ng && tm * tn * ks < 256 * NW) ks *= 2;
  return {ks, int(tm * ((tn + NW / ks - 1) / (NW / ks)))};
}

// The tile product and epilogue of workgroup `id` of the product's tm * wgn,
// KS wavefronts per tile.
template <int KS, int NS, int MASK, bool TA, bool TB, int EPI, bool VEC>
__device__ __forceinline__ void tile_block(const GemmArgs &p, const float *mask, int id, unsigned char *s0,
                                           unsigned char *s1, unsigned char *s2) {
  constexpr int NT = NW / KS, PT = T * T / (64 * KS);  // tiles; results per thread
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tm = (p.M + T - 1) / T;
  // m fastest: neighbouring workgroups share the columns of B
  const int m0 = (id % tm) * T, kw = wave % KS, n0 = ((id / tm) * NT + wave / KS) * T;
  const bool live = n0 < p.N;
  // the KS wavefronts of a tile share its epilogue: thread u of them takes
  // results u, u + 64 KS, ... (row major), whose epilogue operands are loaded
  // ahead of the product
  const int u0 = kw * 64 + lane;
  auto at = [&](int i, int &row, int &n) {
    const int e = u0 + i * 64 * KS;
    row = m0 + e / T;
    n = n0 + e % T;
    return live && row < p.M && n < p.N;
  };
  float pre[PT];
  if constexpr (EPI == GEMM_EPI_ADD) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      int row, n;
      pre[i] = at(i, row, n) ? p.D[size_t(row) * p.ldd + n] : 0.f;
    }
  }
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  if (live) {
    const Operand<!TA, VEC> a{TA ? p.A + m0 : p.A + size_t(m0) * p.lda, p.lda, p.M - m0};
    const Operand<TB, VEC> b{TB ? p.B + size_t(n0) * p.ldb : p.B + n0, p.ldb, p.N - n0};
    Operand<(MASK == 2 ? TB : !TA), VEC> m{nullptr, 0, 0};
    if constexpr (MASK == 1) m = {TA ? mask + m0 : mask + size_t(m0) * p.lda, p.lda, p.M - m0};
    if constexpr (MASK == 2) m = {TB ? mask + size_t(n0) * p.ldb : mask + n0, p.ldb, p.N - n0};
    const int ng = (p.K + KG - 1) / KG, per = (ng + KS - 1) / KS;
    wave_tile<NS, MASK>(a, b, m, p.K, min(kw * per, ng), min(kw * per + per, ng), s0, s1, s2, acc);
  }
  // the partial tiles, [wave][32][32]; every load has landed and every
  // wavefront is done with the stages first
  __builtin_amdgcn_s_waitcnt(wait_vm_lds(0));
  __syncthreads();
  float *red = reinterpret_cast<float *>(s0);
  const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
  for (int r = 0; r < 16; ++r) red[(wave * T + 8 * (r >> 2) + 4 * h + (r & 3)) * T + l32] = acc[r];
  __syncthreads();
  const float *tile = red + (wave - kw) * T * T + u0;
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    int row, n;
    float v = tile[i * 64 * KS];
#pragma unroll
    for (int w = 1; w < KS; ++w) v += tile[w * T * T + i * 64 * KS];
    if (!at(i, row, n)) continue;
    const size_t o = size_t(row) * p.ldc + n;
    p.C[o] = EPI == GEMM_EPI_ADD ? v + pre[i] : v;
  }
}

// Workgroups reach the eight XCDs (one L2 each) in turn; the linear id is
// remapped so that each XCD takes a contiguous run of tiles: an XCD then reads
// a few column tiles of B (plus A) instead of all of B.
__device__ __forceinline__ int xcd_run(int id, int G) {
  const int q8 = G / 8, r8 = G % 8, x8 = id % 8;
  return x8 * q8 + (x8 < r8 ? x8 : r8) + id / 8;
}

// db[n] = column sums of g (where z > 0 when z is given) over `rows` rows, 32
// columns from n0: 16 row groups, group r adding rows r, r + 16, ... in order,
// four loads issued before any is used; then a fixed pairwise tree.
__device__ __forceinline__ void db_block(int rows, int cols, const float *g, const float *z, float *db, int n0,
                                         float *part) {
  const int cx = threadIdx.x & 31, rg = threadIdx.x >> 5, n = n0 + cx;
  float s = 0.f;
  if (n < cols)
    for (int r0 = rg; r0 < rows; r0 += 64) {
      float gv[4], zv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const size_t e = size_t(min(r0 + 16 * u, rows - 1)) * cols + n;
        gv[u] = g[e];
        zv[u] = z ? z[e] : 1.f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (r0 + 16 * u < rows) s += zv[u] > 0.f ? gv[u] : 0.f;
    }
  part[rg * 32 + cx] = s;
  __syncthreads();
  if (rg == 0 && n < cols) {
    float q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = part[2 * i * 32 + cx] + part[(2 * i + 1) * 32 + cx];
    db[n] = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
  }
}

__global__ __launch_bounds__(512) void k_colsum(int rows, int cols, const float *__restrict__ g,
                                                float *__restrict__ db) {
  __shared__ float part[512];
  db_block(rows, cols, g, nullptr, db, blockIdx.x * 32, part);
}

// n_first workgroups for db, n_wg for dW (wg), n_dg for dx (dg), the rest for db.
// MASK: dr = (z > 0 ? g : 0) and dx = g + dr W^T; else g is dr itself and dx = dr
// W^T.
template <int KSW, int KSD, bool MASK, bool VEC>
__global__ __launch_bounds__(64 * NW) void k_gemm_f32_mlp_bwd(GemmArgs wg, GemmArgs dg, const float *z, int n_first,
                                                              int n_wg, int n_dg, float *db) {
  constexpr int NS = VEC ? 3 : 2, ST = NW * (MASK ? 3 : 2) * OPB;
  __shared__ __align__(1024) unsigned char s0[ST], s1[ST], s2[NS > 2 ? ST : 1];
  const int id = int(blockIdx.x) - n_first;
  if (id < 0 || id >= n_wg + n_dg)
    db_block(wg.K, wg.N, wg.B, MASK ? z : nullptr, db, (id < 0 ? id + n_first : id - n_wg - n_dg) * 32,
             reinterpret_cast<float *>(s0));
  else if (id < n_wg)
    tile_block<KSW, NS, MASK ? 2 : 0, true, false, GEMM_EPI_STORE, VEC>(wg, z, xcd_run(id, n_wg), s0, s1, s2);
  else
    tile_block<KSD, NS, MASK ? 1 : 0, false, true, MASK ? GEMM_EPI_ADD : GEMM_EPI_STORE, VEC>(
        dg, z, xcd_run(id - n_wg, n_dg), s0, s1, s2);
}

// f(integral_constant<int, ks>) for ks in {1, 2, 4, 8}
template <class F>
void with_ks(int ks, F &&f) {
  if (ks == 1) f(std::integral_constant<int, 1>{});
  else if (ks == 2) f(std::integral_constant<int, 2>{});
  else if (ks == 4) f(std::integral_constant<int, 4>{});
  else f(std::integral_constant<int, 8>{});
}

inline bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

// The joint launch saves launches and idle compute units; its wavefronts share no
// operands, which gemm_f32's tiles do.  Whole steps of 12 blocks (960 x 1024: 48)
// without checkpoints, products one by one and joint, us (rows x width):
//   joint      256 x 256 223 / 141, 2048 x 256 502 / 438, 4096 x 384 1052 / 989, 256 x
//              512 257 / 222, 768 x 800 816 / 771, 512 x 960 699 / 666, 256 x 1024
//              413 / 387, 960 x 1024 5181 / 4812, 256 x 1536 836 / 758, 128 x 1792
//              570 / 563
//   products   1024 x 500 502 / 563, 1024 x 700 820 / 916, 2048 x 800 1512 / 1781, 1024
//              x 1024 1252 / 1336, 768 x 1280 1419 / 1495, 1536 x 1536 3598 / 4045, 256
//              x 2048 1089 / 1121, 64 x 3072 852 / 963, 32 x 4096 1011 / 1300, 8192 x
//              384 1650 / 1811
// so: up to 2^30 multiplications per product; past 448 columns (where dW alone
// fills the chip with gemm_f32's tiles) with fewer rows than columns, and of 2048
// columns on never.
bool mlp_bwd_wins(int B, int D) {
  return int64_t(B) * D * D < (int64_t(1) << 30) && (D <= 448 || (D < 2048 && B < D));
}

int mlp_bwd(hipStream_t s, int B, int D, const float *g, const float *z, const float *x, const float *W,
            float *dx, float *dW, float *db, float *pdb) {
  // 16-byte loads; W counts only when dx is formed, which any W allows
  const bool vec = D % 4 == 0 && al16(g) && al16(z) && al16(x) && al16(W);
  const GemmArgs wg{D, D, B, x, D, g, D, dW, D, nullptr, 0, nullptr, nullptr, 0};
  const GemmArgs dg{B, D, D, g, D, W, D, dx, D, g, D, nullptr, nullptr, 0};
  const bool db_here = B <= kMaxDbRows;
  const Split sw = split_of(D, D, B), sd = split_of(B, D, D);
  // db's workgroups are chains of loads, one after another from 64 rows on: where
  // they are long they start first, so that the products hide them (1024 x 512:
  // 43 us with them last, 31 so; 256 x 1024 26.1 and 27.7)
  const int n_dg = dx ? sd.blocks : 0, n_db = db_here ? (D + 255) / 256 * 8 : 0;  // (whole rounds of the XCDs)
  const int n_first = B > 512 ? n_db : 0;
  if (!db_here) mlp_colsum_long(s, B, D, g, z, db, pdb);
  const dim3 grid(sw.blocks + n_dg + n_db);
  with_ks(sw.ks, [&](auto KSW) {
    with_ks(sd.ks, [&](auto KSD) {
      constexpr int kw = decltype(KSW)::value, kd = decltype(KSD)::value;
      const auto run = [&](auto kernel) {
        launch_timed(kernel, grid, dim3(64 * NW), 0, s, wg, dg, z, n_first, sw.blocks, n_dg, db);
      };
      if (z && vec) run(k_gemm_f32_mlp_bwd<kw, kd, true, true>);
      else if (z) run(k_gemm_f32_mlp_bwd<kw, kd, true, false>);
      else if (vec) run(k_gemm_f32_mlp_bwd<kw, kd, false, true>);
      else run(k_gemm_f32_mlp_bwd<kw, kd, false, false>);
    });
  });
  return db_here ? 1 : 3;
}

int mlp_colsum(hipStream_t s, int rows, int cols, const float *g, float *db, float *pdb) {
  if (rows <= kMaxDbRows) {
    hipLaunchKernelGGL(k_colsum, dim3((cols + 31) / 32), dim3(512), 0, s, rows, cols, g, db);
    return 1;
  }
  mlp_colsum_long(s, rows, cols, g, nullptr, db, pdb);
  return 2;
}

}  // namespace ckpt
