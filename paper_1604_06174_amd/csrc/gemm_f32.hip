// fp32 GEMM on CDNA4 matrix cores (v_mfma_f32_32x32x2f32).
//
//   C[M,N] = epilogue( op(A)[M,K] * op(B)[K,N] )
//   op(A)(m,k) = TA ? A[k*lda + m] : A[m*lda + k]
//   op(B)(k,n) = TB ? B[n*ldb + k] : B[k*ldb + n]
//
// Two kernels:
//   k_gemm_f32<..>    64 x 64 tiles, four wavefronts in a 2 x 2 grid of 32 x 32
//     accumulators, k slices of 32 staged k-contiguous in LDS ([m][k] and
//     [n][k], rows padded by 4 floats), double-buffered, with the global loads
//     of the next two slices in flight in registers; for products with at
//     least 256 such tiles (one per compute unit).
//   k_gemm_f32_ks<..> 32 x 32 tiles for smaller products, k slices of 128 that
//     four wavefronts split into quarters; their accumulators are added in
//     LDS in wave order ((w0 + w1) + w2) + w3.  One such workgroup per compute
//     unit has to keep the matrix cores busy alone, so eight more wavefronts
//     do nothing but load: slices go from global memory straight into a ring
//     of four LDS stages (one barrier per slice), and the four that multiply
//     read a slice's operands while they multiply the one before.  With four
//     wavefronts doing both (and operands passing through registers) 256 x
//     1024 x 1024 took 12.2 us as a block's forward (9.9 now), 64 x 256 x 256
//     5.0 (4.5) and 200 x 275 x 275, without 16-byte loads, 10.2 (6.3); 0.54
//     GFLOP of matrix work is 3.5 us of the first and a launch 2.3.
// Within a slice's 32-wide k range of a wavefront, MFMA j takes k = 16 h + j in
// lane half h (h = lane / 32) for both operands -- a fixed permutation of the
// reduction, so each lane reads 16 consecutive floats of a k-contiguous
// operand.  Every output element is reduced over K in one order fixed by the
// shape alone.
//
// Epilogues:
//   STORE    C = acc
//   ADD      C = acc + D                      (backward: dx = dy + dr W^T)
//   MLPFWD   Z = acc + bias;  C = A + relu(Z) (residual block y = x + relu(xW+b);
//                                               requires !TA and K == N)
//   BIAS     C = acc + bias
#include <hip/hip_runtime.h>

#include "common.h"
#include "kernel_args.h"
#include "kernels.h"
#include "launch.h"

namespace ckpt {

typedef float floatx16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int PAD = 4;


// 4 KB of zeros in device memory: an element outside its operand is loaded
// from here (16 bytes per thread, spread over many cache lines), so no loaded
// value is masked afterwards and nothing waits for a load before it is
// written to LDS a slice later.
static __device__ __align__(16) const float g_zero_area[1024] = {};
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const f32x4 global_f32x4;
typedef __attribute__((address_space(1))) const float global_float;

// 4 consecutive elements of a row-major [rows, cols] matrix, zero outside.
// Branch-free (an outside address is replaced by the zero chunk), so the loads
// of a slice stay in flight together; the pointers are cast to the global
// address space so that the loads are global loads.  VEC: one 16-byte load;
// needs ld and cols multiples of 4 and a 16-byte aligned base, so a chunk is
// either wholly inside or wholly outside.
template <bool VEC>
__device__ __forceinline__ float4 ld4(const float *base, int row, int col, int rows, int cols,
                                      int ld) {
  if (VEC) {
    const bool ok = (row < rows) & (col < cols);
    const float *z = g_zero_area + 4 * (threadIdx.x & 255);
    const f32x4 v = *(global_f32x4 *)(ok ? base + size_t(row) * ld + col : z);
    return make_float4(v.x, v.y, v.z, v.w);
  }
  float r[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool ok = (row < rows) & (col + j < cols);
    r[j] = *(global_float *)(ok ? base + size_t(row) * ld + col + j : g_zero_area + 4 * (threadIdx.x & 255));
  }
  return make_float4(r[0], r[1], r[2], r[3]);
}

// What the epilogue of element (m, n) reads besides the product, and the
// element itself.
template <int EPI>
__device__ __forceinline__ float epi_load(const GemmArgs &p, int m, int n) {
  if (EPI == GEMM_EPI_ADD) return p.D[size_t(m) * p.ldd + n];
  if (EPI == GEMM_EPI_MLPFWD) return p.A[size_t(m) * p.lda + n];
  return 0.f;
}
template <int EPI>
__device__ __forceinline__ void emit(const GemmArgs &p, int m, int n, float v, float pre, float bias) {
  float c = v;
  if (EPI == GEMM_EPI_ADD) c = v + pre;
  if (EPI == GEMM_EPI_BIAS) c = v + bias;
  if (EPI == GEMM_EPI_MLPFWD) {
    const float z = v + bias;
    p.Z[size_t(m) * p.ldz + n] = z;
    c = pre + fmaxf(z, 0.f);
  }
  p.C[size_t(m) * p.ldc + n] = c;
}

// Workgroups reach the eight XCDs (one L2 each) in turn; the linear id is
// remapped so that each XCD takes a contiguous run of tiles, m fastest: an
// XCD then reads a few column tiles of B (plus A) instead of all of B.
__device__ __forceinline__ void tile_of_block(int &tm, int &tn) {
  const int G = gridDim.x * gridDim.y, id = blockIdx.x + gridDim.x * blockIdx.y;
  const int q8 = G / 8, r8 = G % 8, x8 = id % 8;
  const int L = x8 * q8 + (x8 < r8 ? x8 : r8) + id / 8;
  tm = L % gridDim.y;
  tn = L / gridDim.y;
}

template <bool TA, bool TB, int EPI, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmArgs p) {
  constexpr int BM = 64, BN = 64;                  // block tile
  constexpr int BK = 32;                           // k slice
  constexpr int LD = BK + PAD;                     // LDS row stride (floats)
  constexpr int NCH = BM * BK / 4 / 256;           // float4 chunks per thread per operand
  static_assert(NCH * 256 * 4 == BM * BK, "tile / thread mismatch");
  __shared__ __attribute__((aligned(16))) float smem[2 * (BM + BN) * LD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int tm, tn;
  tile_of_block(tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;

  auto gload = [&](float4 (&ra)[NCH], float4 (&rb)[NCH], int k0) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int ch = tid + 256 * c;
      if (!TA) {  // A row-major [M,K]: a chunk is 4 k's of one row
        ra[c] = ld4<VEC>(p.A, m0 + ch / (BK / 4), k0 + (ch % (BK / 4)) * 4, p.M, p.K, p.lda);
      } else {    // A stored [K,M]: a chunk is 4 m's of one k
        ra[c] = ld4<VEC>(p.A, k0 + ch / (BM / 4), m0 + (ch % (BM / 4)) * 4, p.K, p.M, p.lda);
      }
      if (TB) {   // B stored [N,K]: 4 k's of one n
        rb[c] = ld4<VEC>(p.B, n0 + ch / (BK / 4), k0 + (ch % (BK / 4)) * 4, p.N, p.K, p.ldb);
      } else {    // B row-major [K,N]: 4 n's of one k
        rb[c] = ld4<VEC>(p.B, k0 + ch / (BN / 4), n0 + (ch % (BN / 4)) * 4, p.K, p.N, p.ldb);
      }
    }
  };
  auto sstore = [&](const float4 (&ra)[NCH], const float4 (&rb)[NCH], int buf) {
    float *As = smem + buf * (BM + BN) * LD, *Bs = As + BM * LD;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int ch = tid + 256 * c;
      if (!TA) {
        *reinterpret_cast<float4 *>(As + (ch / (BK / 4)) * LD + (ch % (BK / 4)) * 4) = ra[c];
      } else {
        const int k = ch / (BM / 4), m = (ch % (BM / 4)) * 4;
        As[(m + 0) * LD + k] = ra[c].x;
        As[(m + 1) * LD + k] = ra[c].y;
        As[(m + 2) * LD + k] = ra[c].z;
        As[(m + 3) * LD + k] = ra[c].w;
      }
      if (TB) {
        *reinterpret_cast<float4 *>(Bs + (ch / (BK / 4)) * LD + (ch % (BK / 4)) * 4) = rb[c];
      } else {
        const int k = ch / (BN / 4), n = (ch % (BN / 4)) * 4;
        Bs[(n + 0) * LD + k] = rb[c].x;
        Bs[(n + 1) * LD + k] = rb[c].y;
        Bs[(n + 2) * LD + k] = rb[c].z;
        Bs[(n + 3) * LD + k] = rb[c].w;
      }
    }
  };

  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;

  const int h = lane >> 5, l32 = lane & 31;
  auto compute = [&](int buf) {
    const float *As = smem + buf * (BM + BN) * LD, *Bs = As + BM * LD;
    const float *pa = As + (wm + l32) * LD + h * 16;
    const float *pb = Bs + (wn + l32) * LD + h * 16;
    float4 a4[4], b4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a4[q] = *reinterpret_cast<const float4 *>(pa + 4 * q);
      b4[q] = *reinterpret_cast<const float4 *>(pb + 4 * q);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[q].x, b4[q].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[q].y, b4[q].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[q].z, b4[q].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[q].w, b4[q].w, acc, 0, 0, 0);
    }
  };

  // slices kt+1 and kt+2 are in flight in registers while slice kt is
  // multiplied out of LDS buffer kt & 1.  The loop body has no branches (a
  // branch there makes the compiler wait for every load at each iteration):
  // it runs while two more slices follow, and the last one or two slices are
  // multiplied after it.
  const int nk = (p.K + BK - 1) / BK;
  // k origin of slice s; a slice past K re-reads the last one (real,
  // spread-out addresses; it is never multiplied)
  auto kslice = [&](int s) { return max(0, min(s, nk - 1)) * BK; };
  float4 ra0[NCH], rb0[NCH], ra1[NCH], rb1[NCH];
  gload(ra0, rb0, kslice(0));
  gload(ra1, rb1, kslice(1));
  sstore(ra0, rb0, 0);
  __syncthreads();
  int kt = 0;
  for (; kt + 2 < nk; kt += 2) {
    gload(ra0, rb0, kslice(kt + 2));
    compute(0);
    sstore(ra1, rb1, 1);
    __syncthreads();
    gload(ra1, rb1, kslice(kt + 3));
    compute(1);
    sstore(ra0, rb0, 0);
    __syncthreads();
  }
  compute(0);  // slice kt
  if (kt + 1 < nk) {
    sstore(ra1, rb1, 1);
    __syncthreads();
    compute(1);
  }

  // accumulator register r of a lane holds element (row, col) of its 32x32 tile
  constexpr bool HAS_BIAS = EPI == GEMM_EPI_BIAS || EPI == GEMM_EPI_MLPFWD;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + wm + 8 * (r >> 2) + 4 * h + (r & 3), n = n0 + wn + l32;
    if (m < p.M && n < p.N) emit<EPI>(p, m, n, acc[r], epi_load<EPI>(p, m, n), HAS_BIAS ? p.bias[n] : 0.f);
  }
}

// ---- 32 x 32 tiles, k split over four wavefronts, eight more that load ----
constexpr int T = 32, SK = 128;         // tile, k slice
constexpr int MW = 4, LW = 8;           // wavefronts that multiply, that load
constexpr int NS = 4;                   // stages
constexpr int OPB = T * SK * 4;         // bytes of one staged operand

typedef __attribute__((address_space(3))) void lds_void_t;

// s_waitcnt immediate: at most n vector-memory operations outstanding
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0xF70; }

// One operand of a tile: 32 rows (or columns) from `base`, n of them inside the
// matrix (an index past them re-reads the last one; its results are dropped).
// KC: element (i, k) at base[i ld + k], staged [i][128 k] with the 16-byte chunk
// c of row i in slot c ^ (i mod 16); else at base[k ld + i], staged [k'][32]
// with k' = k with its bit 0 flipped where bit 4 is set, so that the two lane
// halves of a read, 16 k apart, use different banks.  VEC: 16-byte loads, else
// 4-byte ones.  A k index past K re-reads the last one (masked in the product).
template <bool KC, bool VEC>
struct Operand {
  const float *base;
  int ld, n;
  static constexpr int LOADS = OPB / (VEC ? 1024 : 256) / LW;  // per loading wavefront
  __device__ __forceinline__ void issue(int w, int k0, int K, unsigned char *lds) const {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int u = w * LOADS + i;  // the operand's load instruction
      const float *src;
      if constexpr (KC && VEC) {
        const int row = u * 2 + lane / 32, c = (lane % 32) ^ (row & 15);
        src = base + size_t(min(row, n - 1)) * ld + min(k0 + 4 * c, K - 4);
      } else if constexpr (KC) {
        const int row = u / 2, e = u % 2 * 64 + lane, c = (e / 4) ^ (row & 15);
        src = base + size_t(min(row, n - 1)) * ld + min(k0 + 4 * c + e % 4, K - 1);
      } else if constexpr (VEC) {
        const int kp = u * 8 + lane / 8, k = kp ^ ((kp >> 4) & 1);
        src = base + size_t(min(k0 + k, K - 1)) * ld + min(4 * (lane % 8), n - 4);
      } else {
        const int kp = u * 2 + lane / 32, k = kp ^ ((kp >> 4) & 1);
        src = base + size_t(min(k0 + k, K - 1)) * ld + min(lane % 32, n - 1);
      }
      if constexpr (VEC)
        __builtin_amdgcn_global_load_lds(src, (lds_void_t *)(lds + u * 1024), 16, 0, 0);
      else
        __builtin_amdgcn_global_load_lds(src, (lds_void_t *)(lds + u * 256), 4, 0, 0);
    }
  }
  // wavefront kw's values k = 32 kw + 16 (lane / 32) + j, j = 0..15, of row lane % 32
  __device__ __forceinline__ static void read(const unsigned char *lds, int kw, float (&v)[16]) {
    const int l32 = threadIdx.x & 31, h = (threadIdx.x & 63) >> 5;
    if constexpr (KC) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int slot = (8 * kw + 4 * h + q) ^ (l32 & 15);
        const f32x4 t = *reinterpret_cast<const f32x4 *>(lds + (l32 * (SK / 4) + slot) * 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 * q + j] = t[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int k = 32 * kw + 16 * h + j;
        v[j] = *reinterpret_cast<const float *>(lds + ((k ^ h) * T + l32) * 4);
      }
    }
  }
};

template <bool TA, bool TB, int EPI, bool VEC>
__global__ __launch_bounds__(64 * (MW + LW)) void k_gemm_f32_ks(GemmArgs p) {
  __shared__ __align__(1024) unsigned char s0[2 * OPB], s1[2 * OPB], s2[2 * OPB], s3[2 * OPB];
  typedef Operand<!TA, VEC> OA;
  typedef Operand<TB, VEC> OB;
  constexpr int LPS = OA::LOADS + OB::LOADS;  // loads of a stage per loading wavefront
  static_assert((NS - 2) * LPS <= 63, "loads in flight fit the counter");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  tile_of_block(tm, tn);
  const int m0 = tm * T, n0 = tn * T;
  const int nk = (p.K + SK - 1) / SK;
  auto stage = [&](int t) -> unsigned char * {
    t &= NS - 1;
    return t == 0 ? s0 : t == 1 ? s1 : t == 2 ? s2 : s3;
  };
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  // thread tid < 256 writes rows tid / 32 + 8 i of column tid mod 32; what it
  // reads for that is loaded ahead of the product
  constexpr bool HAS_BIAS = EPI == GEMM_EPI_BIAS || EPI == GEMM_EPI_MLPFWD;
  const int em = m0 + tid / T, en = n0 + tid % T;
  float pre[4], bias = 0.f;
  if (wave < MW) {
    if (HAS_BIAS && en < p.N) bias = p.bias[en];
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[i] = em + 8 * i < p.M && en < p.N ? epi_load<EPI>(p, em + 8 * i, en) : 0.f;
  }
  // Slice t sits in stage t mod NS.  Barrier t (t = 0 .. nk - 1) says that slice
  // t has landed and that slice t - 1 is in the multiplying wavefronts'
  // registers, so its stage may take slice t + NS - 1.
  if (wave >= MW) {
    const int w = wave - MW;
    const OA a{TA ? p.A + m0 : p.A + size_t(m0) * p.lda, p.lda, p.M - m0};
    const OB b{TB ? p.B + size_t(n0) * p.ldb : p.B + n0, p.ldb, p.N - n0};
    auto issue = [&](int t) {
      a.issue(w, t * SK, p.K, stage(t));
      b.issue(w, t * SK, p.K, stage(t) + OPB);
    };
    for (int t = 0; t < NS - 1 && t < nk; ++t) issue(t);
    for (int t = 0; t < nk; ++t) {
      const int ahead = nk - 1 - t;  // slices in flight after slice t
      if (ahead >= 2) __builtin_amdgcn_s_waitcnt(wait_vm(2 * LPS));
      else if (ahead == 1) __builtin_amdgcn_s_waitcnt(wait_vm(LPS));
      else __builtin_amdgcn_s_waitcnt(wait_vm(0));
      __builtin_amdgcn_s_barrier();
      if (t + NS - 1 < nk) issue(t + NS - 1);
    }
  } else {
    const int h = lane >> 5;
    float a0[16], b0[16], a1[16], b1[16];
    auto read = [&](int t, float (&av)[16], float (&bv)[16]) {
      __builtin_amdgcn_s_waitcnt(0xC07F);  // the slice before is in registers
      __builtin_amdgcn_s_barrier();
      OA::read(stage(t), wave, av);
      OB::read(stage(t) + OPB, wave, bv);
    };
    auto mul = [&](int t, float (&av)[16], float (&bv)[16]) {
      if ((t + 1) * SK > p.K) {  // the last, partial slice
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const bool in = t * SK + 32 * wave + 16 * h + j < p.K;
          av[j] = in ? av[j] : 0.f;
          bv[j] = in ? bv[j] : 0.f;
        }
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[j], bv[j], acc, 0, 0, 0);
    };
    read(0, a0, b0);
    int t = 1;
    for (; t + 1 < nk; t += 2) {
      read(t, a1, b1);
      mul(t - 1, a0, b0);
      read(t + 1, a0, b0);
      mul(t, a1, b1);
    }
    if (t < nk) {
      read(t, a1, b1);
      mul(t - 1, a0, b0);
      mul(t, a1, b1);
    } else {
      mul(t - 1, a0, b0);
    }
  }
  // the four quarters, added in wave order, in the first stage's place (every
  // load has landed, and a barrier says every wavefront is done with the stages)
  __syncthreads();
  float *red = reinterpret_cast<float *>(s0);  // [4][32][32]
  if (wave < MW) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      red[(wave * T + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * T + (lane & 31)] = acc[r];
  }
  __syncthreads();
  if (wave < MW) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + i * 64 * MW;
      const float v = ((red[e] + red[T * T + e]) + red[2 * T * T + e]) + red[3 * T * T + e];
      if (em + 8 * i < p.M && en < p.N) emit<EPI>(p, em + 8 * i, en, v, pre[i], bias);
    }
  }
}

template <bool TA, bool TB, int EPI>
void launch(const GemmArgs &a, bool vec, hipStream_t s) {
  const auto run = [&](auto kernel, int tile, int threads) {
    launch_timed(kernel, dim3((a.N + tile - 1) / tile, (a.M + tile - 1) / tile), dim3(threads), 0, s, a);
  };
  // 64 x 64 tiles when they alone give a workgroup per compute unit (up to there
  // the loading wavefronts hold their own at several workgroups per unit too: a
  // block's forward of 512 x 1024 18.4 us without them, 18.0 with, 448 x 2048 60.7
  // and 58.3, 960 x 1024 34.3 and 34.7)
  const long tiles64 = long((a.M + 63) / 64) * ((a.N + 63) / 64);
  if (tiles64 >= 256) {
    if (vec) run(k_gemm_f32<TA, TB, EPI, true>, 64, 256);
    else run(k_gemm_f32<TA, TB, EPI, false>, 64, 256);
  } else {
    if (vec) run(k_gemm_f32_ks<TA, TB, EPI, true>, T, 64 * (MW + LW));
    else run(k_gemm_f32_ks<TA, TB, EPI, false>, T, 64 * (MW + LW));
  }
}

inline bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

void gemm_f32(hipStream_t s, int M, int N, int K, const float *A, int lda, bool ta, const float *B,
              int ldb, bool tb, float *C, int ldc, int epi, const float *D, int ldd,
              const float *bias, float *Z, int ldz) {
  if (M <= 0 || N <= 0) return;
  GemmArgs a{M, N, K, A, lda, B, ldb, C, ldc, D, ldd, bias, Z, ldz};
  // 16-byte operand loads when every contiguous extent and leading dimension
  // is a multiple of 4 floats and both bases are 16-byte aligned
  const bool vec = lda % 4 == 0 && ldb % 4 == 0 && al16(A) && al16(B) &&
                   (ta ? M : K) % 4 == 0 && (tb ? K : N) % 4 == 0;
  if (epi == GEMM_EPI_MLPFWD || epi == GEMM_EPI_BIAS) {
    if (ta || tb) fail(CKPT_E_UNSUPPORTED, "gemm_f32: the bias epilogues take untransposed operands");
    if (epi == GEMM_EPI_MLPFWD) launch<false, false, GEMM_EPI_MLPFWD>(a, vec, s);
    else launch<false, false, GEMM_EPI_BIAS>(a, vec, s);
    return;
  }
#define CKPT_GEMM_CASE(TA_, TB_)                                           \
  if (ta == TA_ && tb == TB_) {                                            \
    if (epi == GEMM_EPI_STORE) launch<TA_, TB_, GEMM_EPI_STORE>(a, vec, s); \
    else launch<TA_, TB_, GEMM_EPI_ADD>(a, vec, s);                         \
    return;                                                                \
  }
  CKPT_GEMM_CASE(false, false)
  CKPT_GEMM_CASE(false, true)
  CKPT_GEMM_CASE(true, false)
  CKPT_GEMM_CASE(true, true)
#undef CKPT_GEMM_CASE
}

}  // namespace ckpt
