// Column-major FP64 GEMM on the matrix cores:  C = alpha A B^T + beta C  with
// C and A column-major (unit stride along m) and B either n-contiguous (a
// column-major N x K matrix) or k-contiguous (a row-major N x K matrix, i.e.
// the K x N column-major right factor of an ordinary product).  These are the
// products of the incomplete and dense Cholesky factorizations and of the
// triangular inverse.
//
// The operands go from global memory straight to LDS, 16 bytes a lane, in the
// order in which the MFMAs read them, so that every fragment is one
// conflict-free ds_read_b128:
//  - m- or n-contiguous: 16 bytes are two neighbouring rows at one k.  A wave
//    load takes a group of 32 rows at four k (2 (l / 16) + j, j the load of
//    the pair), and one 16-byte fragment feeds two 16-row blocks, the even
//    and the odd rows of the group;
//  - k-contiguous: 16 bytes are two neighbouring k of one row; a wave load
//    takes 16 rows at eight k, and one fragment feeds both MFMA slices.
// Both use k = 2 (l / 16) + j in slice j.  The n side is the first MFMA
// operand and the m side the second, so lane l holds the columns m = 2 (l %
// 16) + {0, 1} of a group: C moves as 16-byte pairs, 256 contiguous bytes per
// 16 lanes.
// Rows past M and N read the last valid pair (their results are not stored),
// k past K reads zeros.  Pointers must be 16-byte aligned, leading dimensions
// even; a k-contiguous B of odd K needs finite values at k = K (the zeros of
// A meet them).
// Bound by the FP64 matrix cores (72 TFLOP/s reached by a large library
// product).  Fragments are double-buffered in registers: read right before
// their MFMAs, the waves of both workgroups of a CU met in the same phase and
// the matrix cores idled through the reads.  With 128 x 128 tiles, read first
// and now: M = N = 8192, K = 1024 54 -> 67 TFLOP/s; n = 12544, K = 256 51 -> 56;
// M = 126016, N = 256, K = 1024 59 -> 64; 64 x 64 tiles at M = 2048, N = 1024, K
// = 256 33 -> 41.
#pragma once

#include "gemm.hpp"

namespace ffk {

// BM x BN block tile by WM x WN waves; KS chunks of 8 k per stage, two stages.
template <int BM_, int BN_, int WM_, int WN_, int KS_>
struct Tile64 {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KS = KS_;
  static constexpr int NT = 64 * WM * WN;
};

struct Gemm64Args {
  const double *A, *B;
  int64_t lda, ldb;
  int M, N, K;
  int lower_only;          // tiles with all columns above the diagonal do nothing
  // Batch index z = blockIdx.z: A, B (and C, in the epilogue) move by these
  // strides; with row_step > 0, M (and K when ktrim) shrink to what is left
  // of row_end - z row_step rows, and N to ncol_step z when that is > 0.
  int64_t sA, sB;
  int64_t row_step, row_end;
  int ktrim, ncol_step;
};

__device__ __attribute__((aligned(16))) static const double g_zero64[2] = {0.0, 0.0};

// C[m + n ldc] = alpha acc + beta C (beta = 0: C is not read).  vec: C and ldc
// allow 16-byte pairs.
struct EpiCol64 {
  double* C;
  int64_t ldc, sC;
  double alpha, beta;
  int vec;
};

template <class TL, bool BKC>
__global__ __launch_bounds__(TL::NT) void k_gemm64(Gemm64Args g, EpiCol64 e) {
  constexpr int BM = TL::BM, BN = TL::BN, WM = TL::WM, WN = TL::WN, KS = TL::KS, NW = WM * WN;
  constexpr int BK = 8 * KS;
  constexpr int A_CHUNK = BM * 64, B_CHUNK = BN * 64;      // bytes of 8 k of a tile
  constexpr int STAGE = KS * (A_CHUNK + B_CHUNK);
  constexpr int LA = BM / 16 * KS, LB = BN / 16 * KS;      // 1 KB wave loads per stage
  static_assert(LA % NW == 0 && LB % NW == 0, "loads must split evenly over the waves");
  constexpr int QA = LA / NW, QB = LB / NW, LPT = QA + QB;
  static_assert(LPT < 64, "vmcnt holds at most 63 loads in flight");
  static_assert(KS % 2 == 0, "fragments alternate between two sets");
  constexpr int MB = BM / WM / 16, NB = BN / WN / 16;      // 16-row blocks per wave
  static_assert(MB % 2 == 0 && (BKC || NB % 2 == 0), "pairs of blocks");
  __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const int z = blockIdx.z;
  int M = g.M, N = g.N, K = g.K;
  if (g.row_step > 0) {
    M = (int)min((int64_t)M, g.row_end - z * g.row_step);
    if (g.ktrim) K = min(K, M);
  }
  if (g.ncol_step > 0) N = z * g.ncol_step;
  // the n tiles of one m tile run on one XCD (workgroup w on XCD w % 8), so
  // that its rows of A are read from HBM once
  const int ntn = gridDim.x;
  const int lin = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  const int per = 8 * ntn, grp = lin / per, in = lin % per;
  const int gsz = min((int)gridDim.y - grp * 8, 8);
  const int m0 = (grp * 8 + in % gsz) * BM, n0 = (in / gsz) * BN;
  if (m0 >= M || n0 >= N) return;
  if (g.lower_only && n0 > m0 + BM - 1) return;
  const double* A = g.A + z * g.sA;
  const double* B = g.B + z * g.sB;

  // this lane's source of every load, and its k within the stage
  const double* pa[QA];
  const double* pb[QB];
  int ka[QA], kb[QB];
#pragma unroll
  for (int q = 0; q < QA; ++q) {
    const int idx = wave * QA + q, kc = idx / (BM / 16), rem = idx % (BM / 16);
    const int m = min(m0 + 32 * (rem >> 1) + 2 * (lane & 15), (M - 1) & ~1);
    ka[q] = 8 * kc + 2 * (lane >> 4) + (rem & 1);
    pa[q] = A + m + ka[q] * g.lda;
  }
#pragma unroll
  for (int q = 0; q < QB; ++q) {
    const int idx = wave * QB + q, kc = idx / (BN / 16), rem = idx % (BN / 16);
    if (BKC) {
      const int n = min(n0 + 16 * rem + (lane & 15), N - 1);
      kb[q] = 8 * kc + 2 * (lane >> 4);
      pb[q] = B + n * g.ldb + kb[q];
    } else {
      const int n = min(n0 + 32 * (rem >> 1) + 2 * (lane & 15), (N - 1) & ~1);
      kb[q] = 8 * kc + 2 * (lane >> 4) + (rem & 1);
      pb[q] = B + n + kb[q] * g.ldb;
    }
  }
  const int64_t stepA = (int64_t)BK * g.lda, stepB = BKC ? BK : (int64_t)BK * g.ldb;
  const int T = (K + BK - 1) / BK;
  auto issue = [&](int t) {
    char* st = smem + (t & 1) * STAGE;
    const int left = K - t * BK;   // k < left is valid in this stage
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      dma16(ka[q] < left ? pa[q] : g_zero64, st + (wave * QA + q) * 1024);
      pa[q] += stepA;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      dma16(kb[q] < left ? pb[q] : g_zero64, st + KS * A_CHUNK + (wave * QB + q) * 1024);
      pb[q] += stepB;
    }
  };

  d4 acc[NB][MB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[i][j] = d4{0, 0, 0, 0};

  struct Frag { u4 m[2][MB / 2], n[BKC ? 1 : 2][BKC ? NB : NB / 2]; };
  auto read = [&](int t, int kc, Frag& f) {
    const char* st = smem + (t & 1) * STAGE;
    const char* sa = st + kc * A_CHUNK + wm * (MB / 2) * 2048 + lane * 16;
    const char* sb = st + KS * A_CHUNK + kc * B_CHUNK + wn * NB * 1024 + lane * 16;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int p = 0; p < MB / 2; ++p) f.m[s][p] = *reinterpret_cast<const u4*>(sa + p * 2048 + s * 1024);
    if constexpr (BKC) {
#pragma unroll
      for (int i = 0; i < NB; ++i) f.n[0][i] = *reinterpret_cast<const u4*>(sb + i * 1024);
    } else {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int p = 0; p < NB / 2; ++p) f.n[s][p] = *reinterpret_cast<const u4*>(sb + p * 2048 + s * 1024);
    }
  };
  auto mul = [&](const Frag& f) {
    // the reads of the next fragments stay before these MFMAs
    __builtin_amdgcn_sched_barrier(0);
    auto half = [](const u4& v, int h) { return __hiloint2double((int)v[2 * h + 1], (int)v[2 * h]); };
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) {
          const double a = BKC ? half(f.n[0][i], s) : half(f.n[BKC ? 0 : s][BKC ? 0 : i / 2], i & 1);
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, half(f.m[s][j / 2], j & 1), acc[i][j], 0, 0, 0);
        }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Software pipeline: a chunk's fragments are read while the MFMAs of the one
  // before it run.  At a stage's last chunk the wave has its fragments in
  // registers; past the barrier every wave has, so the next stage's data is
  // complete and this stage's buffer free for the one after it.
  if (T > 0) issue(0);
  if (T > 1) issue(1);
  if (T > 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LPT) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  Frag f[2];
  if (T > 0) read(0, 0, f[0]);
  for (int t = 0; t < T; ++t) {
#pragma unroll
    for (int kc = 0; kc < KS; ++kc) {
      if (kc + 1 < KS) read(t, kc + 1, f[(kc + 1) & 1]);
      else if (t + 1 < T) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (t + 2 < T) issue(t + 2);
        read(t + 1, 0, f[0]);
      }
      mul(f[kc & 1]);
    }
  }

  double* C = e.C + z * e.sC;
  const int mb = m0 + wm * MB * 16 + 2 * (lane & 15);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    double2 c[4][MB / 2];
    if (e.beta != 0.0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 4 * v + (lane >> 4);
        const int n = n0 + wn * NB * 16 + (BKC ? 16 * i + r : 32 * (i / 2) + 2 * r + (i & 1));
#pragma unroll
        for (int p = 0; p < MB / 2; ++p) {
          const int m = mb + 32 * p;
          const double* src = C + m + n * e.ldc;
          c[v][p] = make_double2(0.0, 0.0);
          if (n < N && m < M) {
            if (e.vec && m + 1 < M) c[v][p] = *reinterpret_cast<const double2*>(src);
            else {
              c[v][p].x = src[0];
              if (m + 1 < M) c[v][p].y = src[1];
            }
          }
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 4 * v + (lane >> 4);
      const int n = n0 + wn * NB * 16 + (BKC ? 16 * i + r : 32 * (i / 2) + 2 * r + (i & 1));
#pragma unroll
      for (int p = 0; p < MB / 2; ++p) {
        const int m = mb + 32 * p;
        double2 x = make_double2(e.alpha * acc[i][2 * p][v], e.alpha * acc[i][2 * p + 1][v]);
        if (e.beta != 0.0) {
          x.x += e.beta * c[v][p].x;
          x.y += e.beta * c[v][p].y;
        }
        double* dst = C + m + n * e.ldc;
        if (n < N && m < M) {
          if (e.vec && m + 1 < M) *reinterpret_cast<double2*>(dst) = x;
          else {
            dst[0] = x.x;
            if (m + 1 < M) dst[1] = x.y;
          }
        }
      }
    }
  }
}

}  // namespace ffk
