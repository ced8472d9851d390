// Cholesky factorization and triangular inverse of one 64 x 64 FP64 block in
// LDS, by a block of four waves: panels of 16 columns in the registers of one
// wave, all products between 16 x 16 blocks on FP64 MFMA.  What bounds it is
// the serial chain of 64 pivots, at some ten cycles an instruction of the wave
// that holds them: each of its four rows of lanes keeps a copy of the diagonal
// block (a lane holds a row of it) and a block below it, so that other rows'
// values come by one DPP broadcast for two updates, and the rows below need no
// inverse, barrier or product of their own.  Factor and inverse, with the block
// read from and written to memory: 113 us column by column in LDS with three
// barriers a column, 30 us with diagonal blocks of 16 and readlane, now 18.
#pragma once

#include "gemm.hpp"

namespace ffk {

struct Chol64 {
  double T[64][65];         // in: the lower triangle; out: the factor
  double X[64][65];         // its inverse: the blocks on and below the diagonal
  double W[4][16][17];      // scratch, one per wave
  double d[64], ri[64];     // pivots; inverses of their roots (1 where the pivot is bad)
  unsigned char bad[64];    // pivots that were dropped or not positive
  __device__ double inverse(int r, int c) const { return c >> 4 > r >> 4 ? 0.0 : X[r][c]; }
};

// The value of lane N of each row of 16 lanes, in the whole row.
template <int N> __device__ inline double row_value(double x) {
  return __builtin_amdgcn_mov_dpp(x, 0x150 + N, 0xf, 0xf, true);
}

// s = sqrt(d), ri = 1 / s for 1e-280 < d < 1e280: the hardware's reciprocal
// square root (26 bits) and a Newton step, both results corrected by their
// residuals (the library's square root and divide are a chain twice as long, and
// 64 of them are serial).
__device__ inline void sqrt_and_inverse(double d, double& s, double& ri) {
  double y = __builtin_amdgcn_rsq(d);
  y = fma(0.5 * y, fma(-d * y, y, 1.0), y);
  s = d * y;
  s = fma(fma(-s, s, d), 0.5 * y, s);
  ri = fma(fma(-s, y, 1.0), y, y);
}

// Whether a pivot counts: above thr (DROP), or positive and finite.
template <bool DROP> __device__ inline bool pivot_ok(double d, double thr) {
  return DROP ? d > thr : __builtin_amdgcn_class(d, 0x180);   // positive normal or subnormal
}

// Cholesky of a 16 x 16 block, row r of it in a[0..15] of the lanes l % 16 = r
// of every row of lanes, and the rows p[0..15] below it; the pivots d, their
// roots sq and the roots' inverses ri (of a pivot that does not count: as of one,
// or with DROP the root 0).  a is the factor below the diagonal only.  One
// straight line of code, so that the updates fill the pivots' latency; SAFE
// takes the library's square root and divide.
template <bool DROP, bool SAFE>
__device__ inline void factor16(double (&a)[16], double (&p)[16], double (&d)[16], double (&sq)[16], double (&ri)[16],
                                double thr) {
  static_for<0, 16>([&](auto C) {
    constexpr int c = decltype(C)::value;
    d[c] = row_value<c>(a[c]);
    const bool ok = pivot_ok<DROP>(d[c], thr);
    const double dc = ok ? d[c] : 1.0;
    if (SAFE) {
      sq[c] = sqrt(dc);
      ri[c] = 1.0 / sq[c];
    } else {
      sqrt_and_inverse(dc, sq[c], ri[c]);
    }
    const double f = DROP && !ok ? 0.0 : ri[c];
    if (DROP && !ok) sq[c] = 0.0;
    a[c] *= f;
    p[c] = DROP && !ok ? 0.0 : p[c] * f;
    static_for<c + 1, 16>([&](auto Q) {
      constexpr int q = decltype(Q)::value;
      const double m = row_value<q>(a[c]);
      a[q] = fma(-a[c], m, a[q]);
      p[q] = fma(-p[c], m, p[q]);
    });
  });
}

// acc += A B (B[k][col]) or A B^T (NT: B[col][k]) for 16 x 16 blocks; lane l
// holds column l % 16 and rows 4 v + l / 16 of acc.
template <bool NT, int LA, int LB>
__device__ inline d4 mm16(const double (*A)[LA], int a0, const double (*B)[LB], int b0, d4 acc) {
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = 4 * s + q;
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[r][a0 + k], NT ? B[r][b0 + k] : B[k][b0 + r], acc, 0, 0, 0);
  }
  return acc;
}

// The inverse of the lower-triangular 16 x 16 block whose row r is a[0..15] in
// the lanes l % 16 = r (below the diagonal), with ri the inverses of its
// diagonal; lane c writes column c.
__device__ inline void inv16(const double (&a)[16], const double (&ri)[16], double (*I)[65], int c0) {
  const int lane = threadIdx.x & 63, c = lane & 15;
  double x[16];
  static_for<0, 16>([&](auto R) {
    constexpr int r = decltype(R)::value;
    double s0 = r == c ? 1.0 : 0.0, s1 = 0.0;
    static_for<0, r>([&](auto Q) {
      constexpr int q = decltype(Q)::value;
      const double l = row_value<r>(a[q]);
      if (q & 1) s1 = fma(-l, x[q], s1);
      else s0 = fma(-l, x[q], s0);
    });
    x[r] = (s0 + s1) * ri[r];
  });
  if (lane < 16) {
#pragma unroll
    for (int r = 0; r < 16; ++r) I[r][c0 + c] = x[r];
  }
}

// Diagonal block b of the inverse of the factor s.T, by one wave.
template <bool ROOTS> __device__ inline void tri64_diag(Chol64& s, int b) {
  const int r = threadIdx.x & 15;
  double a[16], ri[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    a[c] = s.T[16 * b + r][16 * b + c];
    ri[c] = ROOTS ? s.ri[16 * b + c] : 1.0 / s.T[16 * b + c][16 * b + c];
  }
  inv16(a, ri, s.X + 16 * b, 16 * b);
}

// W = sum_k T_ik X_kw (w <= k < i), and X_iw = -X_ii W; by one wave.
__device__ inline void tri64_sum(Chol64& s, int i, int w) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q4 = lane >> 4;
  d4 t{0, 0, 0, 0};
  for (int k = w; k < i; ++k) t = mm16<false>(s.T + 16 * i, 16 * k, s.X + 16 * k, 16 * w, t);
#pragma unroll
  for (int v = 0; v < 4; ++v) s.W[wave][4 * v + q4][r] = t[v];
  __builtin_amdgcn_wave_barrier();
}
__device__ inline void tri64_block(Chol64& s, int i, int w) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q4 = lane >> 4;
  const d4 x = mm16<false>(s.X + 16 * i, 16 * i, s.W[wave], 0, d4{0, 0, 0, 0});
#pragma unroll
  for (int v = 0; v < 4; ++v) s.X[16 * i + 4 * v + q4][16 * w + r] = -x[v];
  __builtin_amdgcn_wave_barrier();
}

// The inverse of the factor s.T: wave w forms block column w.
__device__ inline void tri64_inverse(Chol64& s) {
  const int w = threadIdx.x >> 6;
  tri64_diag<false>(s, w);
  __syncthreads();
  for (int i = w + 1; i < 4; ++i) {
    tri64_sum(s, i, w);
    tri64_block(s, i, w);
  }
}

// Factor s.T in place (the part above the diagonal is not read) and form its
// inverse in s.X.  DROP: a pivot that is not above thr becomes a zero column
// (its diagonal counts as one in the inverse).  Otherwise a pivot that is not
// positive and finite is flagged and counts as one.  Rows of the inverse are
// formed by the other waves beside the next panel.  The caller synchronises.
template <bool DROP>
__device__ inline void chol64_inverse(Chol64& s, double thr) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q4 = lane >> 4;
  for (int b = 0; b < 4; ++b) {
    const int c0 = 16 * b;
    if (wave == 0) {
      const bool below = q4 > 0 && b + q4 < 4;
      const int row = below ? c0 + lane : c0 + r;
      double a[16], p[16], d[16], sq[16], ri[16];
      auto load = [&]() {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          a[c] = c <= r ? s.T[c0 + r][c0 + c] : 0.0;
          p[c] = s.T[row][c0 + c];
        }
      };
      load();
      factor16<DROP, false>(a, p, d, sq, ri, thr);
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < 16; ++c) s.d[c0 + c] = d[c];
      }
      __builtin_amdgcn_wave_barrier();
      const double dr = s.d[c0 + r];
      const bool ok = pivot_ok<DROP>(dr, thr);
      if (__any(ok && !(dr > 1e-280 && dr < 1e280))) {
        load();
        factor16<DROP, true>(a, p, d, sq, ri, thr);
        if (lane == 0) {
#pragma unroll
          for (int c = 0; c < 16; ++c) s.d[c0 + c] = d[c];
        }
        __builtin_amdgcn_wave_barrier();
      }
      if (lane < 16) s.bad[c0 + r] = !pivot_ok<DROP>(s.d[c0 + r], thr);
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        if (below) s.T[row][c0 + c] = p[c];
        else if (q4 == 0 && c < r) s.T[row][c0 + c] = a[c];
      }
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          s.T[c0 + c][c0 + c] = sq[c];
          s.ri[c0 + c] = ri[c];
        }
      }
    }
    __syncthreads();
    if (b == 3) break;
    int n = 0;
    for (int i = b + 1; i < 4; ++i)
      for (int j = b + 1; j <= i; ++j)
        if ((n++ & 3) == wave) {   // T_ij -= P_i P_j^T
          const d4 p = mm16<true>(s.T + 16 * i, c0, s.T + 16 * j, c0, d4{0, 0, 0, 0});
#pragma unroll
          for (int v = 0; v < 4; ++v) s.T[16 * i + 4 * v + q4][16 * j + r] -= p[v];
        }
    __syncthreads();
    if (wave == b + 1) {   // beside the next panel: row b of the inverse
      tri64_diag<true>(s, b);
      __builtin_amdgcn_wave_barrier();
      for (int w = 0; w < b; ++w) {
        tri64_sum(s, b, w);
        tri64_block(s, b, w);
      }
    }
  }
  if (wave == 0) tri64_diag<true>(s, 3);
  else tri64_sum(s, 3, wave - 1);
  __syncthreads();
  if (wave > 0) tri64_block(s, 3, wave - 1);
}

}  // namespace ffk
