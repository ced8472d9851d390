// Cholesky factorization and triangular inverse of one 64 x 64 FP64 block in
// LDS, by a block of four waves: 16 x 16 diagonal blocks in the registers of
// one wave (a lane holds a row, other rows' values come by readlane), all
// products between 16 x 16 blocks on FP64 MFMA.  What bounds it is the serial
// chain of 64 pivots; a column-by-column factorization in LDS with three
// barriers a column spent its time in the barriers: 80 us for the factor and 33
// more for its inverse, now 30 us for both.
#pragma once

#include "gemm.hpp"

namespace ffk {

struct Chol64 {
  double T[64][65];         // in: the lower triangle; out: the factor
  double X[64][65];         // its inverse (tri64_inverse)
  double I[4][16][17];      // inverses of the diagonal 16 x 16 blocks
  double W[4][16][17];      // scratch, one per wave
  unsigned char bad[64];    // pivots that were dropped or not positive
};

// s = sqrt(d), ri = 1 / s for 1e-280 < d < 1e280: the hardware's reciprocal
// square root and two Newton steps, both results corrected by their residuals
// (the library's square root and divide are a chain twice as long, and 64 of
// them are serial).
__device__ inline void sqrt_and_inverse(double d, double& s, double& ri) {
  double y = __builtin_amdgcn_rsq(d);
#pragma unroll
  for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-d * y, y, 1.0), y);
  s = d * y;
  s = fma(fma(-s, s, d), 0.5 * y, s);
  ri = fma(fma(-s, y, 1.0), y, y);
}

// Cholesky of a 16 x 16 block, row r of it in a[0..15] of the lanes l % 16 = r;
// ri: the inverses of the pivots' roots; the flagged pivots as bits.  One
// straight line of code, so that the updates fill the pivots' latency; SAFE
// takes the library's square root and divide.  Returns whether a pivot was
// outside the range of sqrt_and_inverse.
template <bool DROP, bool SAFE>
__device__ inline bool factor16(double (&a)[16], double (&ri)[16], double thr, unsigned& flagged) {
  const int r = threadIdx.x & 15;
  bool range = false;
  flagged = 0;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const double d = lane_value(a[c], c);
    const bool ok = DROP ? d > thr : (d > 0.0 && d < __builtin_huge_val());
    double sq, inv;
    if (SAFE) {
      sq = sqrt(d);
      inv = 1.0 / sq;
    } else {
      sqrt_and_inverse(d, sq, inv);
      range |= ok && !(d > 1e-280 && d < 1e280);
    }
    const double none = DROP ? 0.0 : 1.0;
    flagged |= ok ? 0u : 1u << c;
    ri[c] = ok ? inv : 1.0;
    const double f = ok ? inv : none;
    a[c] = r == c ? (ok ? sq : none) : a[c] * f;
#pragma unroll
    for (int q = c + 1; q < 16; ++q) a[q] = fma(-a[c], lane_value(a[c], q), a[q]);
  }
  return range;
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
// lane r, with ri the inverses of its diagonal; lane c writes column c.
__device__ inline void inv16(const double (&a)[16], const double (&ri)[16], double (*I)[17]) {
  const int lane = threadIdx.x & 63, c = lane & 15;
  double x[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    double s0 = r == c ? 1.0 : 0.0, s1 = 0.0;
#pragma unroll
    for (int q = 0; q < r; ++q) {
      const double l = lane_value(a[q], r);
      if (q & 1) s1 = fma(-l, x[q], s1);
      else s0 = fma(-l, x[q], s0);
    }
    x[r] = (s0 + s1) * ri[r];
  }
  if (lane < 16) {
#pragma unroll
    for (int r = 0; r < 16; ++r) I[r][c] = x[r];
  }
}

// Factor s.T in place (the part above the diagonal is not read) and leave the
// inverses of its diagonal blocks in s.I.  DROP: a pivot that is not above thr
// becomes a zero column (its diagonal counts as one in the inverse).
// Otherwise a pivot that is not positive and finite is flagged and counts as one.
template <bool DROP>
__device__ inline void chol64(Chol64& s, double thr) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q4 = lane >> 4;
  for (int b = 0; b < 4; ++b) {
    const int c0 = 16 * b;
    if (wave == 0) {
      double a[16], ri[16];
      auto load = [&]() {
#pragma unroll
        for (int c = 0; c < 16; ++c) a[c] = c <= r ? s.T[c0 + r][c0 + c] : 0.0;
      };
      unsigned flagged;
      load();
      if (factor16<DROP, false>(a, ri, thr, flagged)) {
        load();
        factor16<DROP, true>(a, ri, thr, flagged);
      }
      if (lane < 16) s.bad[c0 + lane] = (flagged >> lane) & 1;
      if (lane < 16) {
#pragma unroll
        for (int c = 0; c < 16; ++c)
          if (c <= r) s.T[c0 + r][c0 + c] = a[c];
      }
      inv16(a, ri, s.I[b]);
    }
    __syncthreads();
    const int rb = b + 1 + wave;
    if (rb < 4) {   // rows below: P = T L^-T
      const d4 p = mm16<true>(s.T + 16 * rb, c0, s.I[b], 0, d4{0, 0, 0, 0});
      const bool drop = DROP && s.bad[c0 + r];
#pragma unroll
      for (int v = 0; v < 4; ++v) s.T[16 * rb + 4 * v + q4][c0 + r] = drop ? 0.0 : p[v];
    }
    __syncthreads();
    int n = 0;
    for (int i = b + 1; i < 4; ++i)
      for (int j = b + 1; j <= i; ++j)
        if ((n++ & 3) == wave) {   // T_ij -= P_i P_j^T
          const d4 p = mm16<true>(s.T + 16 * i, c0, s.T + 16 * j, c0, d4{0, 0, 0, 0});
#pragma unroll
          for (int v = 0; v < 4; ++v) s.T[16 * i + 4 * v + q4][16 * j + r] -= p[v];
        }
    __syncthreads();
  }
}

// The inverses of the four diagonal blocks of the factor s.T, one per wave.
__device__ inline void tri64_diag(Chol64& s) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15;
  double a[16], ri[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) a[c] = c <= r ? s.T[16 * wave + r][16 * wave + c] : 0.0;
#pragma unroll
  for (int c = 0; c < 16; ++c) ri[c] = 1.0 / lane_value(a[c], c);
  inv16(a, ri, s.I[wave]);
}

// s.X = the inverse of the factor s.T from s.I, zero above the diagonal: wave
// w forms block column w, X_iw = -I_i sum_k T_ik X_kw.
__device__ inline void tri64_inverse(Chol64& s) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, q4 = lane >> 4;
  for (int i = 0; i < 4; ++i) {
    d4 x{0, 0, 0, 0};
    if (i == w) {
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = s.I[w][4 * v + q4][r];
    } else if (i > w) {
      d4 t{0, 0, 0, 0};
      for (int k = w; k < i; ++k) t = mm16<false>(s.T + 16 * i, 16 * k, s.X + 16 * k, 16 * w, t);
#pragma unroll
      for (int v = 0; v < 4; ++v) s.W[w][4 * v + q4][r] = t[v];
      __builtin_amdgcn_wave_barrier();
      x = mm16<false>(s.I[i], 0, s.W[w], 0, d4{0, 0, 0, 0});
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = -x[v];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) s.X[16 * i + 4 * v + q4][16 * w + r] = x[v];
    __builtin_amdgcn_wave_barrier();
  }
}

}  // namespace ffk
