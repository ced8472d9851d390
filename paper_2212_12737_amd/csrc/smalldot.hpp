// Dot products of a few FP64 rows on the matrix cores without LDS staging: the
// operands of a 16 x 16 tile go from global memory (L2) to registers, four to
// eight 8-wide steps of K in flight.  For tiles so few that latency, not the matrix
// rate, decides; rows may have any length and 8-byte alignment.
#pragma once

#include "gemm.hpp"

namespace ffk {

typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// elements k, k + 1 of a row of length D, zero past its end
__device__ inline d2u row_pair(const double* p, int k, int D) {
  if (k + 1 < D) return *reinterpret_cast<const d2u*>(p + k);
  d2u v;
  v[0] = k < D ? p[k] : 0.0;
  v[1] = 0.0;
  return v;
}

// g[i] += A_i X^T and, with BOTH, p[i] += A_i U^T over the 8-wide steps [s0,
// s1) of K = D.  a[i], x, u: the rows (l % 16) of this lane; lane l takes k = 8
// s + 2 (l / 16) + j in MFMA j.  Results: column l % 16, rows 4 v + l / 16.
template <int TB, bool BOTH>
__device__ inline void rows_dot(const double* const (&a)[TB], const double* x, const double* u, int D, int s0, int s1,
                                d4 (&g)[TB], d4 (&p)[TB]) {
  constexpr int UN = 4;
  const int kq = 2 * ((threadIdx.x & 63) >> 4);
  struct Steps { d2u a[UN][TB], x[UN], u[UN]; };
  auto load = [&](int s, Steps& f) {
#pragma unroll
    for (int e = 0; e < UN; ++e)
      if (s + e < s1) {
        const int k = 8 * (s + e) + kq;
#pragma unroll
        for (int i = 0; i < TB; ++i) f.a[e][i] = row_pair(a[i], k, D);
        f.x[e] = row_pair(x, k, D);
        if (BOTH) f.u[e] = row_pair(u, k, D);
      }
  };
  auto mul = [&](int s, const Steps& f) {
#pragma unroll
    for (int e = 0; e < UN; ++e)
      if (s + e < s1) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int i = 0; i < TB; ++i) {
            g[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.a[e][i][j], f.x[e][j], g[i], 0, 0, 0);
            if (BOTH) p[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.a[e][i][j], f.u[e][j], p[i], 0, 0, 0);
          }
      }
  };
  Steps f0, f1;   // the next four steps load while these multiply
  if (s0 < s1) load(s0, f0);
  for (int s = s0; s < s1; s += 2 * UN) {
    if (s + UN < s1) load(s + UN, f1);
    mul(s, f0);
    if (s + UN >= s1) break;
    if (s + 2 * UN < s1) load(s + 2 * UN, f0);
    mul(s + UN, f1);
  }
}

// dA = a(r) - a(0) and B = b(r) of the Matern-5/2 Hessian at squared distance
// r2 (rounding may have made it negative); inv_len = sqrt(5) / sigma.
__device__ inline void matern_coeffs(double r2, double inv_len, double a0, double bcoef, double& dA, double& B) {
  const double z = sqrt(r2 < 0.0 ? 0.0 : r2) * inv_len;
  const double em = expm1(-z);
  dA = a0 * ((1.0 + z) * em + z);
  B = -bcoef * (em + 1.0);
}

}  // namespace ffk
