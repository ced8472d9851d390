// Descriptor build and iteration-invariant kernel coefficients.
//
// x_pq = 1/|R_p - R_q| for p > q (row-major lower-triangle order), the column
// mean over geometries, X_c = X - mean (differences x_i - x_j, hence the
// kernel, do not change; centring keeps the Gram-matrix route to distances
// well conditioned), |x_c,i|^2, then from the FP64 Gram matrix X_c X_c^T:
//   r_ij = sqrt(max(|x_i|^2 + |x_j|^2 - 2 x_i.x_j, 0)),  z = sqrt(5) r / sigma,
//   dA_ij = a(r) - a(0) = a0 ((1 + z) expm1(-z) + z),   a0 = 5 / (3 sigma^2),
//   B_ij  = b(r) = -25/(3 sigma^4) e^-z,
// the Matern-5/2 Hessian coefficients H = a I + b d d^T of the force kernel.
// Reduced-precision copies are derived from the FP64 arrays on first use.
#include <algorithm>

#include "smalldot.hpp"

namespace ffk {

// Pair d of the strict lower triangle, whose row p starts at p (p - 1) / 2.
__device__ inline void pair_of(int64_t d, int& p, int& q) {
  p = (int)((1.0 + sqrt(1.0 + 8.0 * (double)d)) * 0.5);
  while ((int64_t)p * (p - 1) / 2 > d) --p;
  while ((int64_t)p * (p + 1) / 2 <= d) ++p;
  q = (int)(d - (int64_t)p * (p - 1) / 2);
}

// x of the pair (p, q) of one geometry; flags coincident atoms and what is not finite.
__device__ inline double descriptor_entry(const double* Rg, int p, int q, int* bad) {
  const double dx = Rg[3 * p] - Rg[3 * q], dy = Rg[3 * p + 1] - Rg[3 * q + 1],
               dz = Rg[3 * p + 2] - Rg[3 * q + 2];
  const double r2 = dx * dx + dy * dy + dz * dz;
  const double x = 1.0 / sqrt(r2);
  if (!(r2 > 0.0) || !isfinite(x)) *bad = 1;
  return x;
}

// Descriptor, pairs and the copies the system keeps: thread e takes element e of X
// and of R.
__global__ void k_descriptor(const double* __restrict__ R, int64_t N, int M, int64_t D, double* __restrict__ X,
                             int* __restrict__ pairs, double* __restrict__ Rcopy, int* __restrict__ bad) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < N * M * 3) Rcopy[e] = R[e];
  if (e >= N * D) return;
  const int64_t g = e / D, d = e % D;
  int p, q;
  pair_of(d, p, q);
  if (g == 0) pairs[d] = p << 16 | q;
  X[e] = descriptor_entry(R + g * 3 * M, p, q, bad);
}

// The pair table: (R_p - R_q) / r^3 and 1 / r of every pair of every geometry.
__global__ void k_pair_table(const double* __restrict__ R, const int* __restrict__ pairs, int64_t N, int M, int64_t D,
                             double2* __restrict__ PT) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N * D) return;
  const int64_t g = e / D;
  const int pq = pairs[e % D], p = pq >> 16, q = pq & 0xFFFF;
  const double* Rg = R + g * 3 * M;
  const double dx = Rg[3 * p] - Rg[3 * q], dy = Rg[3 * p + 1] - Rg[3 * q + 1],
               dz = Rg[3 * p + 2] - Rg[3 * q + 2];
  const double x = 1.0 / sqrt(dx * dx + dy * dy + dz * dz);
  const double x3 = x * x * x;
  PT[2 * e] = make_double2(dx * x3, dy * x3);
  PT[2 * e + 1] = make_double2(dz * x3, x);
}

// Twice the size of the descriptor and its centred copy (1.1 GB at M = 60, N =
// 20000), which products, predictions and the stacked copies of a symmetrized system
// do not need: so it is formed here, and where it would be a large part of what
// is left, the columns do without (kernel_columns_src).
bool pair_table(const ffk_system* s, hipStream_t st) {
  std::lock_guard<std::mutex> lock(s->form_lock);
  if (s->PT) return true;
  const size_t bytes = (size_t)(4 * s->N * s->D) * sizeof(double);
  size_t free_bytes = 0, total = 0;
  HIPCHK(hipMemGetInfo(&free_bytes, &total));
  if (bytes > free_bytes / 16) return false;
  DBuf t(bytes);
  k_pair_table<<<cdiv(s->N * s->D, 256), 256, 0, st>>>(s->R.as<double>(), s->pairs.as<int>(), s->N, s->M, s->D,
                                                       t.as<double2>());
  LAUNCHCHK();
  HIPCHK(hipStreamSynchronize(st));   // the next call may come on another stream
  s->PT = std::move(t);
  return true;
}

// The same of at most kFewRows geometries with their mean, centred rows and
// norms, in one block: a thread takes pairs of all geometries.  (Apart,
// with a flag cleared and copied by the GPU, a prediction of one geometry waited
// for their launches: 95 us, 76 with this one, the flag in pinned memory and one
// launch fewer in kernel_predict, at M = 21, N = 2000.)
constexpr int kFewRows = 8;
__global__ __launch_bounds__(1024) void k_descriptor_few(const double* __restrict__ R, int N, int M, int64_t D,
                                                         double* __restrict__ X, int* __restrict__ pairs,
                                                         double* __restrict__ Rcopy, double* __restrict__ mean,
                                                         double* __restrict__ Xc, double* __restrict__ sqn,
                                                         int* __restrict__ bad) {
  __shared__ double red[16][kFewRows];
  for (int e = threadIdx.x; e < N * M * 3; e += 1024) Rcopy[e] = R[e];
  double sq[kFewRows] = {};
  for (int64_t d = threadIdx.x; d < D; d += 1024) {
    int p, q;
    pair_of(d, p, q);
    pairs[d] = p << 16 | q;
    double x[kFewRows], sum = 0.0;
#pragma unroll
    for (int g = 0; g < kFewRows; ++g)
      if (g < N) {
        x[g] = descriptor_entry(R + (int64_t)g * 3 * M, p, q, bad);
        X[g * D + d] = x[g];
        sum += x[g];
      }
    const double mu = sum * (1.0 / (double)N);
    mean[d] = mu;
#pragma unroll
    for (int g = 0; g < kFewRows; ++g)
      if (g < N) {
        const double c = x[g] - mu;
        Xc[g * D + d] = c;
        sq[g] += c * c;
      }
  }
#pragma unroll
  for (int g = 0; g < kFewRows; ++g) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sq[g] += __shfl_xor(sq[g], o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][g] = sq[g];
  }
  __syncthreads();
  if ((int)threadIdx.x < N) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += red[w][threadIdx.x];
    sqn[threadIdx.x] = t;
  }
}

// scale times the sums of the columns of X (N x D) over rows [rows y, rows y +
// rows), in out[y]: 16 columns a block, 16 rows at a time, eight loads in
// flight.  (64 columns a block with the whole column to four lanes ran one
// block per 64 columns whatever N: 127 us at N = 2000, 2.0 ms at N = 20000.)
__global__ __launch_bounds__(256) void k_colmean(const double* __restrict__ X, int64_t N, int64_t D, int64_t rows,
                                                 double scale, double* __restrict__ out) {
  __shared__ double part[16][17];
  const int c = threadIdx.x & 15, rg = threadIdx.x >> 4;
  const int64_t col = min((int64_t)blockIdx.x * 16 + c, D - 1);
  const int64_t r1 = min(((int64_t)blockIdx.y + 1) * rows, N);
  double s = 0.0;
#pragma unroll 8
  for (int64_t r = (int64_t)blockIdx.y * rows + rg; r < r1; r += 16) s += X[r * D + col];
  part[rg][c] = s;
  __syncthreads();
  if (rg == 0 && (int64_t)blockIdx.x * 16 + c < D) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) t += part[q][c];
    out[blockIdx.y * D + col] = t * scale;
  }
}

// X_c = X - mean, and |x_c,i|^2 (one block per geometry).
__global__ void k_center(const double* __restrict__ X, const double* __restrict__ mean, int64_t D,
                         double* __restrict__ Xc, double* __restrict__ sqn) {
  __shared__ double red[256];
  const int64_t g = blockIdx.x;
  double s = 0.0;
  for (int64_t d = threadIdx.x; d < D; d += blockDim.x) {
    const double v = X[g * D + d] - mean[d];
    Xc[g * D + d] = v;
    s += v * v;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) sqn[g] = red[0];
}

void descriptor_build(ffk_system* s, const double* R, hipStream_t st, bool coefficients) {
  const int64_t N = s->N, D = s->D;
  const int M = s->M;
  s->pairs.alloc(D * sizeof(int));
  s->R.alloc(N * M * 3 * sizeof(double));
  s->X.alloc(N * D * sizeof(double));
  s->Xc.alloc(N * D * sizeof(double));
  s->xmean.alloc(D * sizeof(double));
  s->sqn.alloc(N * sizeof(double));
  // column means: sums of 512 rows, then the sum of those
  const int S = cdiv(N, 512);
  DBuf part(S > 1 ? (size_t)S * D * 8 : 0);
  std::lock_guard<std::mutex> lock(s->ctx->flag_lock);
  s->ctx->flag.ensure(sizeof(int));
  int* bad = s->ctx->flag.as<int>();   // looked at once, at the end: nothing below depends on it
  *bad = 0;
  // up to some 10^4 elements: a block's 1024 threads take eight pairs each
  if (N <= kFewRows && N * std::max<int64_t>(D, 3 * M) <= 8192) {
    k_descriptor_few<<<1, 1024, 0, st>>>(R, (int)N, M, D, s->X.as<double>(), s->pairs.as<int>(), s->R.as<double>(),
                                         s->xmean.as<double>(), s->Xc.as<double>(), s->sqn.as<double>(), bad);
    LAUNCHCHK();
  } else {
    k_descriptor<<<cdiv(N * std::max<int64_t>(D, 3 * M), 256), 256, 0, st>>>(
        R, N, M, D, s->X.as<double>(), s->pairs.as<int>(), s->R.as<double>(), bad);
    LAUNCHCHK();
    k_colmean<<<dim3(cdiv(D, 16), S), 256, 0, st>>>(s->X.as<double>(), N, D, 512, S == 1 ? 1.0 / (double)N : 1.0,
                                                    S == 1 ? s->xmean.as<double>() : part.as<double>());
    LAUNCHCHK();
    if (S > 1) {
      k_colmean<<<dim3(cdiv(D, 16), 1), 256, 0, st>>>(part.as<double>(), S, D, S, 1.0 / (double)N,
                                                      s->xmean.as<double>());
      LAUNCHCHK();
    }
    k_center<<<N, 256, 0, st>>>(s->X.as<double>(), s->xmean.as<double>(), D, s->Xc.as<double>(), s->sqn.as<double>());
    LAUNCHCHK();
  }
  try {
    if (coefficients) ensure_coeffs(s, FFK_FP64, st);
  } catch (...) {
    (void)hipStreamSynchronize(st);   // before the flag is another build's
    throw;
  }
  HIPCHK(hipStreamSynchronize(st));
  if (*bad) fail(FFK_ERR_NONFINITE, "descriptor_build: coincident atoms or non-finite coordinates");
}

// ------------------------------------------------------------ conversions ----

// hi/lo split of a rows x cols FP64 matrix into padded bf16 arrays
// (rows_p x ld_out); entries outside rows x cols are written as zero.
// hi (+ lo) split of a rows x cols FP64 matrix into a rows_p x ld_out
// operand in fragment-major layout (K = ld_out), zero outside.
__global__ void k_split_pad(const double* __restrict__ a, int64_t rows, int64_t cols, int64_t lda,
                            int64_t rows_p, int64_t ld_out, bf16_t* __restrict__ hi,
                            bf16_t* __restrict__ lo) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows_p * ld_out) return;
  const int64_t r = e / ld_out, c = e % ld_out;
  float x = 0.f;
  if (r < rows && c < cols) x = (float)a[r * lda + c];
  const bf16_t h = f2bf(x);
  const int64_t o = frag_off(r, c, ld_out / 32);
  hi[o] = h;
  if (lo) lo[o] = f2bf(x - bf2f(h));
}

// FP32 copy of a rows x cols FP64 matrix into a padded rows_p x ld_out array.
__global__ void k_f32_pad(const double* __restrict__ a, int64_t rows, int64_t cols, int64_t lda,
                          int64_t rows_p, int64_t ld_out, float* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows_p * ld_out) return;
  const int64_t r = e / ld_out, c = e % ld_out;
  out[e] = (r < rows && c < cols) ? (float)a[r * lda + c] : 0.f;
}

// Transposed hi/lo split: a is rows x cols (lda); output cols_p x ld_out
// (fragment-major, K = ld_out) with out[c][r] = split(a[r][c]), zero
// outside.  64 x 64 tiles through LDS.
__global__ void k_split_transpose(const double* __restrict__ a, int64_t rows, int64_t cols, int64_t lda,
                                  int64_t cols_p, int64_t ld_out, bf16_t* __restrict__ hi,
                                  bf16_t* __restrict__ lo) {
  __shared__ float tile[64][65];
  const int64_t r0 = (int64_t)blockIdx.x * 64, c0 = (int64_t)blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;   // 256 threads: 64 x 4
  for (int i = ty; i < 64; i += 4) {
    const int64_t r = r0 + i, c = c0 + tx;
    tile[i][tx] = (r < rows && c < cols) ? (float)a[r * lda + c] : 0.f;
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int64_t c = c0 + i, r = r0 + tx;
    if (c < cols_p && r < ld_out) {
      const float x = tile[tx][i];
      const bf16_t h = f2bf(x);
      const int64_t o = frag_off(c, r, ld_out / 32);
      hi[o] = h;
      if (lo) lo[o] = f2bf(x - bf2f(h));
    }
  }
}

static int64_t rup(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

// out[c][r] = (T)a[r][c] for the rows x cols FP64 matrix a (lda), into a
// cols_p x ld_out array, zero outside.  64 x 64 tiles through LDS.
template <typename T>
__global__ void k_pad_transpose(const double* __restrict__ a, int64_t rows, int64_t cols, int64_t lda,
                                int64_t cols_p, int64_t ld_out, T* __restrict__ out) {
  __shared__ double tile[64][65];
  const int64_t r0 = (int64_t)blockIdx.x * 64, c0 = (int64_t)blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int64_t r = r0 + i, c = c0 + tx;
    tile[i][tx] = (r < rows && c < cols) ? a[r * lda + c] : 0.0;
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int64_t c = c0 + i, r = r0 + tx;
    if (c < cols_p && r < ld_out) out[c * ld_out + r] = (T)tile[tx][i];
  }
}

// (T)a into a rows_p x ld_out array (row-major), zero outside rows x cols.
template <typename T>
__global__ void k_pad_copy(const double* __restrict__ a, int64_t rows, int64_t cols, int64_t lda, int64_t rows_p,
                           int64_t ld_out, T* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows_p * ld_out) return;
  const int64_t r = e / ld_out, c = e % ld_out;
  out[e] = (r < rows && c < cols) ? (T)a[r * lda + c] : T(0);
}



void k_split_transpose_launch(const double* a, int64_t rows, int64_t cols, int64_t lda, int64_t cols_p,
                              int64_t ld_out, bf16_t* hi, bf16_t* lo, hipStream_t st) {
  dim3 grid(cdiv(ld_out, 64), cdiv(cols_p, 64));
  k_split_transpose<<<grid, 256, 0, st>>>(a, rows, cols, lda, cols_p, ld_out, hi, lo);
  LAUNCHCHK();
}

template <typename T>
static void padded_rows(const ffk_system* s, DBuf& P, hipStream_t st) {
  if (P) return;
  const int64_t Nr = pad_rows(s->N), Dk = rup(s->D, 64);
  DBuf t(Nr * Dk * sizeof(T));
  k_pad_copy<T><<<cdiv(Nr * Dk, 256), 256, 0, st>>>(s->Xc.as<double>(), s->N, s->D, s->D, Nr, Dk, t.as<T>());
  LAUNCHCHK();
  P = std::move(t);
}
template <typename T>
static void padded_columns(const ffk_system* s, DBuf& PT, hipStream_t st) {
  if (PT) return;
  const int64_t Nr = pad_rows(s->N), Dr = pad_rows(s->D);
  DBuf t(Dr * Nr * sizeof(T));
  dim3 grid(cdiv(Nr, 64), cdiv(Dr, 64));
  k_pad_transpose<T><<<grid, 256, 0, st>>>(s->Xc.as<double>(), s->N, s->D, s->D, Dr, Nr, t.as<T>());
  LAUNCHCHK();
  PT = std::move(t);
}

// The FP64 copies for a reader that is not a product of the system (a large
// prediction): a product may have formed them on another stream, whose work is still
// queued, and the next one may come on another stream than this call's.  So they
// are complete on return; the wait is once for each system.
void complete_padded(const ffk_system* s, hipStream_t st) {
  std::lock_guard<std::mutex> lock(s->form_lock);
  if (s->padded_complete) return;
  const bool formed = (bool)s->Xp64 || (bool)s->XpT64;
  padded_rows<double>(s, s->Xp64, st);
  padded_columns<double>(s, s->XpT64, st);
  if (formed) HIPCHK(hipDeviceSynchronize());
  else HIPCHK(hipStreamSynchronize(st));
  s->padded_complete = true;
}

void ensure_lowp_descriptor(ffk_system* s, int prec, hipStream_t st) {
  const int64_t N = s->N, D = s->D;
  if (prec == FFK_FP64) {
    std::lock_guard<std::mutex> lock(s->form_lock);
    padded_rows<double>(s, s->Xp64, st);
    padded_columns<double>(s, s->XpT64, st);
  }
  if (prec == FFK_FP32) {
    padded_rows<float>(s, s->Xp32, st);
    padded_columns<float>(s, s->XpT32, st);
  }
  if ((prec == FFK_BF16 || prec == FFK_BF16X3) && !s->Xch) {
    const int64_t Nr = pad_rows(N), Dk = rup(D, 64), Dr = pad_rows(D);
    s->Xch.alloc(Nr * Dk * 2);
    s->Xcl.alloc(Nr * Dk * 2);
    k_split_pad<<<cdiv(Nr * Dk, 256), 256, 0, st>>>(s->Xc.as<double>(), N, D, D, Nr, Dk,
                                                    s->Xch.as<bf16_t>(), s->Xcl.as<bf16_t>());
    LAUNCHCHK();
    s->XcTh.alloc(Dr * Nr * 2);
    s->XcTl.alloc(Dr * Nr * 2);
    dim3 grid(cdiv(Nr, 64), cdiv(Dr, 64));
    k_split_transpose<<<grid, 256, 0, st>>>(s->Xc.as<double>(), N, D, D, Dr, Nr, s->XcTh.as<bf16_t>(),
                                            s->XcTl.as<bf16_t>());
    LAUNCHCHK();
  }
}

// Coefficients dA = a(r) - a(0), B = b(r) of the pairs (target i, source j)
// from the Gram matrix X_t X_s^T of the centred descriptors (both centred with
// one mean): r^2 = |x_i|^2 + |x_j|^2 - 2 x_i . x_j, set to exactly zero where
// the source is the target itself (j = i + diag_off) or rounding makes it
// negative.  Rows Nt, columns Ns, stored with leading dimension ld.
struct EpiCoeffPair {
  const double *sqr, *sqc;
  double *dA, *B;
  int Nt, Ns;
  int64_t ld, diag_off;
  double inv_len, a0, bcoef;   // sqrt(5)/sigma, 5/(3 sigma^2), 25/(3 sigma^4)
  int mirror;                  // a tile below the diagonal is stored above it too
  __device__ inline void pair(int r, int c, double gram, double& d, double& b) const {
    matern_coeffs(c == r + diag_off ? 0.0 : sqr[r] + sqc[c] - 2.0 * gram, inv_len, a0, bcoef, d, b);
  }
  template <typename T, int TM, int TN, class Acc>
  __device__ void run(const Acc (&acc)[TM][TN], const FragCoord& f, char*) const {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = f.row(i, v), c = f.col(j);
          if (r < Nt && c < Ns) {
            double d, b;
            pair(r, c, (double)acc[i][j][v], d, b);
            dA[(int64_t)r * ld + c] = d;
            B[(int64_t)r * ld + c] = b;
            if (mirror && f.n0 < f.m0) {
              dA[(int64_t)c * ld + r] = d;
              B[(int64_t)c * ld + r] = b;
            }
          }
        }
  }
};

// The same for few pairs: a 16 x 16 tile a workgroup, its waves split K, rows
// straight from L2; the padding (rows to gridDim.y 16, columns to gridDim.x 16)
// is written as zeros.
__global__ __launch_bounds__(256) void k_coeff_small(const double* __restrict__ Xt, const double* __restrict__ Xs,
                                                     int D, EpiCoeffPair e) {
  __shared__ double red[4][16][17];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = blockIdx.y * 16, c0 = blockIdx.x * 16;
  const int r = r0 + (threadIdx.x >> 4), c = c0 + (threadIdx.x & 15);
  double d = 0.0, b = 0.0;
  if (r0 < e.Nt && c0 < e.Ns) {
    const int steps = (D + 7) / 8;
    const double* a[1] = {Xt + (int64_t)min(r0 + (lane & 15), e.Nt - 1) * D};
    d4 g[1] = {d4{0, 0, 0, 0}}, none[1];
    rows_dot<1, false>(a, Xs + (int64_t)min(c0 + (lane & 15), e.Ns - 1) * D, nullptr, D, steps * wave / 4,
                       steps * (wave + 1) / 4, g, none);
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][4 * v + (lane >> 4)][lane & 15] = g[0][v];
    __syncthreads();
    if (r < e.Nt && c < e.Ns) {
      const int t = threadIdx.x >> 4, s = threadIdx.x & 15;
      e.pair(r, c, (red[0][t][s] + red[1][t][s]) + (red[2][t][s] + red[3][t][s]), d, b);
    }
  }
  e.dA[(int64_t)r * e.ld + c] = d;
  e.B[(int64_t)r * e.ld + c] = b;
}

// Zeros right of column Ns and below row Nt of two Ntr x ld arrays.
__global__ void k_zero_padding(double* __restrict__ a, double* __restrict__ b, int64_t Nt, int64_t Ns, int64_t Ntr,
                               int64_t ld) {
  const int64_t w = ld - Ns, right = Nt * w;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < right + (Ntr - Nt) * ld;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t o = e < right ? e / w * ld + Ns + e % w : Nt * ld + (e - right);
    a[o] = 0.0;
    b[o] = 0.0;
  }
}

// The coefficients of e (e.Nt padded to Ntr rows) from the padded rows Xt and Xs.
static void coeff_gemm(const double* Xt, const double* Xs, int64_t D, int64_t Ntr, bool lower_only,
                       const EpiCoeffPair& e, hipStream_t st) {
  k_zero_padding<<<1024, 256, 0, st>>>(e.dA, e.B, e.Nt, e.Ns, Ntr, e.ld);
  LAUNCHCHK();
  const int64_t Dk = rup(D, 64);
  DmaArgs g{};
  g.nseg = 1;
  g.lower_only = lower_only;
  g.seg[0] = SegD{Xt, nullptr, Xs, nullptr, Dk, Dk, (int)rup(D, 8), 0};
  typedef RowTile<128, 128, 2, 4, 2> TL;
  gemm_row_kernel<double, TL, EpiCoeffPair><<<dim3(cdiv(e.Ns, 128), cdiv(e.Nt, 128)), TL::NT, 0, st>>>(g, e);
  LAUNCHCHK();
}

void rect_coeffs(const ffk_system* src, const double* Xc, const double* sq, int64_t T, int64_t Tr, int64_t ld,
                 double* Xp, double* dA, double* B, double* W, hipStream_t st) {
  const int64_t D = src->D, Dk = rup(D, 64);
  k_pad_copy<double><<<cdiv(Tr * Dk, 256), 256, 0, st>>>(Xc, T, D, D, Tr, Dk, Xp);
  LAUNCHCHK();
  k_zero_padding<<<1024, 256, 0, st>>>(W, W, T, src->N, Tr, ld);
  LAUNCHCHK();
  // (no row is a source: no column is at row + diag_off)
  const EpiCoeffPair e{sq, src->sqn.as<double>(), dA, B, (int)T, (int)src->N, ld, INT64_MIN / 2,
                       sqrt(5.0) / src->sigma, src->a0, src->bcoef, 0};
  coeff_gemm(Xp, src->Xp64.as<double>(), D, Tr, false, e, st);
}

void ensure_coeffs_pair(const ffk_system* t, const ffk_system* src, CoeffSet* sets, int prec, int64_t diag_off,
                        hipStream_t st) {
  const int64_t Nt = t->N, Ns = src->N;
  const int64_t Ntr = pad_rows(Nt), Nsr = pad_rows(Ns);
  CoeffSet& c64 = sets[FFK_FP64];
  if (!c64.ready) {
    c64.dA_hi.alloc(Ntr * Nsr * sizeof(double));
    c64.B.alloc(Ntr * Nsr * sizeof(double));
    const bool square = t == src && diag_off == 0;
    EpiCoeffPair e{t->sqn.as<double>(), src->sqn.as<double>(), c64.dA_hi.as<double>(), c64.B.as<double>(), (int)Nt,
                   (int)Ns, Nsr, diag_off, sqrt(5.0) / t->sigma, t->a0, t->bcoef, square};
    // Up to some 2000^2 pairs the small tiles, which fill the GPU at once and need
    // no padded operands; beyond, where they would read every row from L2 N /
    // 16 times, the pipelined engine, on and below the diagonal if the matrix
    // is symmetric.  The line is lower for longer rows.  Of a system's memory the
    // runtime keeps 64 MB for the next; with the padded copy, which a system that never
    // multiplies does not need, it may have to give back and map anew.  Build and
    // release, small tiles and engine, us: M = 16, N = 1500 135, 154, N = 2000 156, 492;
    // M = 30, N = 1500 210, 258, N = 1700 247, 531, N = 2000 554, 547; M = 33, N = 2000 647,
    // 546; M = 36, N = 1500 258, 283, N = 1700 589, 551; M = 48, N = 1500 318, 622.
    const int64_t most = t->D <= 448 ? 2048 * 2048 : 1536 * 1536;
    if (Ntr * Nsr <= most) {
      k_coeff_small<<<dim3((unsigned)(Nsr / 16), (unsigned)(Ntr / 16)), 256, 0, st>>>(
          t->Xc.as<double>(), src->Xc.as<double>(), (int)t->D, e);
      LAUNCHCHK();
    } else {
      for (const ffk_system* x : {t, src}) {
        std::lock_guard<std::mutex> lock(x->form_lock);
        padded_rows<double>(x, x->Xp64, st);
      }
      coeff_gemm(t->Xp64.as<double>(), src->Xp64.as<double>(), t->D, Ntr, square, e, st);
    }
    c64.ready = true;
  }
  if (prec == FFK_FP64) return;
  CoeffSet& cs = sets[prec];
  if (cs.ready) return;
  const int64_t cnt = Ntr * Nsr;
  if (prec == FFK_FP32) {
    cs.dA_hi.alloc(cnt * sizeof(float));
    cs.B.alloc(cnt * sizeof(float));
    k_pad_copy<float><<<cdiv(cnt, 256), 256, 0, st>>>(c64.dA_hi.as<double>(), Nt, Ns, Nsr, Ntr, Nsr,
                                                      cs.dA_hi.as<float>());
    LAUNCHCHK();
    k_pad_copy<float><<<cdiv(cnt, 256), 256, 0, st>>>(c64.B.as<double>(), Nt, Ns, Nsr, Ntr, Nsr, cs.B.as<float>());
    LAUNCHCHK();
  } else if (use_fused(prec, t->D, Nt, Ns)) {
    // one array in the fused product's layout: dA (hi and lo) and B
    cs.dA_hi.alloc(cnt * 8);
    fused_coef_build(c64.dA_hi.as<double>(), c64.B.as<double>(), Nt, Ns, Nsr, Ntr, Nsr, cs.dA_hi.get(), st);
  } else {
    const bool x3 = (prec == FFK_BF16X3);
    cs.dA_hi.alloc(cnt * 2);
    if (x3) cs.dA_lo.alloc(cnt * 2);
    cs.B.alloc(cnt * sizeof(float));
    k_split_pad<<<cdiv(cnt, 256), 256, 0, st>>>(c64.dA_hi.as<double>(), Nt, Ns, Nsr, Ntr, Nsr,
                                                cs.dA_hi.as<bf16_t>(), x3 ? cs.dA_lo.as<bf16_t>() : nullptr);
    LAUNCHCHK();
    k_f32_pad<<<cdiv(cnt, 256), 256, 0, st>>>(c64.B.as<double>(), Nt, Ns, Nsr, Ntr, Nsr, cs.B.as<float>());
    LAUNCHCHK();
  }
  cs.ready = true;
}

void ensure_coeffs(ffk_system* s, int prec, hipStream_t st) { ensure_coeffs_pair(s, s, s->coef, prec, 0, st); }

}  // namespace ffk
