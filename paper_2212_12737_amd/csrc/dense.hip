// FP64 dense linear algebra on FP64 MFMA: column-major GEMM, blocked Cholesky
// and triangular inversion (column-major, lower).  Used for the k x k Woodbury
// core of the preconditioner (Eq. 4), the panel updates of the incomplete
// Cholesky and the dense factorization behind the exact leverage scores.
#include "chol64.hpp"
#include "gemm64.hpp"

namespace ffk {

// Tiles of the column-major GEMM: 16 k between barriers and, where the tile
// allows it, eight waves in two workgroups a CU.  At M = N = 8192, K = 1024 the
// 128 x 128 tile runs at 67 TFLOP/s with eight waves, 66 with four (64 x 64
// each), 62 with 32 k and one workgroup a CU, 64 as 256 x 128 by one workgroup.
typedef Tile64<128, 128, 2, 4, 2> T64L;
typedef Tile64<64, 64, 2, 2, 2> T64S;
typedef Tile64<128, 64, 4, 2, 2> T64N;
typedef Tile64<128, 96, 4, 1, 2> T64W;    // 64 < N <= 96, B k-contiguous
typedef Tile64<128, 32, 4, 1, 2> T64R;    // N <= 32
typedef Tile64<256, 64, 8, 1, 2> T64H;    // in place for M = K <= 256 (C = B) or N <= 64 (C = A)

template <class TL, bool BKC>
static void launch64(const Gemm64Args& g, EpiCol64 e, int ntn, int ntm, int batch, hipStream_t st) {
  require(reinterpret_cast<uintptr_t>(g.A) % 16 == 0 && reinterpret_cast<uintptr_t>(g.B) % 16 == 0 &&
              g.lda % 2 == 0 && g.ldb % 2 == 0 && g.sA % 2 == 0 && g.sB % 2 == 0,
          "gemm64: operands need 16-byte alignment and even leading dimensions");
  e.vec = reinterpret_cast<uintptr_t>(e.C) % 16 == 0 && e.ldc % 2 == 0 && e.sC % 2 == 0;
  k_gemm64<TL, BKC><<<dim3(ntn, ntm, batch), TL::NT, 0, st>>>(g, e);
  LAUNCHCHK();
}

template <class TL>
static void launch64(const Gemm64Args& g, const EpiCol64& e, bool b_kcontig, hipStream_t st, int batch = 1) {
  const int ntn = cdiv(g.N, TL::BN), ntm = cdiv(g.M, TL::BM);
  if (b_kcontig) launch64<TL, true>(g, e, ntn, ntm, batch, st);
  else launch64<TL, false>(g, e, ntn, ntm, batch, st);
}

void gemm64(int M, int N, int K, double alpha, const double* A, int64_t lda, const double* B, int64_t ldb,
            bool b_kcontig, double beta, double* C, int64_t ldc, bool lower_only, hipStream_t st) {
  if (M <= 0 || N <= 0) return;
  Gemm64Args g{};
  g.A = A; g.B = B; g.lda = lda; g.ldb = ldb;
  g.M = M; g.N = N; g.K = K;
  g.lower_only = lower_only;
  const EpiCol64 e{C, ldc, 0, alpha, beta, 0};
  // The larger tile where it gives every CU one: at N = 64 = K it is 24
  // against 17 TFLOP/s at M = 126016 and 9.6 against 11.2 at M = 12544, at M =
  // 2048, N = 1024, K = 256 22 against 35.  N <= 64 takes a tile
  // that spans the columns always, which is safe in place; the taller one where
  // it too gives every CU a tile and a half (M = 126016, N = 64, K = 192: 42
  // against 38).  65 to 96 columns have a tile of their own width: 203 against
  // 330 us at M = 126000 and depths about 1000, where the selection meets them.
  const int64_t large = (int64_t)cdiv(M, 128) * cdiv(N, 128) / (lower_only ? 2 : 1);
  if (large < 256) launch64<T64S>(g, e, b_kcontig, st);
  else if (N <= 32) launch64<T64R>(g, e, b_kcontig, st);
  else if (N <= 64 && large >= 768) launch64<T64H>(g, e, b_kcontig, st);
  else if (N <= 64) launch64<T64N>(g, e, b_kcontig, st);
  else if (N <= 96) launch64<T64W>(g, e, b_kcontig, st);
  else launch64<T64L>(g, e, b_kcontig, st);
}

template <bool AKC, bool BKC>
static void gemm64_in32_t(int M, int N, int K, double alpha, View32 A, View32 B, double beta, double* C, int64_t scm,
                          int64_t scn, hipStream_t st) {
  ScalarArgs<float> g{};
  g.M = M;
  g.N = N;
  g.seg = SegS<float>{A.p, A.s0, A.s1, B.p, B.s0, B.s1, K};
  EpiAxpby<double> e{C, scm, scn, M, N, alpha, beta};
  dim3 grid(cdiv(N, 128), cdiv(M, 128));
  gemm_scalar_kernel<double, 128, 128, 16, AKC, BKC, EpiAxpby<double>, float><<<grid, 256, 0, st>>>(g, e);
  LAUNCHCHK();
}

void gemm64_in32(int M, int N, int K, double alpha, View32 A, View32 B, double beta, double* C, int64_t scm,
                 int64_t scn, hipStream_t st) {
  if (M <= 0 || N <= 0) return;
  const bool akc = (A.s1 == 1), bkc = (B.s1 == 1);
  require(akc || A.s0 == 1, "gemm64_in32: A needs a unit stride");
  require(bkc || B.s0 == 1, "gemm64_in32: B needs a unit stride");
  if (akc && bkc) gemm64_in32_t<true, true>(M, N, K, alpha, A, B, beta, C, scm, scn, st);
  else if (akc) gemm64_in32_t<true, false>(M, N, K, alpha, A, B, beta, C, scm, scn, st);
  else if (bkc) gemm64_in32_t<false, true>(M, N, K, alpha, A, B, beta, C, scm, scn, st);
  else gemm64_in32_t<false, false>(M, N, K, alpha, A, B, beta, C, scm, scn, st);
}

// ------------------------------------- Cholesky and triangular inversion ----
constexpr int NB = 64, NB2 = 256;

// Cholesky of the jb x jb diagonal block at A (in place, zero above its
// diagonal) and its inverse Linv (NB x NB row-major, unit rows past jb); the
// first failing column (offset by j0) goes to info.
__global__ __launch_bounds__(256) void k_potf2(double* A, int jb, int64_t lda, int64_t j0, int64_t* info,
                                               double* Linv) {
  __shared__ Chol64 s;
  const int r = threadIdx.x % NB, cq = threadIdx.x / NB;   // a thread's elements: row r, columns cq + 4 q
  double t[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) t[q] = A[min(r, jb - 1) + min(cq + 4 * q, jb - 1) * lda];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int c = cq + 4 * q;
    s.T[r][c] = r < jb && c <= r ? t[q] : (r == c ? 1.0 : 0.0);
  }
  __syncthreads();
  chol64_inverse<false>(s, 0.0);
  __syncthreads();
  if (threadIdx.x < 64) {
    const unsigned long long bad = __ballot(s.bad[threadIdx.x] != 0);
    if (threadIdx.x == 0 && bad)
      atomicMin(reinterpret_cast<unsigned long long*>(info), (unsigned long long)(j0 + __ffsll((long long)bad) - 1));
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int c = cq + 4 * q, e = threadIdx.x + 256 * q;
    if (r < jb && c < jb) A[r + c * lda] = r >= c ? s.T[r][c] : 0.0;
    Linv[e] = s.inverse(e / NB, e % NB);
  }
}

// In-place inverse of every 64 x 64 lower-triangular diagonal block of the
// n x n matrix A, one block each; zero above their diagonals.
__global__ __launch_bounds__(256) void k_tri64(double* A, int64_t n, int64_t lda) {
  __shared__ Chol64 s;
  const int64_t j0 = (int64_t)blockIdx.x * NB;
  const int jb = (int)min((int64_t)NB, n - j0);
  double* D = A + j0 + j0 * lda;
  const int r = threadIdx.x % NB, cq = threadIdx.x / NB;
  double t[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) t[q] = D[min(r, jb - 1) + min(cq + 4 * q, jb - 1) * lda];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int c = cq + 4 * q;
    s.T[r][c] = r < jb && c <= r ? t[q] : (r == c ? 1.0 : 0.0);
  }
  __syncthreads();
  tri64_inverse(s);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int c = cq + 4 * q;
    if (r < jb && c < jb) D[r + c * lda] = s.inverse(r, c);
  }
}

// Zero the entries above the diagonal of every 256 x 256 diagonal block of A
// and, for odd n, its padding row n, which a product with a k-contiguous
// operand of odd depth reads.
__global__ void k_zero_upper_blocks(double* A, int64_t n, int64_t lda) {
  const int64_t c = blockIdx.x, j0 = c / NB2 * NB2;
  for (int64_t r = j0 + threadIdx.x; r < c; r += blockDim.x) A[r + c * lda] = 0.0;
  if ((n & 1) && threadIdx.x == 0) A[n + c * lda] = 0.0;
}

// Lower Cholesky in 256-wide panels of four 64-wide columns each.  A 64-wide
// column is one small kernel (diagonal block and its inverse), one product
// that solves the rows below it and one that updates the rest of the panel;
// the trailing matrix takes one K = 256 product per panel.  (K = 64 updates of
// the whole trailing matrix ran at the speed of HBM: about 2 TB at n = 31500.)
int64_t potrf_lower(double* A, int64_t n, int64_t lda, hipStream_t st) {
  DBuf info(8), Xinv(NB * NB * 8);
  const unsigned long long none = ~0ull;
  HIPCHK(hipMemcpyAsync(info.get(), &none, 8, hipMemcpyHostToDevice, st));
  for (int64_t J0 = 0; J0 < n; J0 += NB2) {
    const int64_t J1 = std::min<int64_t>(J0 + NB2, n);
    for (int64_t j0 = J0; j0 < J1; j0 += NB) {
      const int jb = (int)std::min<int64_t>(NB, J1 - j0);
      k_potf2<<<1, 256, 0, st>>>(A + j0 + j0 * lda, jb, lda, j0, info.as<int64_t>(), Xinv.as<double>());
      LAUNCHCHK();
      const int64_t j1 = j0 + jb;
      double* P = A + j1 + j0 * lda;   // panel <- panel L_jj^-T
      gemm64((int)(n - j1), jb, jb, 1.0, P, lda, Xinv.as<double>(), NB, true, 0.0, P, lda, false, st);
      gemm64((int)(n - j1), (int)(J1 - j1), jb, -1.0, P, lda, P, lda, false, 1.0, A + j1 + j1 * lda, lda, true, st);
    }
    const double* P = A + J1 + J0 * lda;
    gemm64((int)(n - J1), (int)(n - J1), (int)(J1 - J0), -1.0, P, lda, P, lda, false, 1.0, A + J1 + J1 * lda, lda,
           true, st);
  }
  unsigned long long h = 0;
  HIPCHK(hipMemcpyAsync(&h, info.get(), 8, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  return h == none ? -1 : (int64_t)h;
}

// In-place inverse of the lower-triangular A (n x n, lda).  The 256-wide
// diagonal blocks are inverted first, all at once: 64-wide blocks by one
// kernel, then pairs of them twice, [X11 0; -X22 L21 X11 X22], as batched
// products.  Then, with C = L below the diagonal blocks, from the first block
// column on: T = C_>j,j X_jj, C_>j,<j -= T C_j,<j (one K = 256 product over the
// whole trailing part), C_>j,j <- T, and at the end X_k,<k = -X_kk C_k,<k.
// Every large product has many tiles of equal depth.  (Block columns from the
// last on, T = X22 A21, gave at most n / 64 tiles, of depths up to n.)
void trtri_lower(double* A, int64_t n, int64_t lda, hipStream_t st) {
  if (n <= 0) return;
  const int64_t nblk = cdiv(n, NB2);
  k_tri64<<<cdiv(n, NB), 256, 0, st>>>(A, n, lda);
  LAUNCHCHK();
  if (n <= NB) return;   // one block, and nothing beside it (labels at n = 9: 116 us with the rest's launches, now 93)
  k_zero_upper_blocks<<<(unsigned)n, 64, 0, st>>>(A, n, lda);
  LAUNCHCHK();
  // products of the pairs (the second level's are the larger), later one panel
  const int64_t ldt = (n + 1) / 2 * 2;
  const size_t tb = std::max<size_t>((size_t)nblk * (NB2 / 2) * (NB2 / 2) * 8, (size_t)ldt * NB2 * 8);
  DBuf T(tb);
  HIPCHK(hipMemsetAsync(T.get(), 0, tb, st));
  for (int h = NB; h < NB2 && h < n; h *= 2) {
    const int pairs = cdiv(n, 2 * h);
    const int64_t step = 2 * h * (1 + lda);   // from one pair to the next
    Gemm64Args g{};
    g.M = h; g.N = h; g.K = h;
    g.row_step = 2 * h;
    g.row_end = n - h;   // rows left for the second block of a pair
    g.A = A + h; g.lda = lda; g.sA = step;   // L21 X11 -> T
    g.B = A; g.ldb = lda; g.sB = step;
    launch64<T64S>(g, EpiCol64{T.as<double>(), h, (int64_t)h * h, 1.0, 0.0, 0}, true, st, pairs);
    g.A = A + h + h * lda;                   // -X22 T -> X21
    g.B = T.as<double>(); g.ldb = h; g.sB = (int64_t)h * h;
    g.ktrim = 1;
    launch64<T64S>(g, EpiCol64{A + h, lda, step, -1.0, 0.0, 0}, true, st, pairs);
  }
  for (int64_t j0 = 0; j0 + NB2 < n; j0 += NB2) {
    const int64_t j1 = j0 + NB2;
    double* P = A + j1 + j0 * lda;
    const int rest = (int)(n - j1);
    gemm64(rest, NB2, NB2, 1.0, P, lda, A + j0 + j0 * lda, lda, true, 0.0, T.as<double>(), ldt, false, st);
    gemm64(rest, (int)j0, NB2, -1.0, T.as<double>(), ldt, A + j0, lda, true, 1.0, A + j1, lda, false, st);
    HIPCHK(hipMemcpy2DAsync(P, lda * 8, T.get(), ldt * 8, (size_t)rest * 8, NB2, hipMemcpyDeviceToDevice, st));
  }
  if (nblk > 1) {   // rows of block k >= 1, all its columns left of the diagonal block, in place
    Gemm64Args g{};
    g.M = NB2; g.N = (int)((nblk - 1) * NB2); g.K = NB2;
    g.A = A; g.lda = lda; g.sA = NB2 * (1 + lda);
    g.B = A; g.ldb = lda; g.sB = NB2;
    g.row_step = NB2; g.row_end = n;
    g.ktrim = 1;
    g.ncol_step = NB2;
    launch64<T64H>(g, EpiCol64{A, lda, NB2, -1.0, 0.0, 0}, true, st, (int)nblk);
  }
  HIPCHK(hipStreamSynchronize(st));   // T is released on return
}

}  // namespace ffk
