// Inducing-column selection (section 3, "Column selection strategies").
//
//  * uniform: the k columns with the largest SplitMix64 draws u_i (stream 0);
//  * weighted (leverage / scores): Efraimidis-Spirakis keys log(u_i)/w_i, k largest;
//    the ordering is (key descending, index ascending), done by a bitonic sort;
//  * pivoted (incomplete) Cholesky, Algorithm 1: greedy pivot on the largest
//    remaining diagonal of the Schur complement, in blocks of pivots (below);
//  * leverage: ridge-leverage estimates from a uniform pilot set S0,
//    tau_i = (K_ii - K_iS0 (K_S0S0 + lambda I)^-1 K_S0i) / lambda, obtained as
//    (K_ii - |row i of L0|^2)/lambda with L0 the incomplete Cholesky factor of
//    K + lambda I in the pilot order; clipped to [1e-12, 1], pilot columns 1.
#include "common.hpp"

namespace ffk {

constexpr double kWeightFloor = 1e-12;

__device__ inline bool before(double ka, int ia, double kb, int ib) {
  return ka > kb || (ka == kb && ia < ib);
}

__global__ void k_keys_uniform(int64_t n, int64_t P, uint64_t seed, int stream, double* key, int* idx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  key[i] = i < n ? uniform01_at(seed, (uint64_t)stream, (uint64_t)i) : -INFINITY;
  idx[i] = i < n ? (int)i : 0x7FFFFFFF;
}

__global__ void k_keys_weighted(int64_t n, int64_t P, const double* w, uint64_t seed, int stream, double* key,
                                int* idx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  if (i < n) {
    const double u = uniform01_at(seed, (uint64_t)stream, (uint64_t)i);
    key[i] = log(u) / fmax(w[i], kWeightFloor);
    idx[i] = (int)i;
  } else {
    key[i] = -INFINITY;
    idx[i] = 0x7FFFFFFF;
  }
}

// One global bitonic compare-exchange step (size kk, distance j).
__global__ void k_bitonic_global(double* key, int* idx, int64_t P, int64_t kk, int64_t j) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  const int64_t l = i ^ j;
  if (l <= i) return;
  const bool up = (i & kk) == 0;
  const double ki = key[i], kl = key[l];
  const int ii = idx[i], il = idx[l];
  const bool swap = up ? before(kl, il, ki, ii) : before(ki, ii, kl, il);
  if (swap) {
    key[i] = kl; key[l] = ki;
    idx[i] = il; idx[l] = ii;
  }
}

// All steps with distance <= 256 of stage kk, inside 512-element blocks.
__global__ __launch_bounds__(256) void k_bitonic_shared(double* key, int* idx, int64_t kk, int64_t jmax) {
  __shared__ double sk[512];
  __shared__ int si[512];
  const int64_t base = (int64_t)blockIdx.x * 512;
  const int t = threadIdx.x;
  sk[t] = key[base + t];
  si[t] = idx[base + t];
  sk[t + 256] = key[base + t + 256];
  si[t + 256] = idx[base + t + 256];
  __syncthreads();
  for (int64_t j = jmax; j > 0; j >>= 1) {
    const int a = (int)((t / j) * 2 * j + (t % j));   // lower element of the pair
    const int b = a + (int)j;
    const bool up = ((base + a) & kk) == 0;
    const double ka = sk[a], kb = sk[b];
    const int ia = si[a], ib = si[b];
    const bool swap = up ? before(kb, ib, ka, ia) : before(ka, ia, kb, ib);
    if (swap) {
      sk[a] = kb; sk[b] = ka;
      si[a] = ib; si[b] = ia;
    }
    __syncthreads();
  }
  key[base + t] = sk[t];
  idx[base + t] = si[t];
  key[base + t + 256] = sk[t + 256];
  idx[base + t + 256] = si[t + 256];
}

__global__ void k_take(const int* idx, int64_t k, int64_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < k) out[i] = idx[i];
}

static int64_t pow2_at_least(int64_t n) {
  int64_t p = 512;
  while (p < n) p <<= 1;
  return p;
}

static void bitonic_sort(double* key, int* idx, int64_t P, hipStream_t st) {
  for (int64_t kk = 2; kk <= P; kk <<= 1) {
    int64_t j = kk >> 1;
    for (; j > 256; j >>= 1) {
      k_bitonic_global<<<cdiv(P, 256), 256, 0, st>>>(key, idx, P, kk, j);
      LAUNCHCHK();
    }
    k_bitonic_shared<<<(unsigned)(P / 512), 256, 0, st>>>(key, idx, kk, j);
    LAUNCHCHK();
  }
}

static void topk_from_keys(int64_t n, int64_t k, DBuf& key, DBuf& idx, int64_t P, int64_t* out, hipStream_t st) {
  bitonic_sort(key.as<double>(), idx.as<int>(), P, st);
  k_take<<<cdiv(k, 256), 256, 0, st>>>(idx.as<int>(), k, out);
  LAUNCHCHK();
  HIPCHK(hipStreamSynchronize(st));
}

void select_uniform_n(int64_t n, int64_t k, uint64_t seed, int stream, int64_t* out, hipStream_t st) {
  const int64_t P = pow2_at_least(n);
  DBuf key(P * 8), idx(P * 4);
  k_keys_uniform<<<cdiv(P, 256), 256, 0, st>>>(n, P, seed, stream, key.as<double>(), idx.as<int>());
  LAUNCHCHK();
  topk_from_keys(n, k, key, idx, P, out, st);
}

void select_uniform(const ffk_system* s, int64_t k, uint64_t seed, int64_t* out, hipStream_t st) {
  select_uniform_n(s->n, k, seed, 0, out, st);
}

void select_weighted(int64_t n, const double* w, int64_t k, uint64_t seed, int stream, int64_t* out,
                     hipStream_t st) {
  const int64_t P = pow2_at_least(n);
  DBuf key(P * 8), idx(P * 4);
  k_keys_weighted<<<cdiv(P, 256), 256, 0, st>>>(n, P, w, seed, stream, key.as<double>(), idx.as<int>());
  LAUNCHCHK();
  topk_from_keys(n, k, key, idx, P, out, st);
}

// ---------------------------------------------------------- pivoted ICD ----
// Algorithm 1 in blocks of pivots.  One pivot at a time needs the whole factor
// for every column (K[:, p] - L L[p, :]^T, n m 8 bytes per pivot).  Instead a
// pool holds the Schur-complement columns of up to kPool candidates, the rows
// with the largest remaining diagonals: new ones are formed together by one
// GEMM over the factor, and each block of accepted pivots updates the rest by
// another.  Within a block the greedy choice is made on the candidates' own
// small matrix and is exact: every row outside the pool has a diagonal below
// `bound`, diagonals only fall, so as long as the best candidate is not below
// the bound it is the best of all rows (ties by index as before).  The block
// ends when it is, or when the rank test stops the factorization.  What a
// pivot costs is then a share of a few passes over n x kPool and of a K = m
// product instead of a pass over the factor: at n = 126000, k = 2000
// 415 ms became 39, of which 14 are the products that form new candidates.
constexpr int kPool = 128;       // candidates (two per lane of the greedy waves)
constexpr int kBins = 2048;      // histogram of the diagonals, 2^-10 of an octave each
constexpr int kBinShift = 10;    // of the high word

struct PivState {
  double best, bound;   // largest remaining diagonal; all rows outside the pool are below
  int s;                // pivots of the last block
  int stop;             // the largest diagonal is at the rank threshold
  int count;            // candidates listed
  int fresh;            // of them, without a column in the pool
  int first;            // lowest row with the largest diagonal
  int ones;             // pivots taken one at a time since the host last looked
  int hist[kBins];
  int list[kPool];      // candidate rows
  int row[kPool];       // pool: the row of every slot, -1 = free
  int64_t new_row[kPool];
  int new_slot[kPool];
  // the block's pivots: row, slot, pivot value, and the factor's rows at them,
  // Lt[b][j] = L[pivot j, b] for b < j
  int prow[kPool], pslot[kPool];
  double pval[kPool], pinv[kPool];   // and its inverse
  double Lt[kPool * kPool];
};

// What the host reads of a block, in pinned memory: the pivots behind the greedy
// kernel's event, the others behind the matching's.
struct PivHost {
  int s, stop, fresh;
};
class PivEvent {
 public:
  PivEvent() { HIPCHK(hipEventCreateWithFlags(&e_, hipEventDisableTiming)); }
  ~PivEvent() {   // (what the host buffer's kernels still write comes first)
    (void)hipEventSynchronize(e_);
    (void)hipEventDestroy(e_);
  }
  PivEvent(const PivEvent&) = delete;
  PivEvent& operator=(const PivEvent&) = delete;
  void record(hipStream_t st) { HIPCHK(hipEventRecord(e_, st)); }
  void wait() { HIPCHK(hipEventSynchronize(e_)); }

 private:
  hipEvent_t e_;
};

// ---- one pivot at a time: while blocks are short, the passes over the factor
// cost less than a block's launches
struct Cand {
  double v;
  int i;
};
__device__ inline Cand better(Cand a, Cand b) { return before(a.v, a.i, b.v, b.i) ? a : b; }

__device__ inline Cand block_best(Cand c, Cand* sh) {
  sh[threadIdx.x] = c;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] = better(sh[threadIdx.x], sh[threadIdx.x + o]);
    __syncthreads();
  }
  return sh[0];
}

// Best rows of blocks of 256 diagonals.
__global__ __launch_bounds__(256) void k_argmax_part(const double* d, int64_t n, Cand* part) {
  __shared__ Cand sh[256];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  Cand c{-INFINITY, 0x7FFFFFFF};
  if (i < n) c = Cand{d[i], (int)i};
  c = block_best(c, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = c;
}

__device__ inline int piv_pair(int a, int b) { return a > b ? a * (a - 1) / 2 + b : b * (b - 1) / 2 + a; }
__device__ inline double piv_wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Pivot m and column m of L.  Every block finds the best row from the partials
// (the same fixed order everywhere; block 0 writes it down) or that the rank
// test stops here.  One wave per 64 of a target geometry's 3M rows then evaluates
// them of the kernel column (lanes are rows; pair vectors from the system's table,
// PTs and Xs of the source's), subtracts L[:, :m] times the pivot's row, scales, and
// lowers the diagonals, and the block leaves its best row for the next pivot.
// A symmetrized kernel takes one launch per group element (pinv maps the
// column's atom), summed in L[:, m]; the last one finishes.
// Bound by latency at small m, by reading L later: 19 us a pivot at N = 2000 and
// small m, where a selection, a column and an update kernel took 33.  With all of a
// geometry's rows in one wave and eight loads of L in flight instead of sixteen
// 69 pivots at M = 24, N = 1092 took 1.63 ms, now 1.44 (130 at M = 22, N = 1005
// 3.62 and 2.89).
__global__ __launch_bounds__(256) void k_piv_step(const double* __restrict__ PT, const double* __restrict__ X,
                                                  const double* __restrict__ PTs, const double* __restrict__ Xs,
                                                  const int32_t* __restrict__ pinv, int64_t N, int M, int64_t D,
                                                  double inv_len, double a0, double bcoef, int add, int finish,
                                                  double* __restrict__ L, int64_t ld, int64_t m,
                                                  double thr, const Cand* __restrict__ part_in, int np_in,
                                                  PivState* __restrict__ st, int64_t* __restrict__ piv,
                                                  double* __restrict__ d, Cand* __restrict__ part_out) {
  extern __shared__ double sm[];
  constexpr int CH = 512;
  const int nw = blockDim.x >> 6;
  double* sv = sm;                       // CH values of the pivot's row
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* dW = sv + CH + wave * (D + M);
  double* uW = dW + D;
  __shared__ Cand sh[256];
  const int m3 = 3 * M;
  Cand c{-INFINITY, 0x7FFFFFFF};
  for (int e = threadIdx.x; e < np_in; e += blockDim.x) c = better(c, part_in[e]);
  c = block_best(c, sh);
  const bool go = c.i != 0x7FFFFFFF && c.v > thr;   // the same for the whole grid
  if (blockIdx.x == 0 && finish) {
    if (threadIdx.x == 0) {
      if (go) piv[m] = c.i;
      if (go) st->ones += 1;
      else st->stop = 1;
    }
    if (go && threadIdx.x < 64) {
      if (st->row[threadIdx.x] == c.i) st->row[threadIdx.x] = -1;
      if (st->row[threadIdx.x + 64] == c.i) st->row[threadIdx.x + 64] = -1;
    }
  }
  if (!go) {   // and the next launches stop here too
    if (finish && threadIdx.x == 0) part_out[blockIdx.x] = Cand{-INFINITY, 0x7FFFFFFF};
    return;
  }
  const double one_val = sqrt(c.v), one_inv = 1.0 / one_val;
  const int64_t pivot = c.i, g = pivot / m3;
  const int loc = (int)(pivot % m3), t = loc % 3;
  const int p = pinv ? pinv[loc / 3] : loc / 3;
  const int nch = (m3 + 63) / 64;   // waves of a geometry
  const int64_t task = (int64_t)blockIdx.x * nw + wave, i = task / nch;
  const bool active = i < N;
  const double* Pi = PT + (active ? i : 0) * D * 4;
  double r2 = 0.0, du = 0.0;
  if (active) {
#pragma unroll 4
    for (int64_t e = lane; e < D; e += 64) {
      const double dd = X[i * D + e] - Xs[g * D + e];
      dW[e] = dd;
      r2 = fma(dd, dd, r2);
    }
    for (int b = lane; b < M; b += 64) {
      const double w = PTs[(g * D + (b != p ? piv_pair(p, b) : 0)) * 4 + t];
      uW[b] = b == p ? 0.0 : (p > b ? -w : w);
    }
    __builtin_amdgcn_wave_barrier();
    for (int b = lane; b < M; b += 64)
      if (b != p) du = fma(dW[piv_pair(p, b)], uW[b], du);
    r2 = piv_wave_sum(r2);
    du = piv_wave_sum(du);
  }
  const double z = sqrt(r2) * inv_len;
  const double ez = exp(-z);
  const double a = a0 * (1.0 + z) * ez, bdu = -bcoef * ez * du;
  c = Cand{-INFINITY, 0x7FFFFFFF};
  {
    const int o = (int)(task % nch) * 64 + lane;
    const bool row_ok = active && o < m3;
    const int q = row_ok ? o / 3 : 0, s = row_ok ? o % 3 : 0;
    const int64_t row = i * m3 + o;
    double raw = 0.0;
    if (row_ok) {
      double jd = 0.0, ju = 0.0;   // (J^T d)_q and (J^T u)_q, component s
      constexpr int W = 12;          // pair vectors in flight
      for (int b0 = 0; b0 < M; b0 += W) {
        double w[W];
#pragma unroll
        for (int x = 0; x < W; ++x) {
          const int b = min(b0 + x, M - 1);
          w[x] = Pi[4 * (b != q ? piv_pair(q, b) : 0) + s];
        }
#pragma unroll
        for (int x = 0; x < W; ++x) {
          const int b = min(b0 + x, M - 1);
          const bool pair = b != q && b0 + x < M;
          const double ws = pair ? (q > b ? w[x] : -w[x]) : 0.0;
          jd = fma(-dW[pair ? piv_pair(q, b) : 0], ws, jd);
          ju = fma(-(q == p ? uW[b] : (b == p ? uW[q] : 0.0)), ws, ju);
        }
      }
      raw = a * ju + bdu * jd;
      if (add) raw += L[row + m * ld];
      if (!finish) L[row + m * ld] = raw;
    }
    if (!finish) return;
    constexpr int B = 16;   // columns of L in flight
    double s0 = 0.0, s1 = 0.0;
    for (int64_t j0 = 0; j0 < m; j0 += CH) {
      const int jn = (int)min((int64_t)CH, m - j0);
      __syncthreads();
      for (int j = threadIdx.x; j < (jn + B - 1) / B * B; j += blockDim.x)
        sv[j] = j < jn ? L[pivot + (j0 + j) * ld] : 0.0;
      __syncthreads();
      if (row_ok) {
        const double* Li = L + row + j0 * ld;
        for (int j = 0; j < jn; j += B) {   // columns past the last read that one, against zeros
          double v[B];
#pragma unroll
          for (int x = 0; x < B; ++x) v[x] = Li[min(j + x, jn - 1) * ld];
#pragma unroll
          for (int x = 0; x < B; x += 2) {
            s0 = fma(v[x], sv[j + x], s0);
            s1 = fma(v[x + 1], sv[j + x + 1], s1);
          }
        }
      }
    }
    if (row_ok) {
      double dn = d[row], l = 0.0;
      if (row == pivot) {
        l = one_val;
        d[row] = -INFINITY;
      } else if (dn != -INFINITY) {
        l = (raw - (s0 + s1)) * one_inv;
        dn = fma(-l, l, dn);
        d[row] = dn;
        c = better(c, Cand{dn, (int)row});
      }
      L[row + m * ld] = l;
    }
  }
  __syncthreads();
  c = block_best(c, sh);
  if (threadIdx.x == 0) part_out[blockIdx.x] = c;
}

// ---- blocks of pivots

// Columns [m, m + s) of L for this thread's row by forward substitution with
// the block's pivot rows (the arithmetic and order of Algorithm 1 within the
// block), the diagonal update and its block maxima.  A selected row has the
// diagonal -inf.  The rows of Lt are scalar loads.
__global__ __launch_bounds__(256) void k_piv_panel(double* __restrict__ L, int64_t n, int64_t ld, int64_t m,
                                                   const double* __restrict__ pool, const PivState* __restrict__ st,
                                                   double* __restrict__ d, double* __restrict__ pmax) {
  constexpr int W = 32;
  __shared__ double sh[256];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int s = st->s;
  double dn = -INFINITY;
  if (i < n) {
    dn = d[i];
    bool gone = dn == -INFINITY;
    double* Li = L + i + m * ld;
    for (int c0 = 0; c0 < s; c0 += W) {
      const int w = min(W, s - c0);
      double r[W];
#pragma unroll
      for (int j = 0; j < W; ++j) r[j] = j < w ? pool[i + st->pslot[c0 + j] * ld] : 0.0;
      for (int b = 0; b < c0; ++b) {
        const double lb = Li[b * ld];
        const double* t = st->Lt + b * kPool + c0;
#pragma unroll
        for (int j = 0; j < W; ++j) r[j] = fma(-lb, t[j], r[j]);
      }
#pragma unroll
      for (int j = 0; j < W; ++j) {
        if (j < w) {   // uniform; a break would leave the loop rolled and r in memory
          const bool own = i == st->prow[c0 + j];
          const double l = own ? st->pval[c0 + j] : (gone ? 0.0 : r[j] * st->pinv[c0 + j]);
          gone = gone || own;
          Li[(c0 + j) * ld] = l;
          if (!gone) dn = fma(-l, l, dn);
          const double* t = st->Lt + (c0 + j) * kPool + c0;
#pragma unroll
          for (int q = j + 1; q < W; ++q) r[q] = fma(-l, t[q], r[q]);
        }
      }
    }
    if (gone) dn = -INFINITY;
    d[i] = dn;
  }
  sh[threadIdx.x] = dn;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) pmax[blockIdx.x] = sh[0];
}

// Largest diagonal, the rank test, and cleared counters for the next listing.
__global__ __launch_bounds__(1024) void k_piv_begin(const double* __restrict__ pmax, int np, double thr, PivState* st) {
  __shared__ double sh[1024];
  double v = -INFINITY;
  for (int e = threadIdx.x; e < np; e += 1024) v = fmax(v, pmax[e]);
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + o]);
    __syncthreads();
  }
  for (int e = threadIdx.x; e < kBins; e += 1024) st->hist[e] = 0;
  if (threadIdx.x == 0) {
    st->best = sh[0];
    st->stop = !(sh[0] > thr);
    st->count = 0;
    st->first = 0x7FFFFFFF;
  }
}

// Histogram of the diagonals below the largest, by the high words' distance:
// bin 0 holds the largest ones.  Diagonals at the rank threshold can never be
// pivots and are left out.
__device__ inline int piv_bin(double v, double best) {
  return (int)((unsigned)(__double2hiint(best) - __double2hiint(v)) >> kBinShift);
}
__global__ __launch_bounds__(256) void k_piv_hist(const double* __restrict__ d, int64_t n, double thr, PivState* st) {
  __shared__ int h[kBins];
  for (int e = threadIdx.x; e < kBins; e += 256) h[e] = 0;
  __syncthreads();
  const double best = st->best;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double v = d[i];
    if (!(v > thr)) continue;
    const int b = piv_bin(v, best);
    if (b < kBins) atomicAdd(&h[b], 1);
    if (v == best) atomicMin(&st->first, (int)i);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kBins; e += 256)
    if (h[e]) atomicAdd(&st->hist[e], h[e]);
}

// List the rows of the first bins that together hold at most `most` rows (in
// any order); if the first bin alone holds more, only the best row.
__global__ __launch_bounds__(256) void k_piv_list(const double* __restrict__ d, int64_t n, double thr, int most,
                                                  PivState* st) {
  __shared__ int sum[256];
  __shared__ int cut;   // bins taken
  const int t = threadIdx.x;
  constexpr int PER = kBins / 256;
  int own[PER], acc = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    own[e] = st->hist[t * PER + e];
    acc += own[e];
  }
  sum[t] = acc;
  if (t == 0) cut = 0;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {   // inclusive scan
    const int x = t >= o ? sum[t - o] : 0;
    __syncthreads();
    sum[t] += x;
    __syncthreads();
  }
  int before_me = sum[t] - acc;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    before_me += own[e];
    if (before_me <= most) atomicMax(&cut, t * PER + e + 1);
  }
  __syncthreads();
  const double best = st->best;
  const int taken = cut;
  if (blockIdx.x == 0 && t == 0) {
    if (taken == 0) {
      // (the next double up: rows outside the pool may be at best itself, so that
      // after this pivot none of the pool may be taken before them)
      st->bound = __longlong_as_double(__double_as_longlong(best) + 1);
      st->list[0] = st->first;
      st->count = 1;
    } else {
      // rows not listed: high word <= that of best - (taken << shift)
      st->bound = __hiloint2double(__double2hiint(best) - (taken << kBinShift) + 1, 0);
    }
  }
  if (taken == 0) return;
  for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < n; i += (int64_t)gridDim.x * 256) {
    const double v = d[i];
    if (v > thr && piv_bin(v, best) < taken) st->list[atomicAdd(&st->count, 1)] = (int)i;
  }
}

// Match the listed rows (sorted, so that nothing depends on the order of the
// atomics) with the pool; the others get free slots, then those of rows no
// longer listed.
__global__ __launch_bounds__(kPool) void k_piv_match(PivState* st, int slots, PivHost* host) {
  __shared__ int key[kPool], row[kPool], used[kPool], avail[kPool];
  const int t = threadIdx.x;
  const int count = st->stop ? 0 : min(st->count, slots);
  key[t] = t < count ? st->list[t] : 0x7FFFFFFF;
  row[t] = t < slots ? st->row[t] : -1;
  used[t] = 0;
  __syncthreads();
  for (int kk = 2; kk <= kPool; kk <<= 1)
    for (int j = kk >> 1; j > 0; j >>= 1) {
      const int l = t ^ j;
      if (l > t) {
        const bool up = (t & kk) == 0;
        const int a = key[t], b = key[l];
        if (up ? a > b : a < b) {
          key[t] = b;
          key[l] = a;
        }
      }
      __syncthreads();
    }
  int mine = -1;   // (slots past the last hold row -1, which is no key)
#pragma unroll 16
  for (int q = 0; q < kPool; ++q)
    if (row[q] == key[t]) mine = q;
  if (t >= count) mine = -1;
  __syncthreads();
  if (mine >= 0) used[mine] = 1;
  __syncthreads();
  // this entry's rank among the unmatched ones, and this slot's among the
  // available ones: the free slots, then those whose row is no longer listed
  const bool fresh = t < count && mine < 0;
  const bool open = t < slots && row[t] < 0, stale = t < slots && row[t] >= 0 && !used[t];
  __shared__ unsigned long long bits[3][2];
  const int w = t >> 6;
  const unsigned long long bf = __ballot(fresh), bo = __ballot(open), bs = __ballot(stale);
  if ((t & 63) == 0) {
    bits[0][w] = bf;
    bits[1][w] = bo;
    bits[2][w] = bs;
  }
  __syncthreads();
  auto lower = [&](int e) {   // threads before this one
    return __popcll(bits[e][w] & ((1ull << (t & 63)) - 1)) + (w ? __popcll(bits[e][0]) : 0);
  };
  const int rank = lower(0), pos = lower(open ? 1 : 2);
  const int nfresh = __popcll(bits[0][0]) + __popcll(bits[0][1]), nopen = __popcll(bits[1][0]) + __popcll(bits[1][1]);
  if (open) avail[pos] = t;
  if (stale) avail[nopen + pos] = t;
  __syncthreads();
  if (fresh) {
    const int q = avail[rank];
    st->row[q] = key[t];
    st->new_row[rank] = key[t];
    st->new_slot[rank] = q;
  }
  if (t == 0) {
    st->fresh = nfresh;
    host->fresh = nfresh;
    host->stop = st->stop;
  }
}

// G[c][j] = L[rows[c], j0 + j] for j < w, zero for w <= j < ldg and rows of
// free slots (row-major, ldg)
template <typename I>
__global__ void k_piv_rows(const double* __restrict__ L, int64_t ld, int64_t j0, const I* __restrict__ rows, int nr,
                           int64_t w, int64_t ldg, double* __restrict__ G) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nr * ldg) return;
  const int64_t c = e / ldg, j = e % ldg;
  const int64_t r = rows[c];
  G[e] = j < w && r >= 0 ? L[r + (j0 + j) * ld] : 0.0;
}

// pool[:, new_slot[c]] = stage[:, c]
__global__ __launch_bounds__(256) void k_piv_place(const double* __restrict__ stage, int64_t n, int64_t ld,
                                                   const PivState* __restrict__ st, double* __restrict__ pool) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) pool[i + st->new_slot[blockIdx.y] * ld] = stage[i + blockIdx.y * ld];
}

// Largest value of a wave, in every lane: rotations within rows of 16 lanes,
// then the four rows' values by readlane.
template <int CTRL> __device__ inline double dpp_move(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
__device__ inline double wave_max(double x) {
  x = fmax(x, dpp_move<0x128>(x));   // row_ror:8, 4, 2, 1
  x = fmax(x, dpp_move<0x124>(x));
  x = fmax(x, dpp_move<0x122>(x));
  x = fmax(x, dpp_move<0x121>(x));
  double y = -INFINITY;
#pragma unroll
  for (int l = 0; l < 64; l += 16) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), l);
    y = fmax(y, __hiloint2double(hi, lo));
  }
  return y;
}

// A[q][c] = pool[row of slot c, slot q]: 16384 scattered reads, a few per CU (by
// the greedy block's own CU they took 40 us).
__global__ __launch_bounds__(kPool) void k_piv_gather(const double* __restrict__ pool, int64_t ld, int slots,
                                                      const PivState* __restrict__ st, double* __restrict__ A) {
  const int q = blockIdx.x, c = threadIdx.x;
  const int rq = q < slots ? st->row[q] : -1, rc = c < slots ? st->row[c] : -1;
  A[q * kPool + c] = rq >= 0 && rc >= 0 ? pool[rc + q * ld] : 0.0;
}

__device__ inline unsigned wave_max(unsigned x) {
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true));
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xF, 0xF, true));
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xF, 0xF, true));
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xF, 0xF, true));
  unsigned y = 0;
#pragma unroll
  for (int l = 0; l < 64; l += 16) y = max(y, (unsigned)__builtin_amdgcn_readlane((int)x, l));
  return y;
}

constexpr int kGreedy = 512;   // threads of k_piv_greedy

// The greedy block on the candidates' matrix A[slot][c] = pool[row of c, slot]:
// picks the best candidate, scales its row of A to its column of L over the
// candidates, and lowers the diagonals and the rest of A, until the bound.
// Wave w of eight holds the rows of the slots 16 w .. 16 w + 15 in registers
// (lane l: candidates l and l + 64); the diagonals, and so the choice of the
// pivot, are every wave's own, so that a pivot costs one barrier, behind which
// all read its column.  The choice looks at the diagonals' high words, and at
// all of them only where those tie.  Bound by the chain argmax -> root -> column -> diagonal: one wave
// that gathered A itself and formed each column from the earlier ones in LDS
// took 81 us a block of 34, now 34 and 5 for the gather.
__global__ __launch_bounds__(kGreedy) void k_piv_greedy(const double* __restrict__ A,
                                                     const double* __restrict__ d, double thr, int64_t m, int limit,
                                                     int slots, PivState* st, int64_t* __restrict__ piv, PivHost* host) {
  constexpr int RW = kPool / (kGreedy / 64);
  __shared__ double L[kPool][kPool];   // the pivots' columns
  __shared__ int row[kPool], slot_of[kPool];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int e = threadIdx.x; e < kPool; e += kGreedy) row[e] = e < slots ? st->row[e] : -1;
  __syncthreads();
  double a[RW][2], dc[2];
  int rc[2];
  const double bound = st->bound;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    rc[h] = row[lane + 64 * h];
    dc[h] = rc[h] >= 0 ? d[rc[h]] : -INFINITY;
#pragma unroll
    for (int j = 0; j < RW; ++j) a[j][h] = A[(RW * wave + j) * kPool + lane + 64 * h];
    if (rc[h] < 0) rc[h] = 0x7FFFFFFF;
  }
  int s = 0;
  while (s < limit) {
    // the best candidate: the largest diagonal, then the lowest row of those
    const unsigned k0 = dc[0] > 0.0 ? (unsigned)__double2hiint(dc[0]) : 0u;
    const unsigned k1 = dc[1] > 0.0 ? (unsigned)__double2hiint(dc[1]) : 0u;
    const unsigned top = wave_max(max(k0, k1));
    const unsigned long long at0 = __ballot(k0 == top), at1 = __ballot(k1 == top);
    double v;
    int r, p;
    if (__popcll(at0) + __popcll(at1) == 1) {
      const int owner = __ffsll(at0 | at1) - 1;
      v = lane_value(at1 ? dc[1] : dc[0], owner);
      r = __builtin_amdgcn_readlane(at1 ? rc[1] : rc[0], owner);
      p = owner + (at1 ? 64 : 0);
    } else {
      v = wave_max(fmax(dc[0], dc[1]));
      r = min(dc[0] == v ? rc[0] : 0x7FFFFFFF, dc[1] == v ? rc[1] : 0x7FFFFFFF);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) r = min(r, __shfl_xor(r, o));
      const unsigned long long lower = __ballot(dc[0] == v && rc[0] == r), upper = __ballot(dc[1] == v && rc[1] == r);
      p = lower ? __ffsll(lower) - 1 : __ffsll(upper) + 63;   // (none where all diagonals are NaN: v is no pivot)
    }
    if (!(v > thr) || (s > 0 && !(v >= bound))) break;
    r = __builtin_amdgcn_readfirstlane(r);
    if (wave == p / RW) {
      double x[2] = {a[0][0], a[0][1]};
#pragma unroll
      for (int j = 1; j < RW; ++j)
        if (p % RW == j) {
          x[0] = a[j][0];
          x[1] = a[j][1];
        }
      const double pv = sqrt(v), pinv = 1.0 / pv;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        L[s][lane + 64 * h] = p == lane + 64 * h ? pv : (dc[h] == -INFINITY ? 0.0 : x[h] * pinv);
      if (lane == 0) {
        slot_of[s] = p;
        st->prow[s] = r;
        st->pslot[s] = p;
        st->pval[s] = pv;
        st->pinv[s] = pinv;
        st->row[p] = -1;
        piv[m + s] = r;
      }
    }
    __syncthreads();
    const double x[2] = {L[s][lane], L[s][lane + 64]};
#pragma unroll
    for (int h = 0; h < 2; ++h) dc[h] = p == lane + 64 * h ? -INFINITY : fma(-x[h], x[h], dc[h]);
#pragma unroll
    for (int j = 0; j < RW; ++j) {
      const double lq = L[s][RW * wave + j];
#pragma unroll
      for (int h = 0; h < 2; ++h) a[j][h] = fma(-x[h], lq, a[j][h]);
    }
    ++s;
  }
  // the pivots' columns at the later pivots
  for (int e = threadIdx.x; e < s * kPool; e += kGreedy) {
    const int b = e / kPool, c = e % kPool;
    if (b < c && c < s) st->Lt[e] = L[b][slot_of[c]];
  }
  if (threadIdx.x == 0) {
    st->s = s;
    host->s = s;
  }
}

int64_t select_pivchol(ffk_system* s, int64_t k, int64_t* idx_out, hipStream_t st) {
  require_columns_fit(s);   // before any pivot: the single pivots' kernel would take larger molecules
  const int64_t n = s->n;
  const int64_t ld = (n + 1) / 2 * 2;   // the products move pairs of rows
  const double thr = 1e-12 * max_diag(s, st);
  DBuf L(ld * k * 8), d(n * 8), piv(k * 8), state(sizeof(PivState));
  const int np = cdiv(n, 256);
  DBuf pmax((size_t)np * 8), A(kPool * kPool * 8), pool, stage, G;
  int slots = 0;
  // the pool and its staging columns, fewer where memory is short
  auto make_pool = [&]() {
    for (slots = (int)std::min<int64_t>(kPool, n);; slots = std::max(1, slots / 4)) {
      try {
        pool.alloc(ld * slots * 8);
        stage.alloc(ld * slots * 8);
        G.alloc((size_t)slots * (k + 2) * 8);
        return;
      } catch (const Error&) {
        pool.release();
        stage.release();
        if (slots == 1) throw;
      }
    }
  };
  PivState* ps = state.as<PivState>();
  HIPCHK(hipMemsetAsync(ps, 0, sizeof(PivState), st));
  HIPCHK(hipMemsetAsync(ps->row, 0xFF, sizeof(ps->row), st));   // -1: every slot free
  kernel_diag(s, d.as<double>(), st);
  const int scan = std::min(np, 512);
  int64_t m = 0, m_pool = 0;   // pivots; the columns of L that the pool's columns already account for
  // columns [c, c + nc) of C (n x nc) -= L[:, j0 .. j0 + w) (its rows in G)^T
  auto subtract = [&](double* C, int nc, int64_t j0, int64_t w) {
    gemm64((int)n, nc, (int)w, -1.0, L.as<double>() + j0 * ld, ld, G.as<double>(), (w + 1) / 2 * 2, true, 1.0, C, ld,
           false, st);
  };
  auto panel = [&]() {
    k_piv_panel<<<np, 256, 0, st>>>(L.as<double>(), n, ld, m, pool.as<double>(), ps, d.as<double>(), pmax.as<double>());
    LAUNCHCHK();
  };
  struct { int s, stop, count, fresh, first, ones; } h;
  auto look = [&]() {
    HIPCHK(hipMemcpyAsync(&h, &ps->s, sizeof(h), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
  };
  // up to `want` pivots one at a time (fewer at the rank threshold)
  const int64_t D = s->D;
  int nw = 4;
  auto step_lds = [&](int w) { return (size_t)(512 + w * (D + s->M)) * 8; };
  while (nw > 1 && step_lds(nw) > 65536) nw >>= 1;
  const int np1 = cdiv(s->N * cdiv(3 * s->M, 64), nw);
  DBuf part_a((size_t)std::max(np, np1) * sizeof(Cand)), part_b((size_t)std::max(np, np1) * sizeof(Cand));
  auto singles = [&](int64_t want) {
    want = std::min(want, k - m);
    Cand *in = part_a.as<Cand>(), *out = part_b.as<Cand>();
    k_argmax_part<<<np, 256, 0, st>>>(d.as<double>(), n, in);
    LAUNCHCHK();
    const int S = std::max<int>(1, (int)s->sym.size());
    for (int64_t e = 0; e < want; ++e) {
      for (int q = 0; q < S; ++q) {
        const ffk_system* src = s->sym.empty() ? s : s->sym[q].get();
        k_piv_step<<<np1, 64 * nw, step_lds(nw), st>>>(
            s->PT.as<double>(), s->X.as<double>(), src->PT.as<double>(), src->X.as<double>(),
            s->sym.empty() ? nullptr : s->sym_pinv.as<int32_t>() + (size_t)q * s->M, s->N, s->M, D,
            sqrt(5.0) / s->sigma, s->a0, s->bcoef, q > 0, q == S - 1, L.as<double>(), ld, m + e, thr, in,
            e == 0 ? np : np1, ps, piv.as<int64_t>(), d.as<double>(), out);
        LAUNCHCHK();
      }
      std::swap(in, out);
    }
  };
  // Blocks start short (an early pivot lowers a whole class of rows, those of
  // one coordinate of one atom) and grow past twenty pivots.  A pivot by itself
  // takes 19 us (24 when these lines were drawn) and a pass over L, a block 300
  // us and more, and more with n (M = 22, N = 1005, k = 130: 3.9 ms with three
  // kernels a pivot, 4.1 with blocks from 64 pivots on; M = 12, N = 200, k = 180:
  // 3.7 and 2.1).  So the first pivots go one at a time, more of them at large n,
  // all where few would be left for blocks, and kFew after a block of fewer than
  // kShort while the pass is short (4e8 bytes).
  constexpr int kFew = 16, kShort = 10;
  const int64_t first = n >= 32768 ? 112 : 64;
  bool tables = pair_table(s, st);   // which the single pivots' kernel reads
  for (const auto& q : s->sym) tables = tables && pair_table(q.get(), st);
  int64_t pending = !tables ? 0 : k <= first + 2 * kFew ? k : first;   // pivots to take one at a time next
  if (!tables) panel();   // no columns: the block maxima of the diagonal
  bool running = false;         // a block whose pivot count the host has not read
  bool filled = false;          // the pool holds columns
  // The host reads a block's pivots while the diagonals are listed, and what is
  // new in the pool while its columns are brought up to date (one read of both,
  // after the listing, left the GPU idle for 40 us a block).
  HBuf host;
  PivHost* hp = nullptr;
  PivEvent greedy_done, match_done;
  for (;;) {
    if (pending > 0) {
      if (running) {
        greedy_done.wait();
        m += hp->s;
        if (m >= k) break;
      }
      singles(pending);
      look();
      m += h.ones;
      if (h.stop || m >= k) break;
      HIPCHK(hipMemsetAsync(&ps->ones, 0, sizeof(int), st));
      pending = 0;
      running = false;
      HIPCHK(hipMemsetAsync(&ps->s, 0, sizeof(int), st));
      panel();   // no columns: the block maxima of the diagonal
    }
    if (slots == 0) {
      make_pool();
      host.ensure(sizeof(PivHost));
      hp = host.as<PivHost>();
    }
    k_piv_begin<<<1, 1024, 0, st>>>(pmax.as<double>(), np, thr, ps);
    k_piv_hist<<<scan, 256, 0, st>>>(d.as<double>(), n, thr, ps);
    k_piv_list<<<scan, 256, 0, st>>>(d.as<double>(), n, thr, slots, ps);
    k_piv_match<<<1, kPool, 0, st>>>(ps, slots, hp);
    LAUNCHCHK();
    match_done.record(st);
    if (running) {
      greedy_done.wait();
      const int got = hp->s;
      m += got;
      if (tables && got < kShort && (double)n * m * 8.0 < 4e8) pending = kFew;
      if (m >= k || got == 0) break;   // (no pivot: at the rank threshold, or where a value is NaN)
    }
    if (filled && m > m_pool) {
      const int64_t w = m - m_pool, ldg = (w + 1) / 2 * 2;
      k_piv_rows<int><<<cdiv(slots * ldg, 256), 256, 0, st>>>(L.as<double>(), ld, m_pool, ps->row, slots, w, ldg,
                                                              G.as<double>());
      LAUNCHCHK();
      subtract(pool.as<double>(), slots, m_pool, w);
    }
    match_done.wait();
    h.stop = hp->stop;
    h.fresh = hp->fresh;
    if (h.stop) break;
    m_pool = m;
    filled = true;
    if (h.fresh > 0) {
      kernel_columns(s, ps->new_row, h.fresh, stage.as<double>(), ld, 0.0, st);
      if (m > 0) {
        const int64_t ldg = (m + 1) / 2 * 2;
        k_piv_rows<int64_t><<<cdiv(h.fresh * ldg, 256), 256, 0, st>>>(L.as<double>(), ld, 0, ps->new_row, h.fresh, m,
                                                                      ldg, G.as<double>());
        LAUNCHCHK();
        subtract(stage.as<double>(), h.fresh, 0, m);
      }
      k_piv_place<<<dim3(np, h.fresh), 256, 0, st>>>(stage.as<double>(), n, ld, ps, pool.as<double>());
      LAUNCHCHK();
    }
    k_piv_gather<<<kPool, kPool, 0, st>>>(pool.as<double>(), ld, slots, ps, A.as<double>());
    k_piv_greedy<<<1, kGreedy, 0, st>>>(A.as<double>(), d.as<double>(), thr, m, (int)std::min<int64_t>(k - m, kPool),
                                     slots, ps, piv.as<int64_t>(), hp);
    LAUNCHCHK();
    greedy_done.record(st);
    panel();
    running = true;
  }
  if (m > 0) HIPCHK(hipMemcpyAsync(idx_out, piv.get(), m * 8, hipMemcpyDeviceToDevice, st));
  HIPCHK(hipStreamSynchronize(st));
  return m;
}

// ------------------------------------------------------------- leverage ----
__global__ void k_leverage(const double* L0, int64_t n, int64_t ld, int64_t s, const double* diag, double lambda,
                           const unsigned char* pilot, double* tau) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double a0 = 0.0, a1 = 0.0;
  int64_t j = 0;
  for (; j + 2 <= s; j += 2) {
    const double x0 = L0[i + j * ld], x1 = L0[i + (j + 1) * ld];
    a0 += x0 * x0;
    a1 += x1 * x1;
  }
  for (; j < s; ++j) a0 += L0[i + j * ld] * L0[i + j * ld];
  double t = (diag[i] - (a0 + a1)) / lambda;
  if (pilot[i]) t = 1.0;
  tau[i] = fmin(fmax(t, kWeightFloor), 1.0);
}

__global__ void k_expand_scores(const double* geom, int64_t n, int m3, double* w) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = fmax(geom[i / m3], kWeightFloor);
}

void expand_scores(const double* geom, int64_t N, int M, double* w, hipStream_t st) {
  const int64_t n = N * 3 * M;
  k_expand_scores<<<cdiv(n, 256), 256, 0, st>>>(geom, n, 3 * M, w);
  LAUNCHCHK();
}

__global__ void k_mark(const int64_t* idx, int64_t k, unsigned char* flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < k) flag[idx[i]] = 1;
}

void leverage_estimate(ffk_system* s, const int64_t* pilot, int64_t ns, double lambda, double* tau,
                       hipStream_t st) {
  const int64_t n = s->n;
  const int64_t ld = (n + 1) / 2 * 2;   // the panel products move pairs of rows
  DBuf L0(ld * ns * 8), diag(n * 8), flag(n);
  HIPCHK(hipMemsetAsync(L0.get(), 0, ld * ns * 8, st));
  std::vector<char> kept;
  icd_forced(s, pilot, ns, lambda, L0.as<double>(), ld, &kept, st);
  kernel_diag(s, diag.as<double>(), st);
  HIPCHK(hipMemsetAsync(flag.get(), 0, n, st));
  k_mark<<<cdiv(ns, 256), 256, 0, st>>>(pilot, ns, flag.as<unsigned char>());
  LAUNCHCHK();
  k_leverage<<<cdiv(n, 256), 256, 0, st>>>(L0.as<double>(), n, ld, ns, diag.as<double>(), lambda,
                                           flag.as<unsigned char>(), tau);
  LAUNCHCHK();
  HIPCHK(hipStreamSynchronize(st));
}

}  // namespace ffk
