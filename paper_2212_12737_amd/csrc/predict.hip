// Force prediction F = K(test, train) alpha (section 2.1), FP64.
//
// With U = J alpha over the N training geometries, T test geometries x_t
// (centred with the training mean: the kernel sees differences only) and the
// product's algebra,
//   P = X_t U^T, W = B o (P - 1 pd^T), G = dA U - W X_c + diag(W 1) X_t + a(0) 1 (1^T U),
// a workgroup takes 16 or 32 test geometries and 16 or 64 training ones through
// all of it: the Gram products that give dA and B and those that give P share
// the rows of X_t; dA and W stay in LDS and are the left operand of its part of
// G.  Nothing of size T x N reaches memory, only the parts of G, which a second
// kernel sums in a fixed order (they are more bytes: at M = 42, N = 5000, T = 200
// 134 MB beside the 16 MB of dA and W).  Bound by latency for a few test geometries
// and by reading the training rows from L2 for hundreds; large predictions take the
// product's GEMMs instead (predict_by_gemms).  A prediction (with the
// test system's setup) against the same products as separate scalar GEMMs on
// 128-row tiles with T x N results in memory: 442 -> 95 us at M = 21, N = 2000,
// T = 1; 1894 -> 438 us at M = 42, N = 5000, T = 200, and 360 since two
// workgroups fit a CU and their last round is a full one (205 us in this kernel, 34
// TFLOP/s).  The FP64 product of small systems runs it too (product_few).
#include <type_traits>

#include "smalldot.hpp"

namespace ffk {

struct PredictArgs {
  const double *Xt, *sqt;         // centred test rows (T x D), |x_t|^2
  const double *Xs, *sqs;         // centred training rows (N x D), |x_s|^2
  const double *U, *pd;           // J alpha (N x D), x_s . u_s
  double* part;                   // chunks x T x D parts of G
  double* wpart;                  // T x chunks row sums of W (stride planes)
  int T, N, D, chunks, tiles;
  double inv_len, a0, bcoef;
  int64_t ldu;                    // of U
  const double *dA, *B;           // KNOWN: the coefficients (T x N, ldc)
  int64_t ldc;
  int planes;                     // parts of G altogether: the stride of wpart
};

// TB blocks of 16 test geometries; CB blocks of 16 training ones (1: the four
// waves split K = D; 4: a block each).  Workgroups: the test tiles of a chunk
// of training geometries run one after the other on one XCD (workgroup w on XCD
// w % 8), which reads the chunk's rows into its L2 once.  KNOWN: a product whose
// coefficients are at hand, so that of the Gram products only P is left.
template <int TB, int CB, bool KNOWN>
__global__ __launch_bounds__(256, TB == 2 ? 2 : 1) void k_predict_part(PredictArgs g) {
  constexpr int CH = 16 * CB, TR = 16 * TB;
  __shared__ double sA[TR][CH + 1], sW[TR][CH + 1];
  __shared__ double red[CB == 1 ? 4 : 1][2][CB == 1 ? TR : 1][17];
  __shared__ double rsum[4][TR];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, q16 = lane >> 4;
  const int idx = blockIdx.x / 8, chunk = idx / g.tiles * 8 + blockIdx.x % 8;
  const int t0 = idx % g.tiles * TR, s0 = chunk * CH;
  if (chunk >= g.chunks) return;
  const int D = g.D, steps = (D + 7) / 8;
  const double* a[TB];
#pragma unroll
  for (int i = 0; i < TB; ++i) a[i] = g.Xt + (int64_t)min(t0 + 16 * i + c16, g.T - 1) * D;
  const int64_t srow = min(s0 + (CB == 1 ? 0 : 16 * wave) + c16, g.N - 1);
  d4 gm[TB], pm[TB];
#pragma unroll
  for (int i = 0; i < TB; ++i) gm[i] = pm[i] = d4{0, 0, 0, 0};
  const int k0 = CB == 1 ? steps * wave / 4 : 0, k1 = CB == 1 ? steps * (wave + 1) / 4 : steps;
  constexpr int PB = CB == 1 ? 1 : 4;   // this thread's pairs of a block of test geometries
  double known[KNOWN ? TB : 1][PB][2];
  if constexpr (KNOWN) {
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
      for (int v = 0; v < PB; ++v) {
        const int t = t0 + 16 * i + (CB == 1 ? (int)threadIdx.x >> 4 : 4 * v + q16);
        const int64_t e = (int64_t)min(t, g.T - 1) * g.ldc + min(s0 + (CB == 1 ? 0 : 16 * wave) + c16, g.N - 1);
        known[i][v][0] = g.dA[e];
        known[i][v][1] = g.B[e];
      }
    rows_dot<TB, false>(a, g.U + srow * g.ldu, nullptr, D, k0, k1, pm, gm);
  } else {
    rows_dot<TB, true>(a, g.Xs + srow * D, g.U + srow * g.ldu, D, k0, k1, gm, pm);
  }
  // dA and -W of one (test, training) pair into LDS; returns W
  auto pair = [&](int i, int v, int t, int s, double gram, double p) {
    double dA = 0.0, w = 0.0;
    if (t0 + t < g.T && s0 + s < g.N) {
      double B;
      if constexpr (KNOWN) {
        dA = known[i][v][0];
        B = known[i][v][1];
      } else {
        matern_coeffs(g.sqt[t0 + t] + g.sqs[s0 + s] - 2.0 * gram, g.inv_len, g.a0, g.bcoef, dA, B);
      }
      w = B * (p - g.pd[s0 + s]);
    }
    sA[t][s] = dA;
    sW[t][s] = -w;
    return w;
  };
  auto sum16 = [](double x) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
  };
  if constexpr (CB == 1) {
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (!KNOWN) red[wave][0][16 * i + 4 * v + q16][c16] = gm[i][v];
        red[wave][1][16 * i + 4 * v + q16][c16] = pm[i][v];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TB; ++i) {
      const int t = 16 * i + (threadIdx.x >> 4);
      double x[2] = {0.0, 0.0};
#pragma unroll
      for (int h = KNOWN ? 1 : 0; h < 2; ++h) x[h] = (red[0][h][t][c16] + red[1][h][t][c16]) + (red[2][h][t][c16] + red[3][h][t][c16]);
      const double w = sum16(pair(i, 0, t, c16, x[0], x[1]));
      if (c16 == 0) rsum[0][t] = w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = 16 * i + 4 * v + q16;
        const double w = sum16(pair(i, v, t, 16 * wave + c16, gm[i][v], pm[i][v]));
        if (c16 == 0) rsum[wave][t] = w;
      }
  }
  __syncthreads();
  if (threadIdx.x < TR && t0 + (int)threadIdx.x < g.T) {
    double w = rsum[0][threadIdx.x];
    if (CB > 1) w = (w + rsum[1][threadIdx.x]) + (rsum[2][threadIdx.x] + rsum[3][threadIdx.x]);
    g.wpart[(int64_t)(t0 + threadIdx.x) * g.planes + chunk] = w;
  }
  // this chunk's part of G: a wave takes every fourth block of 16 columns;
  // training rows past the end read the last one, against zeros of dA and W
  double* out = g.part + (int64_t)chunk * g.T * D;
  constexpr int Q = CH / 4 < 8 ? CH / 4 : 8, KB = CH / 4 / Q;   // steps of four training rows in flight, batches
  struct Rows { double u[Q], x[Q]; };
  auto load = [&](int d0, int kb, Rows& r) {
    const int d = min(d0 + c16, D - 1);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int64_t s = min(s0 + 4 * (kb * Q + q) + q16, g.N - 1);
      r.u[q] = g.U[s * g.ldu + d];
      r.x[q] = g.Xs[s * D + d];
    }
  };
  Rows r[2];
  if (16 * wave < D) load(16 * wave, 0, r[0]);
  auto block = [&](int d0, auto first) {   // first: the buffer that holds its first batch
    constexpr int F = decltype(first)::value;
    d4 ga[TB], gw[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i) ga[i] = gw[i] = d4{0, 0, 0, 0};
    // dA and W are read anew for each block: kept in registers they took 128 of
    // them, and a CU one workgroup
    if (TB == 2) asm volatile("" ::: "memory");
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      Rows& cur = r[(F + kb) & 1];
      Rows& nxt = r[(F + kb + 1) & 1];
      if (kb + 1 < KB) load(d0, kb + 1, nxt);
      else if (d0 + 64 < D) load(d0 + 64, 0, nxt);
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int i = 0; i < TB; ++i) {
          const int k = 4 * (kb * Q + q) + q16;
          ga[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(sA[16 * i + c16][k], cur.u[q], ga[i], 0, 0, 0);
          gw[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(sW[16 * i + c16][k], cur.x[q], gw[i], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = t0 + 16 * i + 4 * v + q16;
        if (t < g.T && d0 + c16 < D) out[(int64_t)t * D + d0 + c16] = ga[i][v] + gw[i][v];
      }
  };
  for (int d0 = 16 * wave; d0 < D; d0 += 128) {
    block(d0, std::integral_constant<int, 0>());
    if (d0 + 64 < D) block(d0 + 64, std::integral_constant<int, KB & 1>());
  }
}

// G[t, d] = sum of the chunks' parts + a0 s_d + w_t x_t,d: one workgroup per
// test geometry and 64 columns, its W = 16 waves each sum every sixteenth chunk
// (eight loads in flight), then meet in a fixed order.  Four waves where there are
// no more chunks.
template <int W>
__global__ __launch_bounds__(64 * W) void k_predict_reduce(const double* __restrict__ part, int chunks, int64_t T, int D,
                                                         const double* __restrict__ wpart, const double* __restrict__ s,
                                                         const double* __restrict__ Xt, double a0,
                                                         double* __restrict__ G) {
  __shared__ double sh[W][64];
  __shared__ double shw[W];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t t = blockIdx.y;
  const int d0 = blockIdx.x * 64, d = min(d0 + lane, D - 1);
  const double* p = part + t * D + d;
  double acc = 0.0, w = 0.0;
  for (int z0 = wave; z0 < chunks; z0 += W * 8) {
    double v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = p[(int64_t)min(z0 + W * e, chunks - 1) * T * D];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc += z0 + W * e < chunks ? v[e] : 0.0;
  }
  for (int z = wave * 64 + lane; z < chunks; z += 64 * W) w += wpart[t * chunks + z];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) w += __shfl_xor(w, o);
  sh[wave][lane] = acc;
  if (lane == 0) shw[wave] = w;
  __syncthreads();
  if (wave == 0 && d0 + lane < D) {
    double a = 0.0, ws = 0.0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
      a += sh[q][lane];
      ws += shw[q];
    }
    G[t * D + d] = a + a0 * s[d] + ws * Xt[t * D + d];
  }
}

template <int TB, int CB, bool KNOWN = false>
static void launch_part(const PredictArgs& g, hipStream_t st) {
  const int groups = cdiv(g.chunks, 8);
  k_predict_part<TB, CB, KNOWN><<<(unsigned)(8 * groups * g.tiles), 256, 0, st>>>(g);
  LAUNCHCHK();
}

// One kernel where its workgroups (16 targets, 16 sources up to 256 of them and
// 64 beyond) find a CU each; with D <= 128, whose GEMMs have few tiles too, up to
// 1024 sources.  One kernel against the GEMMs, us a product: M = 9, N = 200 19,
// 29; M = 21, N = 250 22, 40; M = 56, N = 512 111, 154; but M = 56, N = 600 233,
// 174; M = 9, N = 1000 29, 42; M = 16, N = 1024 45, 53; M = 21, N = 1000 61, 59.
// (32 targets a workgroup took 10 to 25% longer from M = 21 on.)
int product_few_chunks(int64_t Nt, int64_t Ns, int64_t D, size_t part_bytes) {
  int chunks = cdiv(Ns, Ns <= 256 ? 16 : 64);
  if (chunks > 16 || (D > 128 && (int64_t)chunks * cdiv(Nt, 16) > device_cus())) return 0;
  if (chunks > 8) chunks = 16;   // (counts that the reduction is compiled for; those past the sources are zeros)
  return chunks <= D && (size_t)(chunks * Nt * D * 8) <= part_bytes ? chunks : 0;
}

void product_few(const double* Xt, const double* Xs, const double* U, int64_t ldu, const double* pd, const double* dA,
                 const double* B, int64_t ldc, int64_t Nt, int64_t Ns, int64_t D, int chunks, double* part,
                 double* wpart, hipStream_t st) {
  const PredictArgs g{Xt, nullptr, Xs, nullptr, U, pd, part, wpart, (int)Nt, (int)Ns, (int)D, chunks, cdiv(Nt, 16),
                      0.0, 0.0, 0.0, ldu, dA, B, ldc, chunks};
  if (Ns <= 256) launch_part<1, 1, true>(g, st);
  else launch_part<1, 4, true>(g, st);
}

// Whether a prediction is large: then the T x N coefficients and the product's GEMMs,
// which keep their tiles' rows in LDS, take less than k_predict_part, which reads them
// from L2 for every tile (28 TFLOP/s at D <= 861, 12 to 17 where rows are longer).
// Kernel and GEMMs, us: M = 60, N = 20000, T = 100 2284 and 2489, 200 3964 and 2850, 1600
// 28105 and 11174; M = 100, N = 10000, T = 64 2373 and 2890, 100 3905 and 2976; M = 100, N
// = 3000, T = 200 1438 and 1656, 300 2283 and 1809; M = 42, N = 20000, T = 400 2157 and
// 2428, 600 3100 and 2387.  Where N is far above D the coefficients cost more than the
// parts of G: M = 21, N = 20000, T = 4000 4185 and 6900; M = 30, T = 1600 3660 and 4048.
static bool predict_by_gemms(int64_t T, int64_t N, int64_t D) {
  return (double)T * N * D >= (D >= 1024 ? 4e9 : 8e9) && 32 * D >= N;
}

// F = K(te, src) v for sources whose descriptors are centred with `mean`, with
// the model's workspace (held by the caller until the stream is done); by the GEMMs.
static void predict_large(const ffk_system* src, const double* mean, const ffk_system* te, const double* v, double* F,
                          DBuf& work, hipStream_t st) {
  const int64_t N = src->N, D = src->D;
  const int M = src->M;
  // test geometries at a time: 512 MB of what there is of them, in batches of about one size
  const int64_t row = (int64_t)(product_rows_bytes(N, D, 1 << 17) - product_rows_bytes(N, D, 1 << 16)) >> 16;
  const int64_t limit = std::max<int64_t>(128, (512ll << 20) / row / 128 * 128);
  const int64_t most = cdiv(te->N, cdiv(te->N, limit));
  work.ensure(product_rows_bytes(N, D, most));
  for (int64_t b0 = 0; b0 < te->N; b0 += most)
    product_rows(src, mean, v, te->R.as<double>() + b0 * 3 * M, te->X.as<double>() + b0 * D,
                 std::min(most, te->N - b0), most, b0 == 0, F + b0 * 3 * M, work.get(), st);
  HIPCHK(hipStreamSynchronize(st));   // the workspace may be the next call's, on another stream
}

// The same by k_predict_part, or by the GEMMs where the prediction is large.
static void predict_from(const ffk_system* src, const double* mean, const ffk_system* te, const double* v, double* F,
                         DBuf& work, hipStream_t st) {
  const int64_t N = src->N, D = src->D;
  const int M = src->M;
  if (predict_by_gemms(te->N, N, D)) {
    try {
      predict_large(src, mean, te, v, F, work, st);
      return;
    } catch (const Error& e) {   // memory is short: the kernel below needs less
      if (e.status != FFK_ERR_OOM) throw;
    }
  }
  // Test geometries at a time: up to 512, fewer where the parts of G in chunks of
  // 64 training geometries would take more than 256 MB (those of 16, of at most a
  // third of them, may double that), and more while they take no more than 16 MB: a
  // batch of a small model is its four launches (M = 3, N = 5, T = 12000: 372 us in batches
  // of 512, 80 before there were batches), while larger parts leave the last-level cache
  // (M = 42, N = 2000, T = 4000: 1.88 ms, 2.23 with 128 MB of them).
  const int64_t row = (int64_t)cdiv(N, 64) * D * 8;
  const int64_t limit = std::max(std::min<int64_t>(512, std::max<int64_t>(32, (256ll << 20) / row / 32 * 32)),
                                 std::min<int64_t>(32768, (16ll << 20) / row / 32 * 32));
  const int64_t batch = std::min<int64_t>(te->N, (cdiv(te->N, cdiv(te->N, limit)) + 31) / 32 * 32);   // of about one size
  // 32 test and 64 training geometries a workgroup where that gives every CU
  // one, else 16 test ones, and 16 training ones where even so some have none
  const int TB = batch > 16 && (int64_t)cdiv(batch, 32) * cdiv(N, 64) >= 256 ? 2 : 1;
  const int tiles = cdiv(batch, 16 * TB);
  const int CB = (int64_t)tiles * cdiv(N, 64) >= 256 ? 4 : 1;
  // Workgroups of 32 and 64 past an XCD's last full round of two a CU, if they
  // fill less than half of one, are cut to 16 and 16: at M = 42, N = 5000, T = 200
  // 70 of them on 64 places took two rounds.
  int chunks = cdiv(N, 16 * CB);
  const int64_t places = device_cus() / 4, most_xcd = (int64_t)tiles * cdiv(chunks, 8);
  int64_t tail = 0;   // training geometries in the smaller workgroups
  const int64_t in_full = most_xcd / places * places / tiles * 8;   // chunks of the full rounds (none of many tiles)
  if (TB == 2 && most_xcd % places < places / 2 && in_full > 0) {
    chunks = (int)std::min<int64_t>(chunks, in_full);
    tail = std::max<int64_t>(0, N - 64ll * chunks);
  }
  const int planes = chunks + cdiv(tail, 16);
  int64_t off = 0;
  auto take = [&](int64_t doubles) {
    const int64_t o = off;
    off += (doubles + 31) / 32 * 32;
    return o;
  };
  const int64_t oU = take(N * D), opd = take(N), os = take(D), ocp = take((int64_t)jv_blocks(N) * D);
  const int64_t oXt = take(batch * D), osq = take(batch), owp = take(batch * planes), oG = take(batch * D);
  const int64_t opart = take((int64_t)planes * batch * D);
  work.ensure(off * 8);
  double* w = work.as<double>();
  jv_fp64(src, v, w + oU, w + opd, w + ocp, w + os, te->X.as<double>(), mean, batch, w + oXt, w + osq, st);
  for (int64_t b0 = 0; b0 < te->N; b0 += batch) {
    const int T = (int)std::min<int64_t>(batch, te->N - b0);
    if (b0 > 0) center_rows(te->X.as<double>() + b0 * D, mean, T, D, w + oXt, w + osq, st);
    PredictArgs g{w + oXt, w + osq, src->Xc.as<double>(), src->sqn.as<double>(), w + oU, w + opd, w + opart, w + owp,
                  T, (int)(N - tail), (int)D, chunks, cdiv(T, 16 * TB), sqrt(5.0) / src->sigma, src->a0, src->bcoef,
                  D, nullptr, nullptr, 0, planes};
    clk_begin(CLK_FUSED, st);
    if (CB == 1) launch_part<1, 1>(g, st);
    else if (TB == 1) launch_part<1, 4>(g, st);
    else launch_part<2, 4>(g, st);
    if (tail > 0) {
      const int64_t r = N - tail;
      g.Xs += r * D; g.sqs += r; g.U += r * D; g.pd += r;
      g.part += (int64_t)chunks * T * D;
      g.wpart += chunks;
      g.N = (int)tail;
      g.chunks = planes - chunks;
      g.tiles = cdiv(T, 16);
      launch_part<1, 1>(g, st);
    }
    clk_end(CLK_FUSED, st);
    auto reduce = [&](auto waves) {
      constexpr int W = decltype(waves)::value;
      k_predict_reduce<W><<<dim3(cdiv(D, 64), T), 64 * W, 0, st>>>(w + opart, planes, T, (int)D, w + owp, w + os,
                                                                   w + oXt, src->a0, w + oG);
    };
    clk_begin(CLK_GEMM2_REDUCE, st);
    if (planes <= 4) reduce(std::integral_constant<int, 4>());
    else reduce(std::integral_constant<int, 16>());
    LAUNCHCHK();
    clk_end(CLK_GEMM2_REDUCE, st);
    jtg_rows(te->R.as<double>() + b0 * 3 * M, w + oG, te->X.as<double>() + b0 * D, T, M, D, F + b0 * 3 * M, st);
  }
  HIPCHK(hipStreamSynchronize(st));   // the workspace may be the next call's, on another stream
}

// F = K(test, train) alpha; a symmetrized training system predicts with its
// stacked permuted copies, sum_q K(test, P_q train) (Pi_q alpha)
void kernel_predict(const ffk_system* tr, const ffk_system* te, const double* alpha, double* F, hipStream_t st) {
  require(tr->M == te->M, "kernel product: the two systems differ in molecule size");
  require(tr->sigma == te->sigma, "kernel product: sigma differs");
  // The workspace stays with the model (releasing and mapping it anew cost
  // milliseconds a call); calls that share the model take turns.
  std::lock_guard<std::mutex> lock(tr->predict_lock);
  if (tr->sym.empty()) {
    predict_from(tr, tr->xmean.as<double>(), te, alpha, F, tr->predict_work, st);
    return;
  }
  tr->predict_v.ensure(tr->stack->n * 8);
  permute_stack(tr, alpha, tr->predict_v.as<double>(), st);
  predict_from(tr->stack.get(), tr->xmean.as<double>(), te, tr->predict_v.as<double>(), F, tr->predict_work, st);
}

}  // namespace ffk
