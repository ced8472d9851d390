// Score network for learned inducing-column selection: D -> H -> H -> 1 with
// exact-erf GELU, trained in FP32 on FP32 MFMA (forward, backward and Adam are
// the kernels below), inferred either in FP32 or in BF16 on MFMA with FP32
// accumulation.  The network maps a standardised descriptor to a predicted
// log block leverage score; sampling weights are exp(prediction) (the
// Efraimidis-Spirakis keys are invariant to a common scale).
//
// Parameter layout (floats): W1 (H x D row-major), b1 (H), W2 (H x H), b2 (H),
// w3 (H), b3 (1); after the parameters: input mean (D) and inverse std (D).
#include <type_traits>

#include "gemm.hpp"

namespace ffk {

__device__ inline float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
struct Offs {
  int64_t W1, b1, W2, b2, w3, b3, mean, istd, end;
};
static Offs offs(int D, int H) {
  Offs o;
  o.W1 = 0;
  o.b1 = o.W1 + (int64_t)H * D;
  o.W2 = o.b1 + H;
  o.b2 = o.W2 + (int64_t)H * H;
  o.w3 = o.b2 + H;
  o.b3 = o.w3 + H;
  o.mean = o.b3 + 1;
  o.istd = o.mean + D;
  o.end = o.istd + D;
  return o;
}

// --------------------------------------------------------------- epilogues ----
// H = gelu(acc + bias[c]) (row-major, ld), in FP32 or bf16.
struct EpiBiasGelu {
  const float* bias;
  float* Hout;
  bf16_t* Hbf;   // optional bf16 copy of H (ldb)
  int64_t ld, ldb;
  int M, N;
  template <typename T, int TM, int TN, class Acc>
  __device__ void run(const Acc (&acc)[TM][TN], const FragCoord& f, char*) const {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = f.row(i, v), c = f.col(j);
          if (r < M && c < N) {
            const float z = (float)acc[i][j][v] + bias[c];
            const float h = gelu_f(z);
            if (Hout) Hout[(int64_t)r * ld + c] = h;
            if (Hbf) Hbf[(int64_t)r * ldb + c] = f2bf(h);
          }
        }
  }
};

// ----------------------------------------------------------- small kernels ----
// out[b] = H2[b] . w3 + b3 (one wave per row)
__global__ __launch_bounds__(256) void k_rowdot(const float* H2, int64_t B, int H, const float* w3, const float* b3,
                                                float* out) {
  const int lane = threadIdx.x & 63;
  const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= B) return;
  float a = 0.f;
  for (int h = lane; h < H; h += 64) a += H2[b * H + h] * w3[h];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  if (lane == 0) out[b] = a + b3[0];
}

// ------------------------------------------- FP32 forward and backward ----
// The layers are small (256 x 256 x 256 in training), so what counts is
// launches, workgroups and latency: a T x T tile (16 or 32) per workgroup, its
// four waves split K, fragments go from global memory (L2) straight to
// registers, four 16-wide steps of K in flight, and everything elementwise or
// reduced rides in the epilogues.  A gradient takes four kernels:
//   1. H1 = gelu(X W1^T + b1), G1 = gelu'
//   2. H2 = gelu(H1 W2^T + b2), G2 = w3 gelu', and the partials of out = H2 w3 + b3
//   3. with dout = 2 (out - y) / B, a scale of the rows:  dZ1 = dout (G2 W2) G1,
//      g_W2 = (dout G2)^T H1, g_b2, g_w3, g_b3 and the loss
//   4. g_W1 = dZ1^T X, g_b1
// At D = 210, H = B = 256 a gradient and Adam step takes 25 us; on 128 x 128
// tiles (four workgroups to a layer) and twelve kernels it took 404.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // rows of odd length

__device__ inline void gelu_both(float x, float& h, float& g) {
  const float c = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
  h = x * c;
  g = c + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

// The wave's part of sum_k A(m, k) B(n, k) for the T x T tile at (m0, n0),
// summed over the waves in red[0].  KC: element (m, k) at A[m lda + k], else
// at A[k lda + m].  kscale (not null): a factor of every k.  Lane l takes rows
// l % 16 and k = 16 s + 4 (l / 16) + j in MFMA j of step s.
template <int T, bool AKC, bool BKC>
__device__ inline void mlp_tile(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
                                int M, int N, int K, int m0, int n0, const float* kscale, float (*red)[T][T + 1]) {
  constexpr int NB = T / 16, U = 4;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, kq = 4 * (lane >> 4);
  const int steps = (K + 15) / 16;
  const int s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
  f4 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f4{0, 0, 0, 0};
  auto fetch = [&](auto kc, const float* P, int64_t ld, int row, int k) {
    f4 v;
    if constexpr (decltype(kc)::value) {
      const float* src = P + row * ld + k;
      if (k + 3 < K) {
        v = *reinterpret_cast<const f4u*>(src);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = k + j < K ? src[j] : 0.f;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x = P[(int64_t)min(k + j, K - 1) * ld + row];
        v[j] = k + j < K ? x : 0.f;
      }
    }
    return v;
  };
  for (int s = s0; s < s1; s += U) {
    f4 a[U][NB], b[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s + u < s1) {
        const int k = 16 * (s + u) + kq;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          a[u][i] = fetch(std::integral_constant<bool, AKC>(), A, lda, min(m0 + 16 * i + r, M - 1), k);
          b[u][i] = fetch(std::integral_constant<bool, BKC>(), B, ldb, min(n0 + 16 * i + r, N - 1), k);
        }
        if (kscale) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float f = k + j < K ? kscale[min(k + j, K - 1)] : 0.f;   // (not the last one: 0 times infinity)
#pragma unroll
            for (int i = 0; i < NB; ++i) a[u][i][j] *= f;
          }
        }
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s + u < s1) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][q], b[u][j][q], acc[i][j], 0, 0, 0);
      }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][16 * i + (lane >> 4) * 4 + v][16 * j + r] = acc[i][j][v];
  __syncthreads();
}
template <int T> __device__ inline float mlp_sum(const float (*red)[T][T + 1], int r, int c) {
  return (red[0][r][c] + red[1][r][c]) + (red[2][r][c] + red[3][r][c]);
}

// Hout = gelu(Z), Z = X W^T + bias for B rows (K inputs, H outputs); with G,
// G = gelu'(Z) (times w3 when given); with w3, outp[tile column][row] = the
// tile's part of Hout . w3.  Hout may be null.
template <int T>
__global__ __launch_bounds__(256) void k_mlp_layer(const float* __restrict__ X, const float* __restrict__ W,
                                                   const float* __restrict__ bias, int B, int K, int H,
                                                   float* __restrict__ Hout, float* __restrict__ G,
                                                   const float* __restrict__ w3, float* __restrict__ outp) {
  __shared__ float red[4][T][T + 1];
  const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
  mlp_tile<T, true, true>(X, K, W, K, B, H, K, m0, n0, nullptr, red);
  for (int e = threadIdx.x; e < T * T; e += 256) {   // T consecutive lanes share a row
    const int r = m0 + e / T, c = n0 + e % T;
    float h, g;
    gelu_both(mlp_sum<T>(red, e / T, e % T) + bias[c], h, g);
    const float w = w3 ? w3[c] : 1.f;
    if (r < B) {
      if (Hout) Hout[(int64_t)r * H + c] = h;
      if (G) G[(int64_t)r * H + c] = w * g;
    }
    if (w3) {
      float p = h * w;
#pragma unroll
      for (int o = T / 2; o > 0; o >>= 1) p += __shfl_xor(p, o);
      if (e % T == 0 && r < B) outp[(int64_t)blockIdx.x * B + r] = p;
    }
  }
}

__device__ inline float mlp_out(const float* outp, int nt, int64_t B, const float* b3, int64_t b) {
  float o = b3[0];
  for (int t0 = 0; t0 < nt; t0 += 16) {   // sixteen loads in flight
    float p[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) p[t] = outp[min(t0 + t, nt - 1) * B + b];
#pragma unroll
    for (int t = 0; t < 16; ++t) o += t0 + t < nt ? p[t] : 0.f;
  }
  return o;
}
__device__ inline float mlp_dout(float out, float y, int64_t B) { return 2.0f * (out - y) / (float)B; }

__global__ void k_mlp_out(const float* __restrict__ outp, int nt, int64_t B, const float* __restrict__ b3,
                          float* __restrict__ out) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) out[b] = mlp_out(outp, nt, B, b3, b);
}
__global__ void k_mlp_dout(const float* __restrict__ outp, int nt, int64_t B, const float* __restrict__ b3,
                           const float* __restrict__ y, float* __restrict__ dout) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) dout[b] = mlp_dout(mlp_out(outp, nt, B, b3, b), y[b], B);
}

// sums of 16 columns over the B rows of a (and of a2, when given), each row
// times f[row] (f null: 1): 16 lanes a row, 16 rows at a time, fixed order
__device__ inline void mlp_colsums(const float* a, const float* a2, int B, int H, int c0, const float* f, float* s1,
                                   float* s2, float (*sh)[16][17]) {
  const int c = threadIdx.x & 15, rg = threadIdx.x >> 4;
  float x = 0.f, x2 = 0.f;
#pragma unroll 8
  for (int b = rg; b < B; b += 16) {
    const float w = f ? f[b] : 1.f;
    x += w * a[(int64_t)b * H + c0 + c];
    if (a2) x2 += w * a2[(int64_t)b * H + c0 + c];
  }
  sh[0][rg][c] = x;
  sh[1][rg][c] = x2;
  __syncthreads();
  if (threadIdx.x < 32) {
    const int which = threadIdx.x >> 4;
    float s = 0.f;
    for (int q = 0; q < 16; ++q) s += sh[which][q][c];
    if (which == 0) s1[c0 + c] = s;
    else if (s2) s2[c0 + c] = s;
  }
}

constexpr int kDoutLds = 1024;   // batches up to this form dout in the LDS of every workgroup that needs it

// Step 3 above.  Workgroups: the tiles of dZ1, then those of g_W2, then H / 16
// for g_b2 and g_w3, then one for the loss and g_b3.  dout: precomputed for
// batches beyond kDoutLds, else null.
template <int T>
__global__ __launch_bounds__(256) void k_mlp_back2(const float* __restrict__ G1, const float* __restrict__ H1,
                                                   const float* __restrict__ G2, const float* __restrict__ H2,
                                                   const float* __restrict__ W2, const float* __restrict__ outp, int nt,
                                                   const float* __restrict__ b3, const float* __restrict__ y,
                                                   const float* __restrict__ dout, int B, int H,
                                                   float* __restrict__ dZ1, float* __restrict__ gW2,
                                                   float* __restrict__ gb2, float* __restrict__ gw3,
                                                   float* __restrict__ gb3, float* __restrict__ loss) {
  __shared__ float red[4][T][T + 1];
  __shared__ float sd[kDoutLds];
  __shared__ float sh[2][16][17];
  const int nh = H / T, ntz = nh * ((B + T - 1) / T), ntw = nh * nh;
  int w = blockIdx.x;
  if (w < ntz) {
    const int m0 = w / nh * T, n0 = w % nh * T;
    if (threadIdx.x < T) {
      const int b = min(m0 + (int)threadIdx.x, B - 1);
      sd[threadIdx.x] = dout ? dout[b] : mlp_dout(mlp_out(outp, nt, B, b3, b), y[b], B);
    }
    mlp_tile<T, true, false>(G2, H, W2, H, B, H, H, m0, n0, nullptr, red);
    for (int e = threadIdx.x; e < T * T; e += 256) {
      const int r = m0 + e / T, c = n0 + e % T;
      if (r < B) {
        const int64_t o = (int64_t)r * H + c;
        dZ1[o] = sd[e / T] * mlp_sum<T>(red, e / T, e % T) * G1[o];
      }
    }
    return;
  }
  w -= ntz;
  const float* f = dout;
  if (!f) {
    for (int b = threadIdx.x; b < B; b += 256) sd[b] = mlp_dout(mlp_out(outp, nt, B, b3, b), y[b], B);
    f = sd;
    __syncthreads();
  }
  if (w < ntw) {
    const int m0 = w / nh * T, n0 = w % nh * T;
    mlp_tile<T, false, false>(G2, H, H1, H, H, H, B, m0, n0, f, red);
    for (int e = threadIdx.x; e < T * T; e += 256)
      gW2[(int64_t)(m0 + e / T) * H + n0 + e % T] = mlp_sum<T>(red, e / T, e % T);
    return;
  }
  w -= ntw;
  if (w < H / 16) {
    mlp_colsums(G2, H2, B, H, 16 * w, f, gb2, gw3, sh);
    return;
  }
  __shared__ double sl[256], sb[256];
  double l = 0.0, g = 0.0;
  for (int b = threadIdx.x; b < B; b += 256) {
    const float d = mlp_out(outp, nt, B, b3, b) - y[b];
    l += (double)d * d;
    g += f[b];
  }
  sl[threadIdx.x] = l;
  sb[threadIdx.x] = g;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sl[threadIdx.x] += sl[threadIdx.x + o];
      sb[threadIdx.x] += sb[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    loss[0] = (float)(sl[0] / (double)B);
    gb3[0] = (float)sb[0];
  }
}

// Step 4: the tiles of g_W1 = dZ1^T X, then H / 16 workgroups for g_b1.
template <int T>
__global__ __launch_bounds__(256) void k_mlp_back1(const float* __restrict__ dZ1, const float* __restrict__ X, int B,
                                                   int D, int H, float* __restrict__ gW1, float* __restrict__ gb1) {
  __shared__ float red[4][T][T + 1];
  __shared__ float sh[2][16][17];
  const int nd = (D + T - 1) / T, nt = nd * (H / T);
  const int w = blockIdx.x;
  if (w < nt) {
    const int m0 = w / nd * T, n0 = w % nd * T;
    mlp_tile<T, false, false>(dZ1, H, X, D, H, D, B, m0, n0, nullptr, red);
    for (int e = threadIdx.x; e < T * T; e += 256) {
      const int c = n0 + e % T;
      if (c < D) gW1[(int64_t)(m0 + e / T) * D + c] = mlp_sum<T>(red, e / T, e % T);
    }
    return;
  }
  mlp_colsums(dZ1, nullptr, B, H, 16 * (w - nt), nullptr, gb1, nullptr, sh);
}

__global__ void k_adam(float* theta, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  theta[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// bf16 copy of a rows x cols FP32 matrix into a zero-padded rows_p x ld array
__global__ void k_f32_to_bf16_pad(const float* a, int64_t rows, int64_t cols, int64_t lda, int64_t rows_p, int64_t ld,
                                  bf16_t* out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows_p * ld) return;
  const int64_t r = e / ld, c = e % ld;
  out[e] = (r < rows && c < cols) ? f2bf(a[r * lda + c]) : (bf16_t)0;
}

// standardised descriptor rows of a system as bf16 (rows_p x ld, zero padded)
__global__ void k_standardize_bf16(const double* X, int64_t N, int64_t D, const float* mean, const float* istd,
                                   int64_t rows_p, int64_t ld, bf16_t* out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows_p * ld) return;
  const int64_t r = e / ld, c = e % ld;
  out[e] = (r < N && c < D) ? f2bf((float)((X[r * D + c] - mean[c]) * istd[c])) : (bf16_t)0;
}

__global__ void k_exp_scores(const float* out, int64_t N, double* scores) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) scores[i] = exp((double)out[i]);
}

// ------------------------------------------------------------------ driver ----
static int64_t rup(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

ffk_mlp* mlp_create(int32_t D, int32_t H, uint64_t seed) {
  std::unique_ptr<ffk_mlp> m(new ffk_mlp());
  m->D = D;
  m->H = H;
  const Offs o = offs(D, H);
  m->nparam = o.mean;
  m->theta.alloc(o.end * 4);
  m->m.alloc(m->nparam * 4);
  m->v.alloc(m->nparam * 4);
  // uniform(-1/sqrt(fan_in), 1/sqrt(fan_in)) weights, zero biases; identity standardisation
  std::vector<float> h(o.end, 0.f);
  uint64_t ctr = 0;
  auto fill = [&](int64_t off, int64_t cnt, int fan_in) {
    const double a = 1.0 / sqrt((double)fan_in);
    for (int64_t i = 0; i < cnt; ++i) h[off + i] = (float)((2.0 * uniform01_at(seed, 4, ctr++) - 1.0) * a);
  };
  fill(o.W1, (int64_t)H * D, D);
  fill(o.W2, (int64_t)H * H, H);
  fill(o.w3, H, H);
  for (int64_t i = 0; i < D; ++i) h[o.istd + i] = 1.f;
  HIPCHK(hipMemcpy(m->theta.get(), h.data(), o.end * 4, hipMemcpyHostToDevice));
  HIPCHK(hipMemset(m->m.get(), 0, m->nparam * 4));
  HIPCHK(hipMemset(m->v.get(), 0, m->nparam * 4));
  return m.release();
}

// Tile edge of the FP32 kernels: 32 where that still makes two workgroups a
// CU, else 16.
static int mlp_edge(int64_t M, int64_t N) { return (int64_t)cdiv(M, 32) * cdiv(N, 32) >= 512 ? 32 : 16; }

// Activations of a batch: H1, G1, H2, G2, dZ1 (B x H each), the partials of
// out (at most H / 16 x B) and dout (B)
static float* act(const ffk_mlp* net, int64_t B) {
  const int64_t need = (6 * B * net->H + 2 * B) * 4;
  ffk_mlp* m = const_cast<ffk_mlp*>(net);
  m->work.ensure(need);
  return m->work.as<float>();
}

static void mlp_layer(const float* X, const float* W, const float* bias, int64_t B, int K, int H, float* Hout, float* G,
                      const float* w3, float* outp, hipStream_t st) {
  if (mlp_edge(B, H) == 32)
    k_mlp_layer<32><<<dim3(H / 32, cdiv(B, 32)), 256, 0, st>>>(X, W, bias, (int)B, K, H, Hout, G, w3, outp);
  else
    k_mlp_layer<16><<<dim3(H / 16, cdiv(B, 16)), 256, 0, st>>>(X, W, bias, (int)B, K, H, Hout, G, w3, outp);
  LAUNCHCHK();
}

static void forward_bf16(const ffk_mlp* net, const bf16_t* Xb, int64_t B, int64_t ldx, float* out, hipStream_t st) {
  const int D = net->D, H = net->H;
  const Offs o = offs(D, H);
  ffk_mlp* m = const_cast<ffk_mlp*>(net);
  const int64_t Dk = rup(D, 64), Hr = rup(H, 128), Br = rup(B, 128);
  require(ldx == Dk, "mlp: bf16 input leading dimension mismatch");
  const float* th = net->theta.as<float>();
  if (!m->wbf_valid) {
    m->wbf.ensure((Hr * Dk + Hr * rup(H, 64)) * 2);
    bf16_t* w1 = m->wbf.as<bf16_t>();
    bf16_t* w2 = w1 + Hr * Dk;
    k_f32_to_bf16_pad<<<cdiv(Hr * Dk, 256), 256, 0, st>>>(th + o.W1, H, D, D, Hr, Dk, w1);
    LAUNCHCHK();
    k_f32_to_bf16_pad<<<cdiv(Hr * rup(H, 64), 256), 256, 0, st>>>(th + o.W2, H, H, H, Hr, rup(H, 64), w2);
    LAUNCHCHK();
    m->wbf_valid = true;
  }
  const bf16_t* w1 = m->wbf.as<bf16_t>();
  const bf16_t* w2 = w1 + Hr * Dk;
  const int64_t Hk = rup(H, 64);
  DBuf h1b(Br * Hk * 2), h2(Br * H * 4);
  HIPCHK(hipMemsetAsync(h1b.get(), 0, Br * Hk * 2, st));
  {
    const Bf16Args g{Xb, w1, Dk, Dk, (int)Dk};
    EpiBiasGelu e{th + o.b1, nullptr, h1b.as<bf16_t>(), 0, Hk, (int)B, H};
    gemm_bf16_kernel<128, 128, 64, EpiBiasGelu><<<dim3(Hr / 128, Br / 128), 256, 0, st>>>(g, e);
    LAUNCHCHK();
  }
  {
    const Bf16Args g{h1b.as<bf16_t>(), w2, Hk, Hk, (int)Hk};
    EpiBiasGelu e{th + o.b2, h2.as<float>(), nullptr, H, 0, (int)B, H};
    gemm_bf16_kernel<128, 128, 64, EpiBiasGelu><<<dim3(Hr / 128, Br / 128), 256, 0, st>>>(g, e);
    LAUNCHCHK();
  }
  k_rowdot<<<cdiv(B, 4), 256, 0, st>>>(h2.as<float>(), B, H, th + o.w3, th + o.b3, out);
  LAUNCHCHK();
  HIPCHK(hipStreamSynchronize(st));   // temporaries are freed on return
}

// Whether a forward pass is large: whose tiles of 128 x 128 (64 wide for H = 64) make two
// a CU, or one with a first layer that is deep.  Tiles of 32 from L2 read every operand
// four times as often, and are ahead only where the larger ones leave CUs idle.  A
// pass by tiles of 32 and through LDS, us: D = 1770, H = 1024, B = 8192 1059 and 601; D =
// 210, H = 256, B = 32768 210 and 166; one tile a CU, D = 861, H = 256, B = 16384 254 and
// 201, but D = 210, H = 512, B = 8192 161 and 195.
static bool forward_through_lds(int64_t B, int D, int H) {
  const int64_t tiles = (int64_t)cdiv(B, 128) * cdiv(H, 128), cus = device_cus();
  return tiles >= 2 * cus || (tiles >= cus && D >= 512);
}

// Hout = gelu(X W^T + bias) through LDS: 128 x 128 tiles (64 wide for H = 64).
static void mlp_layer_lds(const float* X, const float* W, const float* bias, int64_t B, int K, int H, float* Hout,
                          hipStream_t st) {
  ScalarArgs<float> g{};
  g.M = (int)B;
  g.N = H;
  g.seg = SegS<float>{X, K, 1, W, K, 1, K};
  const EpiBiasGelu e{bias, Hout, nullptr, H, 0, (int)B, H};
  // three of the wider tiles share a CU, so that a few past that many start alone (D =
  // 36, H = 128, B = 100000 179 us, 146 by the narrower)
  const int64_t wide = (int64_t)cdiv(H, 128) * cdiv(B, 128), cus = device_cus();
  if (H <= 64 || (wide > 3 * cus && wide <= 4 * cus))
    gemm_scalar_kernel<float, 128, 64, 16, true, true, EpiBiasGelu>
        <<<dim3(cdiv(H, 64), cdiv(B, 128)), 256, 0, st>>>(g, e);
  else
    gemm_scalar_kernel<float, 128, 128, 16, true, true, EpiBiasGelu>
        <<<dim3(cdiv(H, 128), cdiv(B, 128)), 256, 0, st>>>(g, e);
  LAUNCHCHK();
}

void mlp_forward(const ffk_mlp* net, const float* X, int64_t B, float* out, int prec, hipStream_t st) {
  if (prec == FFK_FP32) {
    const int D = net->D, H = net->H;
    const Offs o = offs(D, H);
    const float* th = net->theta.as<float>();
    float* H1 = act(net, B);
    if (forward_through_lds(B, D, H)) {
      float* H2 = H1 + B * H;
      mlp_layer_lds(X, th + o.W1, th + o.b1, B, D, H, H1, st);
      mlp_layer_lds(H1, th + o.W2, th + o.b2, B, H, H, H2, st);
      k_rowdot<<<cdiv(B, 4), 256, 0, st>>>(H2, B, H, th + o.w3, th + o.b3, out);
      LAUNCHCHK();
      return;
    }
    float* outp = H1 + B * H;
    mlp_layer(X, th + o.W1, th + o.b1, B, D, H, H1, nullptr, nullptr, nullptr, st);
    mlp_layer(H1, th + o.W2, th + o.b2, B, H, H, nullptr, nullptr, th + o.w3, outp, st);
    k_mlp_out<<<cdiv(B, 256), 256, 0, st>>>(outp, H / mlp_edge(B, H), B, th + o.b3, out);
    LAUNCHCHK();
    return;
  }
  const int64_t Dk = rup(net->D, 64), Br = rup(B, 128);
  DBuf xb(Br * Dk * 2);
  k_f32_to_bf16_pad<<<cdiv(Br * Dk, 256), 256, 0, st>>>(X, B, net->D, net->D, Br, Dk, xb.as<bf16_t>());
  LAUNCHCHK();
  forward_bf16(net, xb.as<bf16_t>(), B, Dk, out, st);
}

void mlp_grad(ffk_mlp* net, const float* X, const float* y, int64_t B, float* loss, float* grad, hipStream_t st) {
  const int D = net->D, H = net->H;
  const Offs o = offs(D, H);
  const float* th = net->theta.as<float>();
  const int64_t bh = B * H;
  float *H1 = act(net, B), *G1 = H1 + bh, *H2 = H1 + 2 * bh, *G2 = H1 + 3 * bh, *dZ1 = H1 + 4 * bh;
  float *outp = H1 + 5 * bh, *dout = H1 + 6 * bh;
  mlp_layer(X, th + o.W1, th + o.b1, B, D, H, H1, G1, nullptr, nullptr, st);
  mlp_layer(H1, th + o.W2, th + o.b2, B, H, H, H2, G2, th + o.w3, outp, st);
  const int nt = H / mlp_edge(B, H);
  if (B > kDoutLds) {
    k_mlp_dout<<<cdiv(B, 256), 256, 0, st>>>(outp, nt, B, th + o.b3, y, dout);
    LAUNCHCHK();
  } else {
    dout = nullptr;
  }
  auto back = [&](auto edge) {
    constexpr int T = decltype(edge)::value;
    const int grid = H / T * cdiv(B, T) + H / T * (H / T) + H / 16 + 1;
    k_mlp_back2<T><<<grid, 256, 0, st>>>(G1, H1, G2, H2, th + o.W2, outp, nt, th + o.b3, y, dout, (int)B, H, dZ1,
                                         grad + o.W2, grad + o.b2, grad + o.w3, grad + o.b3, loss);
    LAUNCHCHK();
  };
  if (mlp_edge(B, H) == 32) back(std::integral_constant<int, 32>());
  else back(std::integral_constant<int, 16>());
  if (mlp_edge(H, D) == 32)
    k_mlp_back1<32><<<cdiv(D, 32) * (H / 32) + H / 16, 256, 0, st>>>(dZ1, X, (int)B, D, H, grad + o.W1, grad + o.b1);
  else
    k_mlp_back1<16><<<cdiv(D, 16) * (H / 16) + H / 16, 256, 0, st>>>(dZ1, X, (int)B, D, H, grad + o.W1, grad + o.b1);
  LAUNCHCHK();
}

void mlp_adam(ffk_mlp* net, const float* grad, float lr, hipStream_t st) {
  net->t += 1;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float c1 = (float)(1.0 - pow((double)b1, (double)net->t));
  const float c2 = (float)(1.0 - pow((double)b2, (double)net->t));
  k_adam<<<cdiv(net->nparam, 256), 256, 0, st>>>(net->theta.as<float>(), grad, net->m.as<float>(), net->v.as<float>(),
                                                  net->nparam, lr, b1, b2, eps, c1, c2);
  LAUNCHCHK();
  net->wbf_valid = false;
}

void mlp_scores(const ffk_mlp* net, const ffk_system* s, double* scores, hipStream_t st) {
  const int D = net->D;
  const Offs o = offs(D, net->H);
  const int64_t N = s->N, Dk = rup(D, 64), Br = rup(N, 128);
  const float* th = net->theta.as<float>();
  DBuf xb(Br * Dk * 2), out(N * 4);
  k_standardize_bf16<<<cdiv(Br * Dk, 256), 256, 0, st>>>(s->X.as<double>(), N, D, th + o.mean, th + o.istd, Br, Dk,
                                                          xb.as<bf16_t>());
  LAUNCHCHK();
  forward_bf16(net, xb.as<bf16_t>(), N, Dk, out.as<float>(), st);
  k_exp_scores<<<cdiv(N, 256), 256, 0, st>>>(out.as<float>(), N, scores);
  LAUNCHCHK();
  HIPCHK(hipStreamSynchronize(st));
}

// ---------------------------------------------------- training-data helpers ----
// X_out (N x D float) = descriptor rows of a system, standardised with the
// network's mean / inverse std when `standardize`.
__global__ void k_prepare(const double* X, int64_t N, int64_t D, const float* mean, const float* istd, int standardize,
                          float* out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N * D) return;
  const int64_t c = e % D;
  out[e] = standardize ? (float)((X[e] - mean[c]) * istd[c]) : (float)X[e];
}

void mlp_prepare_inputs(const ffk_mlp* net, const ffk_system* s, float* out, int standardize, hipStream_t st) {
  const Offs o = offs(net->D, net->H);
  const float* th = net->theta.as<float>();
  k_prepare<<<cdiv(s->N * s->D, 256), 256, 0, st>>>(s->X.as<double>(), s->N, s->D, th + o.mean, th + o.istd,
                                                    standardize, out);
  LAUNCHCHK();
}

// mean and inverse standard deviation of the B rows of X (B x D), per column
__global__ void k_fit_norm(const float* X, int64_t B, int D, float* mean, float* istd) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= D) return;
  double s = 0.0, s2 = 0.0;
  for (int64_t b = 0; b < B; ++b) {
    const double x = X[b * D + c];
    s += x;
    s2 += x * x;
  }
  const double m = s / (double)B;
  const double var = s2 / (double)B - m * m;
  mean[c] = (float)m;
  istd[c] = (float)(1.0 / sqrt(var > 1e-30 ? var : 1e-30));
}

void mlp_fit_norm(ffk_mlp* net, const float* X, int64_t B, hipStream_t st) {
  const Offs o = offs(net->D, net->H);
  float* th = net->theta.as<float>();
  k_fit_norm<<<cdiv(net->D, 128), 128, 0, st>>>(X, B, net->D, th + o.mean, th + o.istd);
  LAUNCHCHK();
}

// y_g = log(sum of the 3M column scores of geometry g) - mean over g
__global__ __launch_bounds__(256) void k_block_log(const double* tau, int64_t N, int m3, float* y) {
  __shared__ double sh[256];
  double acc = 0.0;
  for (int64_t g = threadIdx.x; g < N; g += 256) {
    double s = 0.0;
    for (int c = 0; c < m3; ++c) s += tau[g * m3 + c];
    const double l = log(s > 1e-300 ? s : 1e-300);
    y[g] = (float)l;
    acc += l;
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  const float mu = (float)(sh[0] / (double)N);
  for (int64_t g = threadIdx.x; g < N; g += 256) y[g] -= mu;
}

void block_log_scores(const double* tau, int64_t N, int M, float* y, hipStream_t st) {
  k_block_log<<<1, 256, 0, st>>>(tau, N, 3 * M, y);
  LAUNCHCHK();
}

}  // namespace ffk
