// MFMA GEMM engines for gfx950.
//
// Every engine computes a BM x BN tile of  acc = sum_k A(m, k) B(n, k)  (an
// "A B^T" product); a wave owns a sub-tile made of 16 x 16 MFMA blocks.  Operand
// lane layout (all three instructions): lane l supplies row l%16 and the
// K-slice l/16.  Output lane layout: lane l, register v holds column l%16 and
// row 4*(l/16) + v for the FP32-output instructions, but row 4*v + l/16 for
// v_mfma_f64_16x16x4_f64.
// After the K loop the engine hands the accumulators to an epilogue functor,
// which does all stores (and any fused elementwise work and row reductions).
//
// gemm_row_kernel: FP32 and FP64 products of padded row-major operands (the
//   kernel product, its coefficients, the Gram matrix of the factor).
//
// gemm_dma_kernel: BF16 and split-BF16 products of fragment-major operands.
//
// gemm_scalar_kernel: products of strided views, in double (v_mfma_f64_16x16x4_f64;
//   the stored type may be narrower: the low-memory build, whose factor is held in
//   FP32) or float (v_mfma_f32_16x16x4_f32; the score network's large FP32 layers).
//   One operand element per lane per instruction, so operands may be K-contiguous
//   or M-contiguous; LDS tiles are stored [k][m] with 16 elements of padding per
//   row.  Bounds are checked.  4 waves, 2 x 2.
//
// gemm_bf16_kernel: v_mfma_f32_16x16x32_bf16, FP32 accumulation (the score network).
//   Operands are K-contiguous bf16 arrays whose row count is padded to a multiple of
//   BM (or BN) and whose leading dimension is padded to a multiple of BK with zeros,
//   so tiles are loaded with unpredicated 16-byte vectors.  LDS tiles are [m][k] with
//   8 elements of row padding, which makes the 16-byte operand reads of one 16-lane
//   group hit distinct banks.  4 waves, 2 x 2.
//
// FP64 products of column-major operands are in gemm64.hpp.
#pragma once

#include "common.hpp"

namespace ffk {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma16;
template <> struct Mfma16<double> {
  typedef d4 acc_t;
  __device__ static inline acc_t run(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma16<float> {
  typedef f4 acc_t;
  __device__ static inline acc_t run(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

__device__ inline f4 mfma_bf16(u4 a, u4 b, f4 c) {
  bf8 av = __builtin_bit_cast(bf8, a);
  bf8 bv = __builtin_bit_cast(bf8, b);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c, 0, 0, 0);
}

// Coordinates of accumulator element (tm, tn, v) for this lane, relative to the tile.
struct FragCoord {
  int wm0, wn0, lane;   // absolute origin of this wave's sub-tile
  int m0, n0;           // absolute origin of the block tile
  bool f64;             // FP64 MFMA output layout
  int tn;               // tile column index (n0 / BN)
  int wcol, nwcol;      // this wave's column index among the block's wave columns
  int split;            // K-split index of the block (which partial it writes)
  __device__ inline int row(int tm, int v) const {
    return wm0 + tm * 16 + (f64 ? 4 * v + (lane >> 4) : 4 * (lane >> 4) + v);
  }
  __device__ inline int col(int tn) const { return wn0 + tn * 16 + (lane & 15); }
};

// Operands of the strided GEMM: element (m, k) at p[m*s0 + k*s1].  The
// stored type TI may be narrower than the compute type (float -> double is exact).
template <typename TI> struct SegS {
  const TI* A; int64_t sa0, sa1;
  const TI* B; int64_t sb0, sb1;
  int K;
};

template <typename TI> struct ScalarArgs {
  int M, N;
  SegS<TI> seg;
};

// ---------------------------------------------------------------------------
// Strided-operand MFMA engine (FP64 or FP32 arithmetic)
// ---------------------------------------------------------------------------
template <typename T, int BM, int BN, int BK, bool AKC, bool BKC, class Epi, typename TI = T>
__global__ __launch_bounds__(256) void gemm_scalar_kernel(ScalarArgs<TI> g, Epi epi) {
  constexpr int PAD = 16;
  constexpr int EA = BM * BK / 256;
  constexpr int EB = BN * BK / 256;
  constexpr int TM = BM / 32;   // 16x16 blocks per wave along M
  constexpr int TN = BN / 32;
  typedef typename Mfma16<T>::acc_t acc_t;
  __shared__ T As[2][BK][BM + PAD];
  __shared__ T Bs[2][BK][BN + PAD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * (BN / 2);
  const SegS<TI>& s = g.seg;
  const int T_ = (s.K + BK - 1) / BK;

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

  T ra[EA], rb[EB];
  auto load = [&](int t) {
    const int k0 = t * BK;
#pragma unroll
    for (int i = 0; i < EA; ++i) {
      const int e = tid + 256 * i;
      const int mm = AKC ? e / BK : e % BM;
      const int kk = AKC ? e % BK : e / BM;
      const int m = m0 + mm, k = k0 + kk;
      ra[i] = (m < g.M && k < s.K) ? (T)(s.A[(int64_t)m * s.sa0 + (int64_t)k * s.sa1]) : T(0);
    }
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int e = tid + 256 * i;
      const int nn = BKC ? e / BK : e % BN;
      const int kk = BKC ? e % BK : e / BN;
      const int n = n0 + nn, k = k0 + kk;
      rb[i] = (n < g.N && k < s.K) ? (T)(s.B[(int64_t)n * s.sb0 + (int64_t)k * s.sb1]) : T(0);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < EA; ++i) {
      const int e = tid + 256 * i;
      const int mm = AKC ? e / BK : e % BM;
      const int kk = AKC ? e % BK : e / BM;
      As[buf][kk][mm] = ra[i];
    }
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int e = tid + 256 * i;
      const int nn = BKC ? e / BK : e % BN;
      const int kk = BKC ? e % BK : e / BN;
      Bs[buf][kk][nn] = rb[i];
    }
  };

  if (T_ > 0) {
    load(0);
    store(0);
  }
  __syncthreads();
  for (int t = 0; t < T_; ++t) {
    const int buf = t & 1;
    if (t + 1 < T_) load(t + 1);
#pragma unroll
    for (int k4 = 0; k4 < BK / 4; ++k4) {
      T a[TM], b[TN];
      const int kr = k4 * 4 + (lane >> 4);
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = As[buf][kr][wm0 + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = Bs[buf][kr][wn0 + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = Mfma16<T>::run(a[i], b[j], acc[i][j]);
    }
    if (t + 1 < T_) store(buf ^ 1);
    __syncthreads();
  }
  FragCoord fc{m0 + wm0, n0 + wn0, lane, m0, n0, sizeof(T) == 8, (int)blockIdx.x, wave & 1, 2, 0};
  epi.template run<T, TM, TN>(acc, fc, reinterpret_cast<char*>(&As[0][0][0]));
}

// ---------------------------------------------------------------------------
// BF16 MFMA engine
// ---------------------------------------------------------------------------
struct Bf16Args {
  const bf16_t *A, *B;     // rows padded to a BM (BN) multiple, ld a multiple of BK
  int64_t lda, ldb;
  int K;                   // multiple of BK (padded)
};

template <int BM, int BN, int BK, class Epi>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(Bf16Args g, Epi epi) {
  constexpr int PAD = 8;
  constexpr int LDS_ROW = BK + PAD;
  constexpr int VA = BM * BK / 8 / 256;   // 16-byte vectors per thread
  constexpr int VB = BN * BK / 8 / 256;
  constexpr int TM = BM / 32, TN = BN / 32;
  __shared__ bf16_t As[BM * LDS_ROW];
  __shared__ bf16_t Bs[BN * LDS_ROW];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * (BN / 2);
  const int T_ = g.K / BK;

  f4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f4{0, 0, 0, 0};

  u4 ra[VA], rb[VB];
  auto load = [&](int t) {
    const int k0 = t * BK;
#pragma unroll
    for (int i = 0; i < VA; ++i) {
      const int e = tid + 256 * i;
      const int mm = e / (BK / 8), kv = e % (BK / 8);
      ra[i] = *reinterpret_cast<const u4*>(g.A + (int64_t)(m0 + mm) * g.lda + k0 + kv * 8);
    }
#pragma unroll
    for (int i = 0; i < VB; ++i) {
      const int e = tid + 256 * i;
      const int nn = e / (BK / 8), kv = e % (BK / 8);
      rb[i] = *reinterpret_cast<const u4*>(g.B + (int64_t)(n0 + nn) * g.ldb + k0 + kv * 8);
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int i = 0; i < VA; ++i) {
      const int e = tid + 256 * i;
      const int mm = e / (BK / 8), kv = e % (BK / 8);
      *reinterpret_cast<u4*>(&As[mm * LDS_ROW + kv * 8]) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < VB; ++i) {
      const int e = tid + 256 * i;
      const int nn = e / (BK / 8), kv = e % (BK / 8);
      *reinterpret_cast<u4*>(&Bs[nn * LDS_ROW + kv * 8]) = rb[i];
    }
  };

  if (T_ > 0) {
    load(0);
    store();
  }
  __syncthreads();
  for (int t = 0; t < T_; ++t) {
    if (t + 1 < T_) load(t + 1);
#pragma unroll
    for (int kk = 0; kk < BK / 32; ++kk) {
      const int ko = kk * 32 + 8 * (lane >> 4);
      u4 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        a[i] = *reinterpret_cast<const u4*>(&As[(wm0 + i * 16 + (lane & 15)) * LDS_ROW + ko]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        b[j] = *reinterpret_cast<const u4*>(&Bs[(wn0 + j * 16 + (lane & 15)) * LDS_ROW + ko]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma_bf16(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
    if (t + 1 < T_) {
      store();
      __syncthreads();
    }
  }
  FragCoord fc{m0 + wm0, n0 + wn0, lane, m0, n0, false, (int)blockIdx.x, wave & 1, 2, 0};
  epi.template run<float, TM, TN>(acc, fc, reinterpret_cast<char*>(&As[0]));
}

// ---------------------------------------------------------------------------
// BF16 MFMA engine, pipelined through direct global->LDS loads (gfx950
// global_load_lds_dwordx4).  Each wave-wide load moves 64 x 16 bytes into 1 KB
// of LDS at base + lane*16, so a 16-row x 32-k operand block is fetched with
// lane L taking row L%16 and 16-byte chunk L/16: exactly the lane layout the
// 16x16x32 MFMA reads, hence every ds_read_b128 of an operand fragment is a
// contiguous, conflict-free 1 KB read and no staging registers are needed.
// S stages of BK = 32 keep S-1 tiles in flight behind the MFMAs.
// ---------------------------------------------------------------------------
// gfx9 s_waitcnt immediate for vmcnt(N): low bits [3:0], high bits [15:14];
// expcnt and lgkmcnt left at "no wait".
template <int N> struct VmCnt {
  static constexpr unsigned v = (unsigned)((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
};

__device__ inline void dma16(const void* g, void* lds_base) {
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)g,
                                   (void __attribute__((address_space(3)))*)lds_base, 16, 0, 0);
}

// XCD-aware tile order.  Workgroup w of the grid (x fastest, then y, then z)
// runs on XCD w % 8 as that XCD's (w / 8)-th.  ALL: each XCD gets a
// contiguous range of all (K split, tile) items, whatever their count (the
// tiles of one row of a 79 x 7 grid had gone to seven L2s: split BF16 at M =
// 60, N = 20000, GEMM 1 3.78 -> 3.66 ms and GEMM 2 6.09 -> 5.94 ms; 6% at M =
// 42, N = 5000).  Otherwise the split is blockIdx.z and the tiles of a split
// are remapped only when their count is a multiple of 8 (the FP32 GEMM 2 on
// 128 x 128 tiles, 14 x 158 x splits, measured 17% slower with the general
// remap).  Within a split, tiles are grouped by 8 tile rows, so tiles that
// run together on an XCD share operand rows in its L2.
template <bool ALL>
__device__ inline void tile_coords(int& tm, int& tn, int& tz) {
  const int nt_n = gridDim.x, nt_m = gridDim.y;
  const int T = nt_m * nt_n;
  int lin;
  if constexpr (ALL) {
    const int W = T * (int)gridDim.z;
    const int w = ((int)blockIdx.z * nt_m + (int)blockIdx.y) * nt_n + (int)blockIdx.x;
    const int xcd = w % 8, idx = w / 8, q = W / 8, r = W % 8;
    const int L = (xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q) + idx;
    tz = L / T;
    lin = L % T;
  } else {
    tz = (int)blockIdx.z;
    lin = (int)blockIdx.y * nt_n + (int)blockIdx.x;
    if (T % 8 == 0) lin = (lin % 8) * (T / 8) + lin / 8;
  }
  const int G = 8;
  const int per_group = G * nt_n;
  const int grp = lin / per_group;
  const int first = grp * G;
  const int gsz = min(nt_m - first, G);
  const int in = lin % per_group;
  tm = first + in % gsz;
  tn = in / gsz;
}

// Per element type: what one pair of 16-byte operand fragments (one 64-byte
// K chunk of a 16-row group per lane group) feeds to the matrix cores.
//   bf16:   8 elements, one v_mfma_f32_16x16x32_bf16
//   float:  4 elements, four v_mfma_f32_16x16x4_f32 (instruction j takes
//           element j of every lane: K slot l/16 of instruction j is k = 4(l/16)+j)
//   double: 2 elements, two v_mfma_f64_16x16x4_f64 (k = 2(l/16)+j)
// Every K index is consumed exactly once by A and B alike, so the sum is the
// full dot product whatever the order.
template <typename T> struct DmaMfma;
template <> struct DmaMfma<bf16_t> {
  typedef f4 acc_t;
  typedef float scalar_t;
  static constexpr int SLICES = 1;
  __device__ static inline acc_t slice(const u4& a, const u4& b, acc_t c, int) { return mfma_bf16(a, b, c); }
};
template <> struct DmaMfma<float> {
  typedef f4 acc_t;
  typedef float scalar_t;
  static constexpr int SLICES = 4;
  __device__ static inline acc_t slice(const u4& a, const u4& b, acc_t c, int j) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[j]), __uint_as_float(b[j]), c, 0, 0, 0);
  }
};
template <> struct DmaMfma<double> {
  typedef d4 acc_t;
  typedef double scalar_t;
  static constexpr int SLICES = 2;
  __device__ static inline acc_t slice(const u4& a, const u4& b, acc_t c, int j) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(__hiloint2double((int)a[2 * j + 1], (int)a[2 * j]),
                                                 __hiloint2double((int)b[2 * j + 1], (int)b[2 * j]), c, 0, 0, 0);
  }
};

// Operand segment of the pipelined engines: K-contiguous arrays of T whose row
// count is padded to the tile and whose leading dimension (in elements) and K
// are multiples of 64 bytes; padding is zero.  BF16 operands are in the
// fragment-major layout (frag_off) with KT K tiles to a row group and ignore
// lda/ldb.  K may be less than what is stored: K tiles that are all padding are
// left out.  The lo arrays are used only in the split-BF16 mode.
struct SegD {
  const void *Ah, *Al;
  const void *Bh, *Bl;
  int64_t lda, ldb;   // elements
  int K;              // elements, multiple of 64 bytes
  int KT;             // BF16: K tiles of a stored row group
};
// Items of a Gram product: K in `ranges` ranges, workgroup w on range w %
// ranges (eight: one per XCD, whose L2 then holds the window of the operand that
// its tiles walk through together) as that range's item w / ranges: the first
// `whole` lower tiles in one piece each, the others in `parts`.
struct GramMap {
  int ranges, whole, parts;
};
struct DmaArgs {
  int nseg;
  SegD seg[2];
  int lower_only;   // gemm_row_kernel: square tiles strictly above the diagonal do nothing (symmetric products)
  GramMap gram;
};

// Tile shape of the pipelined engine: BM x BN block tile computed by WM x WN
// waves (each (BM/WM) x (BN/WN)), S pipeline stages.
template <int BM_, int BN_, int WM_, int WN_, int S_, bool HH_ = false>
struct DmaTile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, S = S_;
  static constexpr bool HH = HH_;   // split BF16: hi*hi, hi*lo, lo*hi, the order of large wave tiles, not the reverse
  static constexpr int NT = 64 * WM * WN;
};

template <typename T, class TL, bool X3, class Epi>
__global__ __launch_bounds__(TL::NT) void gemm_dma_kernel(DmaArgs g, Epi epi) {
  static_assert(sizeof(T) == 2, "bf16 operands (FP32 and FP64: gemm_row_kernel)");
  constexpr int BM = TL::BM, BN = TL::BN, WM = TL::WM, WN = TL::WN, S = TL::S, NW = WM * WN;
  constexpr int BK = 64 / (int)sizeof(T);               // one 64-byte chunk of each row per K tile
  constexpr int NARR = X3 ? 2 : 1;
  constexpr int GROUP_BYTES = 1024;                     // 16 rows x 64 bytes
  constexpr int GA = BM / 16, GB = BN / 16;             // row groups per operand tile
  static_assert(GA % NW == 0 && GB % NW == 0, "row groups must split evenly over the waves");
  constexpr int A_BYTES = GA * GROUP_BYTES;
  constexpr int B_BYTES = GB * GROUP_BYTES;
  constexpr int STAGE_BYTES = NARR * (A_BYTES + B_BYTES);
  constexpr int QA = GA / NW, QB = GB / NW;             // groups loaded per wave
  constexpr int LPT = NARR * (QA + QB);                 // wave-wide loads per tile per wave
  static_assert(LPT * (S > 2 ? S - 2 : 0) < 64, "vmcnt holds at most 63 loads in flight");
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;   // 16x16 blocks per wave
  typedef typename DmaMfma<T>::acc_t acc_t;
  __shared__ __attribute__((aligned(1024))) char smem[S * STAGE_BYTES];

  // the wave index in a scalar register, so every operand address is a scalar
  // base plus the lane's offset (228 rather than 252 VGPRs on the split 256 x
  // 256 tile)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tmi, tni, tzi;
  // the 64 x 128 tiles of up to 32 row tiles over the whole grid too: an XCD's 32
  // CUs then hold about one K split, both column tiles of a row beside each
  // other, and read its rows of B from their L2.  M = 21, N = 2000 56.8 -> 55.2
  // us a split-BF16 product (systems in turn), 45.0 -> 43.9 in single BF16; N =
  // 300 26.9 -> 25.9.  With more row tiles it is slower (BF16 N = 4000 90.8 -> 94.6),
  // and on the 128 x 128 tile (M = 60, N = 2000 122 -> 128).
  if constexpr (X3 && TM * TN >= 32) {
    tile_coords<true>(tmi, tni, tzi);
  } else if constexpr (BM == 64 && BN == 128) {
    if (gridDim.y <= 32) tile_coords<true>(tmi, tni, tzi);
    else tile_coords<false>(tmi, tni, tzi);
  } else {
    tile_coords<false>(tmi, tni, tzi);
  }
  const int m0 = tmi * BM, n0 = tni * BN;
  const int wm = wave / WN, wn = wave % WN;
  const int t0 = g.seg[0].K / BK;
  const int T_ = t0 + (g.nseg > 1 ? g.seg[1].K / BK : 0);
  const int tb = (int)((int64_t)T_ * tzi / gridDim.z);
  const int te = (int)((int64_t)T_ * (tzi + 1) / gridDim.z);

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

  // fragment-major operands (frag_off): the 1 KB block of a (row group, K
  // tile) is contiguous, lane L takes bytes 16 L .. 16 L + 15, and whole cache
  // lines move per load.  KT: the K tiles of a stored row group, of which the
  // product may take fewer.
  auto issue = [&](int t) {
    const SegD& sg = (t < t0) ? g.seg[0] : g.seg[1];
    const int64_t tk = (t < t0 ? t : t - t0);
    const int64_t KT = sg.KT;
    char* st = smem + (t % S) * STAGE_BYTES;
#pragma unroll
    for (int h = 0; h < NARR; ++h) {
      const T* A = static_cast<const T*>(h ? sg.Al : sg.Ah);
      const T* B = static_cast<const T*>(h ? sg.Bl : sg.Bh);
#pragma unroll
      for (int q = 0; q < QA; ++q) {
        const int grp = wave * QA + q;
        dma16(A + (((int64_t)(m0 / 16 + grp) * KT + tk) * 512 + lane * 8), st + h * A_BYTES + grp * GROUP_BYTES);
      }
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int grp = wave * QB + q;
        dma16(B + (((int64_t)(n0 / 16 + grp) * KT + tk) * 512 + lane * 8),
              st + NARR * A_BYTES + h * B_BYTES + grp * GROUP_BYTES);
      }
    }
  };

#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (tb + s < te) issue(tb + s);
  for (int t = tb; t < te; ++t) {
    // this wave's loads of tile t have landed; the barrier (without the
    // memory fence of __syncthreads, which would drain every load in flight)
    // makes that true for all waves and frees the stage written next
    if (S > 2 && t + S - 2 < te) __builtin_amdgcn_s_waitcnt(VmCnt<LPT * (S > 2 ? S - 2 : 0)>::v);
    else __builtin_amdgcn_s_waitcnt(VmCnt<0>::v);
    asm volatile("s_barrier" ::: "memory");
    if (t + S - 1 < te) issue(t + S - 1);
    const char* st = smem + (t % S) * STAGE_BYTES;
    u4 ah[TM], bh[TN], al[X3 ? TM : 1], bl[X3 ? TN : 1];
    if constexpr (X3 && TM * TN >= 32) {
      // split BF16 on large wave tiles: the hi fragments, then the hi*hi
      // products with the lo fragment reads slotted between them (two MFMAs,
      // one LDS read), so the lo reads run while the matrix cores work.  At
      // M = 60, N = 20000 on 256 x 256 tiles: GEMM 2 6.45 -> 6.22 ms, GEMM 1
      // 4.01 -> 3.89 ms; issuing the lo reads right after the hi ones (one
      // wait for all) gained nothing.
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bh[j] = *reinterpret_cast<const u4*>(st + NARR * A_BYTES + (wn * TN + j) * GROUP_BYTES + lane * 16);
#pragma unroll
      for (int i = 0; i < TM; ++i) ah[i] = *reinterpret_cast<const u4*>(st + (wm * TM + i) * GROUP_BYTES + lane * 16);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = DmaMfma<T>::slice(ah[i], bh[j], acc[i][j], 0);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bl[j] = *reinterpret_cast<const u4*>(st + NARR * A_BYTES + B_BYTES + (wn * TN + j) * GROUP_BYTES + lane * 16);
#pragma unroll
      for (int i = 0; i < TM; ++i)
        al[i] = *reinterpret_cast<const u4*>(st + A_BYTES + (wm * TM + i) * GROUP_BYTES + lane * 16);
#pragma unroll
      for (int g = 0; g < TM + TN; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // two MFMAs
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
      }
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - 2 * (TM + TN), 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = DmaMfma<T>::slice(ah[i], bl[j], acc[i][j], 0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = DmaMfma<T>::slice(al[i], bh[j], acc[i][j], 0);
      continue;
    }

#pragma unroll
    for (int i = 0; i < TM; ++i) {
      ah[i] = *reinterpret_cast<const u4*>(st + (wm * TM + i) * GROUP_BYTES + lane * 16);
      if (X3) al[X3 ? i : 0] = *reinterpret_cast<const u4*>(st + A_BYTES + (wm * TM + i) * GROUP_BYTES + lane * 16);
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      bh[j] = *reinterpret_cast<const u4*>(st + NARR * A_BYTES + (wn * TN + j) * GROUP_BYTES + lane * 16);
      if (X3) bl[X3 ? j : 0] = *reinterpret_cast<const u4*>(st + NARR * A_BYTES + B_BYTES + (wn * TN + j) * GROUP_BYTES + lane * 16);
    }
    // all fragment reads are issued before the first MFMA: left to itself the
    // scheduler interleaves them in pairs, each behind a full LDS-latency wait
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (X3 && TL::HH) {
          acc[i][j] = DmaMfma<T>::slice(ah[i], bh[j], acc[i][j], 0);
          acc[i][j] = DmaMfma<T>::slice(ah[i], bl[j], acc[i][j], 0);
          acc[i][j] = DmaMfma<T>::slice(al[i], bh[j], acc[i][j], 0);
          continue;
        }
        if (X3) {
          acc[i][j] = DmaMfma<T>::slice(al[X3 ? i : 0], bh[j], acc[i][j], 0);
          acc[i][j] = DmaMfma<T>::slice(ah[i], bl[X3 ? j : 0], acc[i][j], 0);
        }
        acc[i][j] = DmaMfma<T>::slice(ah[i], bh[j], acc[i][j], 0);
      }
  }
  __syncthreads();
  FragCoord fc{m0 + wm * (BM / WM), n0 + wn * (BN / WN), lane, m0, n0, sizeof(T) == 8, tni, wn, WN, tzi};
  epi.template run<typename DmaMfma<T>::scalar_t, TM, TN>(acc, fc, smem);
}

// ---------------------------------------------------------------------------
// FP32 and FP64 MFMA engine for row-major (K-contiguous) operands, the same
// direct global->LDS loads: a wave load takes 16 rows x 64 bytes, lane L row
// L % 16 and 16-byte chunk L / 16, the lane layout of the fragments.
// Bound by the matrix cores.  A stage holds two chunks of 64 bytes of K, two
// stages: a wave meets a barrier every 64 (FP64) or 128 (FP32) MFMAs of a 64 x
// 32 tile, and the 128 x 128 tile by eight waves leaves room for two
// workgroups, 16 waves, on a CU (at most 128 registers: hence the bound of four
// waves a SIMD).  Fragments are double-buffered in registers; read right before
// their MFMAs, the waves of both workgroups met in the same phase and the
// matrix cores idled 30% of the time.  K order within an element's sum does not
// depend on the tile shape.  Four waves of 64 x 64 with a barrier per chunk and
// four stages, eight waves with two chunks, and now: the FP64 product at M =
// 42, N = 5000 4.18, 2.86, 2.42 ms (53 TFLOP/s; matrix cores busy 77% of GEMM
// 2); FP32 at M = 21, N = 10000 1.72, 1.54, 1.55 ms; the Gram matrix of the
// factor at n = 126000, k = 2000 18.4, 11.5, 10.3 ms (8.5 in GramMap's items).
// BN need not be a power of two: the column tiles can fit the operand's width.
// ---------------------------------------------------------------------------
template <int BM_, int BN_, int WM_, int WN_, int KS_>
struct RowTile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KS = KS_;
  static constexpr int NT = 64 * WM * WN;
};

// GRAM: the lower tiles of a symmetric product in the items of GramMap.
// Otherwise the order of tile_coords<false>.
template <typename T, class TL, class Epi, bool GRAM = false>
__global__ __launch_bounds__(TL::NT, TL::NT == 512 ? 4 : 1) void gemm_row_kernel(DmaArgs g, Epi epi) {
  static_assert(sizeof(T) >= 4, "FP32 or FP64 operands");
  constexpr int BM = TL::BM, BN = TL::BN, WM = TL::WM, WN = TL::WN, KS = TL::KS, NW = WM * WN;
  constexpr int BK = 64 / (int)sizeof(T);
  constexpr int GA = BM / 16, GB = BN / 16, CHUNK = (GA + GB) * 1024;
  constexpr int QA = (KS * GA + NW - 1) / NW, QB = (KS * GB + NW - 1) / NW;   // 1 KB loads of a wave per stage
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  static_assert(TM * WM * 16 == BM && TN * WN * 16 == BN, "16 x 16 blocks per wave");
  static_assert(KS == 2, "the fragments of a stage's chunks alternate between two sets");
  typedef typename DmaMfma<T>::acc_t acc_t;
  __shared__ __attribute__((aligned(1024))) char smem[2 * KS * CHUNK];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tmi, tni, tzi;
  int part = 0, parts = 1;
  if constexpr (GRAM) {
    const int x = (int)blockIdx.x % g.gram.ranges, j = (int)blockIdx.x / g.gram.ranges, rest = j - g.gram.whole;
    const int t = rest < 0 ? j : g.gram.whole + rest / g.gram.parts;
    tmi = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((tmi + 1) * (tmi + 2) / 2 <= t) ++tmi;
    while (tmi * (tmi + 1) / 2 > t) --tmi;
    tni = t - tmi * (tmi + 1) / 2;
    tzi = x * (int)(gridDim.x / g.gram.ranges) + j;
    part = rest < 0 ? x : x * g.gram.parts + rest % g.gram.parts;
    parts = rest < 0 ? g.gram.ranges : g.gram.ranges * g.gram.parts;
  } else {
    tile_coords<false>(tmi, tni, tzi);
    part = tzi;
    parts = (int)gridDim.z;
  }
  if (g.lower_only && tni > tmi) return;
  const int m0 = tmi * BM, n0 = tni * BN;
  const int wm = wave / WN, wn = wave % WN;
  const int t0 = g.seg[0].K / BK;
  const int T_ = t0 + (g.nseg > 1 ? g.seg[1].K / BK : 0);
  const int tb = (int)((int64_t)T_ * part / parts);
  const int te = (int)((int64_t)T_ * (part + 1) / parts);

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

  // wave w takes the loads w, w + NW, ... of a stage of each operand; the
  // second segment has the first's leading dimensions and lies at a distance
  const char *pa[QA], *pb[QB];
#pragma unroll
  for (int q = 0; q < QA; ++q)
    pa[q] = static_cast<const char*>(g.seg[0].Ah) +
            (m0 + (wave + q * NW) % GA * 16 + (lane & 15)) * g.seg[0].lda * (int64_t)sizeof(T) + (lane >> 4) * 16;
#pragma unroll
  for (int q = 0; q < QB; ++q)
    pb[q] = static_cast<const char*>(g.seg[0].Bh) +
            (n0 + (wave + q * NW) % GB * 16 + (lane & 15)) * g.seg[0].ldb * (int64_t)sizeof(T) + (lane >> 4) * 16;
  const int64_t da = (int64_t)((uintptr_t)g.seg[1].Ah - (uintptr_t)g.seg[0].Ah) - (int64_t)t0 * 64;
  const int64_t db = (int64_t)((uintptr_t)g.seg[1].Bh - (uintptr_t)g.seg[0].Bh) - (int64_t)t0 * 64;
  auto issue = [&](int s) {   // stage s: chunks tb + s KS ..
    char* st = smem + (s & 1) * KS * CHUNK;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int idx = wave + q * NW, kc = idx / GA, t = tb + s * KS + kc;
      if (idx < KS * GA && t < te) dma16(pa[q] + ((int64_t)t * 64 + (t < t0 ? 0 : da)), st + kc * CHUNK + idx % GA * 1024);
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int idx = wave + q * NW, kc = idx / GB, t = tb + s * KS + kc;
      if (idx < KS * GB && t < te) dma16(pb[q] + ((int64_t)t * 64 + (t < t0 ? 0 : db)), st + kc * CHUNK + (GA + idx % GB) * 1024);
    }
  };
  struct Frag { u4 a[TM], b[TN]; };
  auto read = [&](int s, int kc, Frag& f) {
    const char* st = smem + (s & 1) * KS * CHUNK + kc * CHUNK;
#pragma unroll
    for (int i = 0; i < TM; ++i) f.a[i] = *reinterpret_cast<const u4*>(st + (wm * TM + i) * 1024 + lane * 16);
#pragma unroll
    for (int j = 0; j < TN; ++j) f.b[j] = *reinterpret_cast<const u4*>(st + (GA + wn * TN + j) * 1024 + lane * 16);
  };
  auto mul = [&](const Frag& f) {
    // the reads of the next fragments stay before these MFMAs
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int sl = 0; sl < DmaMfma<T>::SLICES; ++sl)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = DmaMfma<T>::slice(f.a[i], f.b[j], acc[i][j], sl);
    __builtin_amdgcn_sched_barrier(0);
  };

  // Software pipeline: a chunk's fragments are read while the MFMAs of the one
  // before it run.  At a stage's last chunk the wave has its fragments in
  // registers; past the barrier every wave has, so the next stage's data is
  // complete and this stage's buffer free for the one after it.  The last
  // stage may lack its second chunk: it is read (whatever the LDS holds) but
  // not multiplied.
  const int n = te - tb, ns = (n + KS - 1) / KS;
  if (ns > 0) issue(0);
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  if (ns > 1) issue(1);
  Frag f0, f1;
  if (ns > 0) read(0, 0, f0);
  for (int s = 0; s < ns; ++s) {
    read(s, 1, f1);
    mul(f0);
    if (s + 1 < ns) {
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (s + 2 < ns) issue(s + 2);
      read(s + 1, 0, f0);
    }
    if (2 * s + 1 < n) mul(f1);
  }
  __syncthreads();
  FragCoord fc{m0 + wm * (BM / WM), n0 + wn * (BN / WN), lane, m0, n0, sizeof(T) == 8, tni, wn, WN, tzi};
  epi.template run<typename DmaMfma<T>::scalar_t, TM, TN>(acc, fc, smem);
}

// Shared LDS for epilogues that need it: the engines pass their operand LDS
// after the final barrier of the K loop.

// ---------------------------------------------------------------------------
// Generic epilogue: C(m, n) = alpha * acc + beta * C(m, n) on a strided view.
// ---------------------------------------------------------------------------
template <typename CT> struct EpiAxpby {
  CT* C;
  int64_t scm, scn;
  int M, N;
  double alpha, beta;
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
            CT* p = C + (int64_t)r * scm + (int64_t)c * scn;
            const double val = alpha * (double)acc[i][j][v];
            *p = (CT)(beta == 0.0 ? val : val + beta * (double)*p);
          }
        }
  }
};

// Split-K partial store: part[(z * rows + r) * ldp + c] = acc for r < rows, c < cols.
template <typename PT> struct EpiPart {
  PT* part;
  int64_t ldp;
  int rows, cols;
  template <typename T, int TM, int TN, class Acc>
  __device__ void run(const Acc (&acc)[TM][TN], const FragCoord& f, char*) const {
    PT* base = part + (int64_t)f.split * rows * ldp;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = f.row(i, v), c = f.col(j);
          if (r < rows && c < cols) base[(int64_t)r * ldp + c] = (PT)acc[i][j][v];
        }
  }
};

// The tile as the registers hold it, one after the other by split index: a
// wave's store is 512 contiguous bytes.
template <int BM, int BN> struct EpiTile {
  double* part;
  template <typename T, int TM, int TN, class Acc>
  __device__ void run(const Acc (&acc)[TM][TN], const FragCoord& f, char*) const {
    const int wave = ((f.wm0 - f.m0) / (16 * TM)) * f.nwcol + f.wcol;
    double* base = part + (int64_t)f.split * BM * BN + (int64_t)wave * TM * TN * 256 + f.lane;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) base[((i * TN + j) * 4 + v) * 64] = acc[i][j][v];
  }
};

// Number of K splits that brings a GEMM with `tiles` output tiles to >=
// `target` workgroups while keeping at least two K tiles per split.
inline int pick_splits(int64_t tiles, int64_t ktiles, int64_t target = 512) {
  int s = 1;
  while (tiles * s < target && (int64_t)s * 4 <= ktiles) s *= 2;
  return s;
}

}  // namespace ffk
