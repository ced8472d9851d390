// Single kernel columns K[:, c] and the diagonal diag(K) -- the get_col(i) and
// d := diag(K) inputs of the incomplete Cholesky (appendix, Algorithm 1).
//
// Column c = 3 M g + 3 p + t belongs to source geometry g, atom p, coordinate t.
// Its descriptor image u = J_g e_c is non-zero only on the M-1 pairs {p, b}:
//   u_{pb} = -(R_gp - R_gb)_t / r_gpb^3.
// For each target geometry i, with d = x_i - x_g and (a, b) the Matern-5/2
// Hessian coefficients at r = |d|,
//   K[i-block, c] = J_i^T (a u + b (d . u) d) = a J_i^T u + b (d . u) J_i^T d,
// where (J_i^T h)_q = -sum_{b != q} h_{qb} (R_iq - R_ib) / r_iqb^3.
// A wave handles one target and 64 columns, one per lane, so that everything
// that belongs to the target is uniform: its pair vectors (R_ia - R_ib)/r^3
// and distances come from the system's pair table, sixteen pairs to a register
// (the same in each row of 16 lanes), and reach the arithmetic as the DPP operand
// of the FMA itself.  A pair costs a lane one LDS read (x_g of its column) and four
// FMAs.  A block is four targets of the same 64 columns, which share the staging
// of the columns' x_g rows, in tiles of 8 x 8 atoms.
// Bound by the LDS reads and that arithmetic.  256 columns at M = 21, N = 2000:
// 786 us with one wave per (target, column), lanes over the M atoms, two thirds
// of them idle; 488 with scalar loads, for which there are too few scalar
// registers; 345 with a pair to a lane and two readlanes a value; now 302.
#include "common.hpp"

namespace ffk {

__device__ inline int pair_of(int a, int b) { return a > b ? a * (a - 1) / 2 + b : b * (b - 1) / 2 + a; }

constexpr int kColTile = 64;   // columns per block, one per lane
constexpr int kColWaves = 4;   // targets per block
constexpr int kAtoms = 8;      // atoms per tile side
constexpr int kXStride = kColTile + 1;

static size_t columns_lds(int M) { return (size_t)(kColTile * kXStride + 2 * M * kColTile) * sizeof(double); }

// d_j += w_d (of lane L_j of each row of 16), then v += w d_j: four pairs, of which
// the first two have their vectors in A and the others in B (x, y, z, d).  By
// hand, as the compiler broadcasts with a move of its own; a value that the
// vector unit has just written may not be a DPP operand for two cycles.
template <int L0, int L1, int L2, int L3>
__device__ inline void four_pairs(double (&d)[4], double& vx, double& vy, double& vz, const double (&A)[4],
                                  const double (&B)[4], double one) {
#define FFK_PAIR(D, W, L)                                                       \
  "v_fmac_f64_dpp %[" D "], %[" W "3], %[one] row_newbcast:%[" L "] row_mask:0xf bank_mask:0xf\n\t"    \
  "v_fmac_f64_dpp %[vx], %[" W "0], %[" D "] row_newbcast:%[" L "] row_mask:0xf bank_mask:0xf\n\t"     \
  "v_fmac_f64_dpp %[vy], %[" W "1], %[" D "] row_newbcast:%[" L "] row_mask:0xf bank_mask:0xf\n\t"     \
  "v_fmac_f64_dpp %[vz], %[" W "2], %[" D "] row_newbcast:%[" L "] row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" FFK_PAIR("d0", "a", "l0") FFK_PAIR("d1", "a", "l1") FFK_PAIR("d2", "b", "l2")
          FFK_PAIR("d3", "b", "l3")
      : [d0] "+v"(d[0]), [d1] "+v"(d[1]), [d2] "+v"(d[2]), [d3] "+v"(d[3]), [vx] "+v"(vx), [vy] "+v"(vy), [vz] "+v"(vz)
      : [a0] "v"(A[0]), [a1] "v"(A[1]), [a2] "v"(A[2]), [a3] "v"(A[3]), [b0] "v"(B[0]), [b1] "v"(B[1]),
        [b2] "v"(B[2]), [b3] "v"(B[3]), [one] "v"(one), [l0] "n"(L0), [l1] "n"(L1), [l2] "n"(L2), [l3] "n"(L3));
#undef FFK_PAIR
}
// d_j += w of lane L + j of each row of 16.
template <int L> __device__ inline void four_differences(double (&d)[4], double w, double one) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
      : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3])
      : "v"(w), "v"(one), "n"(L), "n"(L + 1), "n"(L + 2), "n"(L + 3));
}

// Targets (rows) come from PT, X; the source geometry of each column from PTs,
// Xs (the same arrays for a plain kernel, a permuted copy for a symmetrized
// one).  PT: the pair table, four doubles per (geometry, pair a > b): (R_a -
// R_b) / r^3 and 1 / r.  With accumulate the values are added to out.
// LDS: xs[64][65] (-x_g of a tile's pairs; then the outputs on their way out),
// U[M][64] (u on the pairs {p, b} of each column), XP[M][64] (x_g there).
__global__ __launch_bounds__(64 * kColWaves) void k_columns(
    const double* __restrict__ PT, const double* __restrict__ X, const double* __restrict__ PTs,
    const double* __restrict__ Xs, int64_t N, int M, int64_t D, const int64_t* __restrict__ cols, int64_t k,
    double* __restrict__ out, int64_t ldo, double shift, double inv_len, double a0, double bcoef, int accumulate) {
  extern __shared__ double sm[];
  double* xs = sm;
  double* U = xs + kColTile * kXStride;
  double* XP = U + M * kColTile;
  __shared__ int64_t sg_of[kColTile];   // first element of the source's row of X
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m3 = 3 * M;
  const int64_t c0 = (int64_t)blockIdx.y * kColTile;
  // columns past the end and targets past the end repeat the last one and
  // store nothing
  const int64_t cidx = min(c0 + lane, k - 1);
  const int64_t col = cols[cidx];
  const int64_t g = col / m3;
  const int loc = (int)(col % m3), p = loc / 3, t = loc % 3;
  const int64_t i_raw = (int64_t)blockIdx.x * kColWaves + wave;
  const int64_t i = min(i_raw, N - 1);
  const double* Pi = PT + i * D * 4;
  const double* Xi = X + i * D;
  if (tid < kColTile) sg_of[tid] = g * D;
#pragma unroll 4
  for (int b = wave; b < M; b += kColWaves) {   // u_{pb} = -(R_gp - R_gb)_t / r^3
    const double* w = PTs + (g * D + (b != p ? pair_of(p, b) : 0)) * 4;
    const double wt = w[t], x = w[3];
    U[b * kColTile + lane] = b == p ? 0.0 : (p > b ? -wt : wt);
    XP[b * kColTile + lane] = b == p ? 0.0 : x;
  }
  double one = 1.0;
  asm("" : "+v"(one));   // in a register
  // |x_i - x_g|^2 over tiles of 64 consecutive pairs
  double r2 = 0.0;
  for (int64_t e0 = 0; e0 < D; e0 += kColTile) {
    __syncthreads();
    const int64_t e = min(e0 + lane, D - 1);
    double xi[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) xi[h] = Xi[min(e0 + 16 * h + (lane & 15), D - 1)];
#pragma unroll
    for (int c = 0; c < kColTile / kColWaves; ++c) {
      const int cc = wave + kColWaves * c;
      xs[lane * kXStride + cc] = -Xs[sg_of[cc] + e];
    }
    __syncthreads();
    const int ne = (int)min((int64_t)kColTile, D - e0);
    static_for<0, kColTile / 4>([&](auto J) {
      constexpr int q = 4 * decltype(J)::value;
      double d[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) d[j] = xs[(q + j) * kXStride + lane];
      four_differences<q % 16>(d, xi[q / 16], one);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (q + j < ne) r2 = fma(d[j], d[j], r2);
    });
  }
  // d . u, and sum_b u_{pb} (R_ip - R_ib) / r^3
  double du = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
  for (int b0 = 0; b0 < M; b0 += kAtoms) {   // eight pairs' loads in flight; U is zero at b = p
    double w[kAtoms][4];
#pragma unroll
    for (int q = 0; q < kAtoms; ++q) {
      const int b = min(b0 + q, M - 1);
      const double* src = Pi + (b == p ? 0 : pair_of(p, b)) * 4;
#pragma unroll
      for (int v = 0; v < 4; ++v) w[q][v] = src[v];
    }
#pragma unroll
    for (int q = 0; q < kAtoms; ++q) {
      const int b = min(b0 + q, M - 1);
      const double u = b0 + q < M ? U[b * kColTile + lane] : 0.0, us = p > b ? u : -u;
      du = fma(w[q][3] - XP[b * kColTile + lane], u, du);
      sx = fma(us, w[q][0], sx);
      sy = fma(us, w[q][1], sy);
      sz = fma(us, w[q][2], sz);
    }
  }
  const double z = sqrt(r2) * inv_len;
  const double ez = exp(-z);
  const double a = a0 * (1.0 + z) * ez;
  const double bdu = -bcoef * ez * du;

  for (int q0 = 0; q0 < M; q0 += kAtoms) {   // eight atoms' outputs at a time
    double vx[kAtoms], vy[kAtoms], vz[kAtoms];   // -(J_i^T d)_q
#pragma unroll
    for (int q = 0; q < kAtoms; ++q) vx[q] = vy[q] = vz[q] = 0.0;
    for (int b0 = 0; b0 < M; b0 += kAtoms) {
      __syncthreads();
      // the tile's pair l, along the faster atom of their order in memory: its
      // vector towards the atom of q, and zero where it is no pair
      const bool below = q0 >= b0;
      auto pair = [&](int l, double& sg) {
        const int hi = l >> 3, lo = l & 7;
        const int qa = q0 + (below ? hi : lo), ba = b0 + (below ? lo : hi);
        const bool is = qa != ba && qa < M && ba < M;
        sg = is ? (qa > ba ? 1.0 : -1.0) : 0.0;
        return is ? pair_of(qa, ba) : 0;
      };
      double sg;
      double w[4][4];   // of the pairs 16 h + lane % 16: the vector and 1 / r
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const double* src = Pi + 4 * (int64_t)pair(16 * h + (lane & 15), sg);
#pragma unroll
        for (int v = 0; v < 3; ++v) w[h][v] = sg * src[v];
        w[h][3] = src[3];
      }
      const int64_t e = pair(lane, sg);
#pragma unroll
      for (int c = 0; c < kColTile / kColWaves; ++c) {
        const int cc = wave + kColWaves * c;
        xs[lane * kXStride + cc] = -Xs[sg_of[cc] + e];
      }
      __syncthreads();
      // four partners b of an atom q at a time
      auto tile = [&](auto order) {
        static_for<0, 2 * kAtoms>([&](auto J) {
          constexpr int q = decltype(J)::value / 2, b = decltype(J)::value % 2 * 4;
          constexpr bool rows = decltype(order)::value;   // the pairs of an atom q follow one another
          constexpr int l = rows ? q % 2 * kAtoms + b : q;
          if (decltype(J)::value % 4 == 0) __builtin_amdgcn_sched_barrier(0);   // sixteen pairs' reads in flight
          double d[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) d[j] = xs[(rows ? q * kAtoms + b + j : (b + j) * kAtoms + q) * kXStride + lane];
          if constexpr (rows) four_pairs<l, l + 1, l + 2, l + 3>(d, vx[q], vy[q], vz[q], w[q / 2], w[q / 2], one);
          else four_pairs<l, l + kAtoms, l, l + kAtoms>(d, vx[q], vy[q], vz[q], w[b / 2], w[b / 2 + 1], one);
        });
      };
      if (below) tile(std::true_type());
      else tile(std::false_type());
    }
    __syncthreads();
    // outputs of four atoms at a time through LDS, so that a column's twelve
    // consecutive rows are stored together
    constexpr int OW = 12, OS = OW + 1;
    double* st = xs + wave * (kColTile * OS);
    static_assert(kColWaves * kColTile * OS <= kColTile * kXStride, "output staging fits the tile");
#pragma unroll
    for (int h = 0; h < kAtoms; h += 4) {
#pragma unroll
      for (int q = h; q < h + 4; ++q) {
        const int qa = q0 + q;
        if (qa < M) {
          const double* w = Pi + (qa != p ? pair_of(qa, p) : 0) * 4;
          const double u = U[qa * kColTile + lane], us = qa > p ? -u : u;
          const double ux = qa != p ? us * w[0] : -sx;   // (J_i^T u)_q
          const double uy = qa != p ? us * w[1] : -sy;
          const double uz = qa != p ? us * w[2] : -sz;
          const int64_t row = i * m3 + 3 * qa;
          double* o = st + lane * OS + 3 * (q - h);
          o[0] = a * ux - bdu * vx[q] + (row == col ? shift : 0.0);
          o[1] = a * uy - bdu * vy[q] + (row + 1 == col ? shift : 0.0);
          o[2] = a * uz - bdu * vz[q] + (row + 2 == col ? shift : 0.0);
        }
      }
      __builtin_amdgcn_wave_barrier();
      const int na = min(4, M - (q0 + h));   // atoms of this part
      if (na > 0 && i_raw < N) {
        const int nr = 3 * na;
        double* o = out + i * m3 + 3 * (q0 + h);
        for (int e = lane; e < kColTile * nr; e += 64) {
          const int c = e / nr, r = e % nr;
          if (c0 + c < k) {
            double* dst = o + (c0 + c) * ldo + r;
            const double val = st[c * OS + r];
            *dst = accumulate ? *dst + val : val;
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// The same for few columns: a wave takes one (target, column) pair, lanes over the
// pairs and then over the atoms; a block of up to four waves shares the target's
// geometry factors in LDS and walks 64 columns.  Arguments as for k_columns, from the
// geometries R, Rs.
__global__ __launch_bounds__(256) void k_columns_few(
    const double* __restrict__ R, const double* __restrict__ X, const double* __restrict__ Rs,
    const double* __restrict__ Xs, const int* __restrict__ pairs, int M, int64_t D, const int64_t* __restrict__ cols,
    int64_t k, double* __restrict__ out, int64_t ldo, double shift, double inv_len, double a0, double bcoef,
    int accumulate) {
  extern __shared__ double sm[];
  const int nw = blockDim.x >> 6;   // waves per block (1, 2 or 4)
  double* sRi = sm;                 // 3M
  double* sWi = sRi + 3 * M;        // 3D: (R_ia - R_ib)/r^3 for pair (a > b)
  double* sD = sWi + 3 * D;         // nw waves x D
  double* sU = sD + nw * D;         // nw waves x M
  const int64_t i = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m3 = 3 * M;
  const double* Xi = X + i * D;
  for (int e = threadIdx.x; e < m3; e += blockDim.x) sRi[e] = R[i * m3 + e];
  __syncthreads();
  for (int64_t e = threadIdx.x; e < D; e += blockDim.x) {
    const int pq = pairs[e];
    const int a = pq >> 16, b = pq & 0xFFFF;
    const double dx = sRi[3 * a] - sRi[3 * b], dy = sRi[3 * a + 1] - sRi[3 * b + 1], dz = sRi[3 * a + 2] - sRi[3 * b + 2];
    const double ir = 1.0 / sqrt(dx * dx + dy * dy + dz * dz);
    const double ir3 = ir * ir * ir;
    sWi[3 * e] = dx * ir3;
    sWi[3 * e + 1] = dy * ir3;
    sWi[3 * e + 2] = dz * ir3;
  }
  __syncthreads();
  double* dW = sD + wave * D;
  double* uW = sU + wave * M;
  const int64_t c0 = (int64_t)blockIdx.y * kColTile;
  // uniform trip count so that the block barriers below are reached by all waves
  const int cols_here = (int)min((int64_t)kColTile, k - c0);
  for (int it = 0; it < cols_here; it += nw) {
    const int64_t cidx = c0 + it + wave;
    const bool active = it + wave < cols_here;
    int64_t col = 0, g = 0;
    int p = 0, t = 0;
    double r2 = 0.0;
    if (active) {
      col = cols[cidx];
      g = col / m3;
      const int loc = (int)(col % m3);
      p = loc / 3;
      t = loc % 3;
      for (int64_t e = lane; e < D; e += 64) {      // d = x_i - x_g and |d|^2
        const double dd = Xi[e] - Xs[g * D + e];
        dW[e] = dd;
        r2 += dd * dd;
      }
      r2 = wave_sum(r2);
      const double* Rg = Rs + g * m3;
      for (int b = lane; b < M; b += 64) {          // u on the pairs {p, b}
        double u = 0.0;
        if (b != p) {
          const double dx = Rg[3 * p] - Rg[3 * b], dy = Rg[3 * p + 1] - Rg[3 * b + 1],
                       dz = Rg[3 * p + 2] - Rg[3 * b + 2];
          const double ir = 1.0 / sqrt(dx * dx + dy * dy + dz * dz);
          const double comp = t == 0 ? dx : (t == 1 ? dy : dz);
          u = -comp * ir * ir * ir;
        }
        uW[b] = u;
      }
    }
    __syncthreads();
    if (active) {
      double du = 0.0;
      for (int b = lane; b < M; b += 64)
        if (b != p) du += dW[pair_of(p, b)] * uW[b];
      du = wave_sum(du);
      const double z = sqrt(r2) * inv_len;
      const double ez = exp(-z);
      const double a = a0 * (1.0 + z) * ez;
      const double bdu = -bcoef * ez * du;
      for (int q = lane; q < M; q += 64) {
        double jx = 0.0, jy = 0.0, jz = 0.0;   // (J_i^T d)_q
        double ux = 0.0, uy = 0.0, uz = 0.0;   // (J_i^T u)_q
        for (int b = 0; b < M; ++b) {
          if (b == q) continue;
          const int e = pair_of(q, b);
          const double sgn = q > b ? 1.0 : -1.0;   // sWi holds (R_larger - R_smaller)/r^3
          const double wx = sgn * sWi[3 * e], wy = sgn * sWi[3 * e + 1], wz = sgn * sWi[3 * e + 2];
          const double de = dW[e];
          jx -= de * wx;
          jy -= de * wy;
          jz -= de * wz;
          const double ue = (q == p) ? uW[b] : (b == p ? uW[q] : 0.0);
          ux -= ue * wx;
          uy -= ue * wy;
          uz -= ue * wz;
        }
        const int64_t row = i * m3 + 3 * q;
        double* o = out + cidx * ldo + row;
        const double v0 = a * ux + bdu * jx + (row == col ? shift : 0.0);
        const double v1 = a * uy + bdu * jy + (row + 1 == col ? shift : 0.0);
        const double v2 = a * uz + bdu * jz + (row + 2 == col ? shift : 0.0);
        if (accumulate) {
          o[0] += v0;
          o[1] += v1;
          o[2] += v2;
        } else {
          o[0] = v0;
          o[1] = v1;
          o[2] = v2;
        }
      }
    }
    __syncthreads();
  }
}

static int max_lds_bytes() {
  static int max_lds = 0;
  if (max_lds == 0) {
    int dv = 0;
    HIPCHK(hipGetDevice(&dv));
    HIPCHK(hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dv));
  }
  return max_lds;
}

// LDS of a block of k_columns_few, and the waves (1, 2 or 4) that fit.
static size_t few_lds(int w, int M, int64_t D) { return (size_t)(3 * M + 3 * D + w * (D + M)) * sizeof(double); }
static int few_waves(int M, int64_t D) {
  int nw = 4;
  while (nw > 1 && few_lds(nw, M, D) > (size_t)max_lds_bytes()) nw >>= 1;
  return nw;
}

// Whether k columns are few: k_columns takes as long for one as for 64, k_columns_few a
// step for every nw of them, in rounds of the blocks that fit the CUs' LDS.  A step takes
// a tenth to a twelfth of a round of k_columns where molecules are large; from 16 or 24
// columns on (up to 48 of few targets, which leave CUs idle either way), fewer of small
// molecules, most of whose lanes idle, the arithmetic decides.  The call, us, by
// k_columns_few and k_columns: M = 100, N = 1000, k = 4 866 and 753, N = 200, k = 10 564 and
// 701, 14 754 and 705; M = 80, N = 500, k = 10 433 and 466, 14 578 and 464; M = 70, N = 2000,
// k = 10 830 and 758; M = 64, N = 1000, k = 12 277 and 329, 14 343 and 331; M = 60, N = 2000,
// k = 12 466 and 589, 20 734 and 617; M = 43, N = 3000, k = 16 269 and 379, 24 371 and 393,
// N = 100, k = 48 172 and 193; M = 30, N = 5000, k = 24 306 and 317, N = 500, k = 32 109 and
// 119, 48 144 and 123; M = 21, N = 2000, k = 1 53 and 103, 14 101 and 104, 20 117 and 106, N
// = 100, k = 24 74 and 87; M = 9, N = 200, k = 12 53 and 59; M = 8, N = 100, k = 8 52 and 51;
// M = 5, N = 20000, k = 4 112 and 159, 8 178 and 156.
static bool few_columns(int64_t k, int M, int64_t D, int64_t N) {
  const int many = N > 512 ? (M < 24 ? 16 : 24) : M < 16 ? 16 : M < 24 ? 24 : M < 36 ? 32 : 48;
  if (k > (M < 8 ? 4 : M < 12 ? 12 : many)) return false;
  const int64_t cus = device_cus(), lds = max_lds_bytes();
  const int nw = few_waves(M, D);
  const int64_t rounds = cdiv(N, cus * std::min<int64_t>(8, lds / (int64_t)few_lds(nw, M, D)));
  const int64_t tiles = cdiv(cdiv(N, kColWaves), cus * std::min<int64_t>(8, lds / (int64_t)columns_lds(M)));
  const int steps = nw == 1 || (nw == 4 && D < 2200) ? 12 : 10;   // of a round
  return rounds * cdiv(k, nw) <= steps * tiles;
}

// The interface's limit on the molecule: four values per atom and pair in the LDS
// of a block.  The columns' kernel (a tile and two tables of 64 values an atom) and
// the selection's need less than that at every M it allows.
void require_columns_fit(const ffk_system* s) {
  const size_t limit = (size_t)(4 * s->M + 4 * s->D) * sizeof(double);
  if (limit > (size_t)max_lds_bytes() || columns_lds(s->M) > (size_t)max_lds_bytes())
    fail(FFK_ERR_ARG, "kernel_columns: descriptor too large for the LDS staging");
}

// Columns of K(s, src) in the source numbering (src = s for the plain kernel).
void kernel_columns_src(const ffk_system* s, const ffk_system* src, const int64_t* cols, int64_t k, double* out,
                        int64_t ldo, double shift, bool accumulate, hipStream_t st) {
  if (k <= 0) return;
  const int M = s->M;
  const int64_t D = s->D;
  require_columns_fit(s);
  const int64_t per_launch = (int64_t)65535 * kColTile;
  // (without the pair tables, for which memory may be short, any number goes as few do)
  const bool few = few_columns(k, M, D, s->N) || !pair_table(s, st) || !pair_table(src, st);
  const int nw = few_waves(M, D);
  const size_t shm = columns_lds(M);
  if (!few && shm > 65536)
    HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_columns), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)shm));
  for (int64_t c0 = 0; c0 < k; c0 += per_launch) {
    const int64_t kc = std::min(per_launch, k - c0);
    const unsigned tiles = (unsigned)cdiv(kc, kColTile);
    if (few)
      k_columns_few<<<dim3((unsigned)s->N, tiles), 64 * nw, few_lds(nw, M, D), st>>>(
          s->R.as<double>(), s->X.as<double>(), src->R.as<double>(), src->X.as<double>(), s->pairs.as<int>(), M, D,
          cols + c0, kc, out + c0 * ldo, ldo, shift, sqrt(5.0) / s->sigma, s->a0, s->bcoef, accumulate ? 1 : 0);
    else
      k_columns<<<dim3((unsigned)cdiv(s->N, kColWaves), tiles), 64 * kColWaves, shm, st>>>(
          s->PT.as<double>(), s->X.as<double>(), src->PT.as<double>(), src->X.as<double>(), s->N, M, D, cols + c0, kc,
          out + c0 * ldo, ldo, shift, sqrt(5.0) / s->sigma, s->a0, s->bcoef, accumulate ? 1 : 0);
    LAUNCHCHK();
  }
}

void kernel_columns(const ffk_system* s, const int64_t* cols, int64_t k, double* out, int64_t ldo, double shift,
                    hipStream_t st) {
  if (!s->sym.empty()) sym_columns(s, cols, k, out, ldo, shift, st);
  else kernel_columns_src(s, s, cols, k, out, ldo, shift, false, st);
}

// diag(K)_{3Mg + 3p + t} = a(0) sum_{b != p} ((R_gp - R_gb)_t / r^3)^2
__global__ void k_diag(const double* __restrict__ R, int64_t N, int M, double a0, double* __restrict__ d) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N * M) return;
  const int64_t g = e / M;
  const int p = (int)(e % M);
  const double* Rg = R + g * 3 * M;
  double sx = 0.0, sy = 0.0, sz = 0.0;
  for (int b = 0; b < M; ++b) {
    if (b == p) continue;
    const double dx = Rg[3 * p] - Rg[3 * b], dy = Rg[3 * p + 1] - Rg[3 * b + 1], dz = Rg[3 * p + 2] - Rg[3 * b + 2];
    const double ir = 1.0 / sqrt(dx * dx + dy * dy + dz * dz);
    const double ir3 = ir * ir * ir;
    sx += dx * dx * ir3 * ir3;
    sy += dy * dy * ir3 * ir3;
    sz += dz * dz * ir3 * ir3;
  }
  d[3 * e] = a0 * sx;
  d[3 * e + 1] = a0 * sy;
  d[3 * e + 2] = a0 * sz;
}

void kernel_diag(const ffk_system* s, double* d, hipStream_t st) {
  if (!s->sym.empty()) {
    sym_diag(s, d, st);
    return;
  }
  k_diag<<<cdiv(s->N * s->M, 256), 256, 0, st>>>(s->R.as<double>(), s->N, s->M, s->a0, d);
  LAUNCHCHK();
}

double max_diag(ffk_system* s, hipStream_t st) {
  if (s->max_diag > 0) return s->max_diag;
  DBuf d(s->n * 8), m(8), part(kRedParts * 8);
  kernel_diag(s, d.as<double>(), st);
  reduce_max64(d.as<double>(), s->n, part.as<double>(), m.as<double>(), st);
  double h = 0;
  HIPCHK(hipMemcpyAsync(&h, m.get(), 8, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  s->max_diag = h;
  return h;
}

}  // namespace ffk
