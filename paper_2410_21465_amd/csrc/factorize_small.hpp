// Small fp64 linear algebra of the key factorisation (kernels_factorize.hip): the subspace iteration and the
// Rayleigh-Ritz step work on m = rank + oversample vectors of the key width D, a few hundred by a thousand numbers.
// Everything is fp64; contractions run on v_mfma_f64_16x16x4f64 (A lane l holds (m = l % 16, k = l / 16), B lane l holds
// (n = l % 16, k = l / 16), result register j of lane l is (m = 4 j + l / 16, n = l % 16); measured on gfx950).
#pragma once
#include "common.hpp"

namespace skv {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// ---- products ---------------------------------------------------------------------------------------
// C[i][j] = sum_k A[i][k] B(k, j), K a multiple of 16, rows of A 16-byte aligned.  BT: B is given by its columns
// (B(k, j) = B[j][k], as A is); otherwise row-major with Kb rows (A is zero beyond).  Rows of A may be taken through a_rows.  C is written over
// Mw x Nw, zero outside M x N.
// A workgroup is WM x WN tiles of 32 x 32 with the contraction cut WK ways; every operand goes from L2 straight to the
// matrix instruction (a lane's four consecutive elements are four contraction steps), the next 16 steps requested
// before the current ones' 16 instructions.  The products here are small (192 x 1024 x 1024 per sequence), so what
// bounds them is how many waves there are: for one sequence WK = 8 gives 1536 waves of 128 steps each; with several
// sequences the 2 x 2 x 2 form halves the L2 traffic instead.
template <int WM, int WN, int WK, bool BT>
__global__ __launch_bounds__(64 * WM * WN * WK) void gemm64_kernel(const double* __restrict__ A,
                                                                   const double* __restrict__ B, double* __restrict__ C,
                                                                   int M, int N, int K, int Kb, int lda, int ldb, int ldc,
                                                                   int Mw, int Nw, size_t strideA, size_t strideB, size_t strideC,
                                                                   const int32_t* __restrict__ a_rows, int a_rows_stride) {
  __shared__ double red[WM * WN][WK][16][kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int sub = lane & 15, kq = lane >> 4;
  const int wk = wave % WK, wt = wave / WK, wn = wt % WN, wm = wt / WN;
  const int i0 = (blockIdx.y * WM + wm) * 32, j0 = (blockIdx.x * WN + wn) * 32;
  A += blockIdx.z * strideA; B += blockIdx.z * strideB; C += blockIdx.z * strideC;
  if (a_rows) a_rows += (size_t)blockIdx.z * a_rows_stride;
  const double* ap[2];
  const double* bp[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {   // rows and columns past the end repeat the last real one; their results are not used
    const int i = min(i0 + 16 * t + sub, M - 1), j = min(j0 + 16 * t + sub, N - 1);
    ap[t] = A + (size_t)(a_rows ? a_rows[i] : i) * lda + 4 * kq;
    bp[t] = BT ? B + (size_t)j * ldb + 4 * kq : B + j;
  }
  double an[2][4], bn[2][4];
  auto request = [&](int k0) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const double2 lo = *reinterpret_cast<const double2*>(ap[t] + k0), hi = *reinterpret_cast<const double2*>(ap[t] + k0 + 2);
      an[t][0] = lo.x; an[t][1] = lo.y; an[t][2] = hi.x; an[t][3] = hi.y;
      if constexpr (BT) {
        const double2 bl = *reinterpret_cast<const double2*>(bp[t] + k0), bh = *reinterpret_cast<const double2*>(bp[t] + k0 + 2);
        bn[t][0] = bl.x; bn[t][1] = bl.y; bn[t][2] = bh.x; bn[t][3] = bh.y;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) bn[t][e] = bp[t][(size_t)min(k0 + 4 * kq + e, Kb - 1) * ldb];
      }
    }
  };
  f64x4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int step = 16 * WK;
  if (16 * wk < K) request(16 * wk);
  for (int k0 = 16 * wk; k0 < K; k0 += step) {
    double a[2][4], b[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) { a[t][e] = an[t][e]; b[t][e] = bn[t][e]; }
    if (k0 + step < K) request(k0 + step);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x][e], b[y][e], acc[x][y], 0, 0, 0);
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int j = 0; j < 4; ++j) red[wt][wk][(x * 2 + y) * 4 + j][lane] = acc[x][y][j];
  __syncthreads();
  // each of the WK waves of a tile adds up 16 / WK of its registers
#pragma unroll
  for (int u = 0; u < 16 / WK; ++u) {
    const int reg = wk * (16 / WK) + u;
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < WK; ++w) sum += red[wt][w][reg][lane];
    const int i = i0 + 16 * (reg >> 3) + 4 * (reg & 3) + kq, j = j0 + 16 * ((reg >> 2) & 1) + sub;
    if (i < Mw && j < Nw) C[(size_t)i * ldc + j] = (i < M && j < N) ? sum : 0.0;
  }
}

// ---- orthonormalisation: X <- L^-1 Y with Y Y^T = L L^T -------------------------------------------------
// Three launches (the product above, chol_kernel, trsm_kernel) for all vectors of a sequence instead of a chain over
// them.  One pass leaves the vectors orthonormal to (condition of Y)^2 times the rounding unit, two passes to the
// rounding unit; pivots that rounding has eaten are handled as said at chol_kernel.
// 16 x 16 blocks in operand order: element (row, col) of a block is entry 4 (row + 16 (col % 4)) + col / 4, so that lane
// l = row + 16 k-slot reads its four contraction steps as 32 consecutive bytes.
__device__ __forceinline__ int op_index(int row, int col) { return (row + 16 * (col & 3)) * 4 + (col >> 2); }
// block (i, k), i >= k, of the packed lower triangle of nb block columns
__device__ __forceinline__ int tri_block(int nb, int i, int k) { return k * nb - k * (k - 1) / 2 + (i - k); }
constexpr int kMaxFactorBlocks = 18;       // 288 = 256 + 32 vectors
constexpr double kPivotFloor = 1e-13;      // share of a vector's square below which its remainder is rounding

__device__ __forceinline__ double lane_f64(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Cholesky factor of S [m][ld] (lower triangle read), one workgroup of eight waves per sequence.  Lp: packed blocks in
// operand order, off the diagonal -L, on it the inverse of L's block (what trsm_kernel multiplies by).
// The trailing blocks stay in the accumulators of the waves (blocks dealt out in turn, NBW per wave) for the whole
// factorisation; only the current block column goes through LDS.  What bounds it is the chain of pivots: 16 rsqrt + updates
// per diagonal block in one wave, which carries the unit matrix along in a second group of lanes and so ends with the
// inverse as well.
// A pivot below kPivotFloor of the vector's own square is rounding: it is set to that floor, which leaves the vector's
// remainder at a size that the next pass can work on, and nothing is projected on it; a zero vector stays zero.
template <int NBW>
__global__ __launch_bounds__(512) void chol_kernel(const double* __restrict__ S, double* __restrict__ Lp, int m, int ld,
                                                   int nb) {
  __shared__ double col[kMaxFactorBlocks][272];   // current block column: rows at a pitch of 17, then operand order
  __shared__ double inv[256];                     // inverse of the diagonal block, rows of floored pivots zero
  __shared__ double d0[kMaxFactorBlocks * 16];    // squares of the vectors
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int sub = lane & 15, kq = lane >> 4;
  S += (size_t)blockIdx.x * ld * ld;
  Lp += (size_t)blockIdx.x * (nb * (nb + 1) / 2) * 256;
  f64x4 acc[NBW];
  int bi[NBW], bk[NBW];
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    int idx = wave + 8 * t, k = 0;
    while (k < nb && idx >= nb - k) { idx -= nb - k; ++k; }
    bk[t] = k; bi[t] = k + idx;     // k == nb: no block
    acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (k < nb) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = 16 * bi[t] + 4 * j + kq, c = 16 * k + sub;
        if (r < m && c < m) acc[t][j] = S[(size_t)r * ld + c];
        if (r == c) d0[r] = acc[t][j];
      }
    }
  }
  for (int k = 0; k < nb; ++k) {
#pragma unroll
    for (int t = 0; t < NBW; ++t)
      if (bk[t] == k)
#pragma unroll
        for (int j = 0; j < 4; ++j) col[bi[t]][(4 * j + kq) * 17 + sub] = acc[t][j];
    __syncthreads();
    double* out = Lp + (size_t)tri_block(nb, k, k) * 256;
    if (wave == 0) {
      // lanes 0-15: rows of the block; lanes 16-31: columns of the unit matrix, which become those of the inverse
      double a[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) a[j] = lane < 16 ? col[k][sub * 17 + j] : (lane < 32 && j == sub ? 1.0 : 0.0);
      const double e0 = d0[16 * k + sub];
      uint32_t floored = 0;
#pragma unroll
      for (int p = 0; p < 16; ++p) {
        const double d = lane_f64(a[p], p), e = lane_f64(e0, p);
        const bool none = !(e > 0.0), low = !none && d < kPivotFloor * e;
        const double piv = none ? 1.0 : (low ? kPivotFloor * e : d);
        const double mult = a[p] * (1.0 / sqrt(piv));
        a[p] = mult;
        if (none || low) {
          floored |= 1u << p;
        } else {
#pragma unroll
          for (int j = p + 1; j < 16; ++j) a[j] = fma(-mult, lane_f64(mult, j), a[j]);
        }
      }
      if (kq == 1) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          out[op_index(j, sub)] = a[j];
          inv[op_index(j, sub)] = (floored >> j) & 1 ? 0.0 : a[j];
        }
      }
    }
    __syncthreads();
    // L(i, k) = A(i, k) inv^T
    for (int i = k + 1 + wave; i < nb; i += 8) {
      double a[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) a[t] = col[i][sub * 17 + 4 * t + kq];
      f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int t = 0; t < 4; ++t) x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], inv[lane * 4 + t], x, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) col[i][op_index(4 * j + kq, sub)] = x[j];
      double* dst = Lp + (size_t)tri_block(nb, i, k) * 256;
#pragma unroll
      for (int t = 0; t < 4; ++t) dst[lane * 4 + t] = -col[i][lane * 4 + t];
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NBW; ++t)
      if (bk[t] > k && bk[t] < nb) {
#pragma unroll
        for (int x = 0; x < 4; ++x)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-col[bi[t]][lane * 4 + x], col[bk[t]][lane * 4 + x], acc[t], 0, 0, 0);
      }
    __syncthreads();
  }
}

// X = L^-1 Y, rows of length D: one wave per 16 columns holds all its rows in accumulators and goes down the block rows; a
// finished block is in the operand layout already (result register t of a lane is the row of contraction step t).
// The blocks of the next block column are requested while the current one's instructions run, as far as registers go.
template <int NB>
__global__ __launch_bounds__(64) void trsm_kernel(const double* __restrict__ Lp, const double* __restrict__ Y,
                                                  double* __restrict__ X, int m, int nb, int D) {
  const int lane = threadIdx.x, sub = lane & 15, kq = lane >> 4;
  const size_t base = (size_t)blockIdx.y * m * D + blockIdx.x * 16 + sub;
  Lp += (size_t)blockIdx.y * (nb * (nb + 1) / 2) * 256 + lane * 4;
  constexpr bool kAhead = NB <= 14;
  double next[NB][4];
  auto request = [&](int k) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (i >= k && i < nb) {
        const double2* p = reinterpret_cast<const double2*>(Lp + (size_t)tri_block(nb, i, k) * 256);
        const double2 lo = p[0], hi = p[1];
        next[i][0] = lo.x; next[i][1] = lo.y; next[i][2] = hi.x; next[i][3] = hi.y;
      }
  };
  if (kAhead) request(0);
  f64x4 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = 16 * i + 4 * j + kq;
      acc[i][j] = r < m ? Y[base + (size_t)r * D] : 0.0;
    }
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    if (k < nb) {
    double cur[NB][4];
    if (!kAhead) request(k);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t) cur[i][t] = i >= k ? next[i][t] : 0.0;
    if (kAhead && k + 1 < nb) request(k + 1);
    f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 4; ++t) x = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[k][t], acc[k][t], x, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = 16 * k + 4 * j + kq;
      if (r < m) X[base + (size_t)r * D] = x[j];
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (i > k && i < nb)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[i][t], x[t], acc[i], 0, 0, 0);
    }
  }
}

}  // namespace skv
