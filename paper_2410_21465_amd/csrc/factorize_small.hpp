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

}  // namespace skv
