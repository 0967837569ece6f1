// Small fp64 linear algebra of the key factorisation (kernels_factorize.hip): the subspace iteration and the
// Rayleigh-Ritz step work on m = rank + oversample vectors of the key width D, a few hundred by a thousand numbers.
// Everything is fp64; contractions run on v_mfma_f64_16x16x4f64 (A lane l holds (m = l % 16, k = l / 16), B lane l holds
// (n = l % 16, k = l / 16), result register j of lane l is (m = 4 j + l / 16, n = l % 16); measured on gfx950).
#pragma once
#include "common.hpp"

namespace skv {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Of the steps 1, 2, ... a sequence takes every n-th, n = every[sequence] without kMoreSteps (all of them without `every`); with
// `more` those sequences alone whose entry has kMoreSteps, the others are done.
constexpr int kMoreSteps = 4;
struct Every { const int32_t* every; int step; bool more; };
__device__ __forceinline__ bool sequence_done(Every e, int sequence) { return e.more && !(e.every[sequence] & kMoreSteps); }
__device__ __forceinline__ bool step_left_out(Every e, int sequence) {
  return sequence_done(e, sequence) || (e.every && e.step % (e.every[sequence] & ~kMoreSteps) != 0);
}

// What a factor says of the shifted steps of its sequence: b, of whose shares the shifts are, and a power of two that brings the
// longest vector of a step between 1/2 and 1 (see chol_kernel).
struct Shift { double b, scale; };

// ---- products ---------------------------------------------------------------------------------------
// C[i][j] = sum_k A[i][k] B(k, j), K a multiple of 16, rows of A 16-byte aligned.  BT: B is given by its columns
// (B(k, j) = B[j][k], as A is); otherwise row-major with Kb rows (A is zero beyond).  Rows of A may be taken through
// a_rows.  C is written over Mw x Nw, zero outside M x N.  With `shift` (one per sequence; N = K): C = A (B - node b) scale.
// With `every`, see step_left_out; with `lower` blocks above the diagonal are left as they were.
// A workgroup is WM x WN tiles of 16 T x 16 T with the contraction cut WK ways; every operand goes from L2 straight to the
// matrix instruction (a lane's four consecutive elements are four contraction steps), the next 16 steps requested
// before the current ones' 16 instructions.  The products here are small (192 x 1024 x 1024 per sequence), so what
// bounds them is how many waves there are: for one sequence T = 2, WK = 8 gives 1536 waves of 128 steps each; with several
// sequences T = 4 halves the L2 traffic instead; the m x m products have so few tiles that T = 1 is faster.
template <int T, int WM, int WN, int WK, bool BT>
__global__ __launch_bounds__(64 * WM * WN * WK) void gemm64_kernel(const double* __restrict__ A,
                                                                   const double* __restrict__ B, double* __restrict__ C,
                                                                   int M, int N, int K, int Kb, int lda, int ldb, int ldc,
                                                                   int Mw, int Nw, size_t strideA, size_t strideB, size_t strideC,
                                                                   const int32_t* __restrict__ a_rows, int a_rows_stride,
                                                                   const Shift* __restrict__ shift, double node, Every every,
                                                                   bool lower) {
  if (step_left_out(every, blockIdx.z) || (lower && blockIdx.x * WN >= (blockIdx.y + 1) * WM)) return;
  __shared__ double red[WM * WN][WK][4 * T * T][kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int sub = lane & 15, kq = lane >> 4;
  const int wk = wave % WK, wt = wave / WK, wn = wt % WN, wm = wt / WN;
  const int i0 = (blockIdx.y * WM + wm) * 16 * T, j0 = (blockIdx.x * WN + wn) * 16 * T;
  A += blockIdx.z * strideA; B += blockIdx.z * strideB; C += blockIdx.z * strideC;
  if (a_rows) a_rows += (size_t)blockIdx.z * a_rows_stride;
  const double* ap[T];
  const double* bp[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {   // rows and columns past the end repeat the last real one; their results are not used
    const int i = min(i0 + 16 * t + sub, M - 1), j = min(j0 + 16 * t + sub, N - 1);
    ap[t] = A + (size_t)(a_rows ? a_rows[i] : i) * lda + 4 * kq;
    bp[t] = BT ? B + (size_t)j * ldb + 4 * kq : B + j;
  }
  double an[T][4], bn[T][4];
  auto request = [&](int k0) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
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
  f64x4 acc[T][T];
#pragma unroll
  for (int x = 0; x < T; ++x)
#pragma unroll
    for (int y = 0; y < T; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int step = 16 * WK;
  if (16 * wk < K) request(16 * wk);
  for (int k0 = 16 * wk; k0 < K; k0 += step) {
    double a[T][4], b[T][4];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) { a[t][e] = an[t][e]; b[t][e] = bn[t][e]; }
    if (k0 + step < K) request(k0 + step);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int x = 0; x < T; ++x)
#pragma unroll
        for (int y = 0; y < T; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x][e], b[y][e], acc[x][y], 0, 0, 0);
  }
#pragma unroll
  for (int x = 0; x < T; ++x)
#pragma unroll
    for (int y = 0; y < T; ++y)
#pragma unroll
      for (int j = 0; j < 4; ++j) red[wt][wk][(x * T + y) * 4 + j][lane] = acc[x][y][j];
  __syncthreads();
  const double theta = shift ? node * shift[blockIdx.z].b : 0.0, scale = shift ? shift[blockIdx.z].scale : 1.0;
  // the WK waves of a tile add up its 4 T T registers in turn
#pragma unroll
  for (int reg = wk; reg < 4 * T * T; reg += WK) {
    const int tile = reg >> 2;
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < WK; ++w) sum += red[wt][w][reg][lane];
    const int i = i0 + 16 * (tile / T) + 4 * (reg & 3) + kq, j = j0 + 16 * (tile % T) + sub;
    if (shift && i < M && j < N) sum = fma(-theta, A[(size_t)i * lda + j], sum) * scale;
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
constexpr double kShiftRatio = 4.0;        // r-th eigenvalue over the last that the vectors hold, from which steps are shifted

__device__ __forceinline__ double lane_f64(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

// 1 / sqrt(x) for a positive normal x: the hardware's estimate and two Newton steps (the library's 1.0 / sqrt(x) is
// three times the chain)
__device__ __forceinline__ double rsqrt_f64(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int i = 0; i < 2; ++i) y = fma(y * 0.5, fma(-x * y, y, 1.0), y);
  return y;
}

// Factorisation of a 16 x 16 diagonal block by one wave, four pivots at a time on the matrix instruction.  Register j of lane
// (sub, kq) holds entry (4 j + kq, sub), by symmetry also (sub, 4 j + kq): register j is the operand of a contraction over
// columns 4 j .. 4 j + 3 as it stands.  Per panel: the reciprocals r of the 4 x 4 block's pivots and the inverse N of its unit
// lower factor in every lane alike; U = N times the panel's rows; the rest of the block less U^T diag(r) U; and the unit matrix
// carried along the same way, of which N times rows 4 j .. 4 j + 3 are, up to the roots of the pivots, rows of the inverse.
// f, d: of rows 4 j + kq these rows (column sub), and the pivots.  CHECK: pivots below `least` (of their row) project nothing.
template <bool CHECK>
__device__ __forceinline__ void factor_panels(f64x4 a, const double (&least)[4], double (&f)[4], double (&d)[4]) {
  const int lane = threadIdx.x & (kWave - 1), sub = lane & 15, kq = lane >> 4, at = 4 * (sub & 3) + kq;
  const bool k1 = kq == 1, k2 = kq == 2, k3 = kq == 3;
  f64x4 e;
#pragma unroll
  for (int j = 0; j < 4; ++j) e[j] = 4 * j + kq == sub ? 1.0 : 0.0;
  each_of(std::make_integer_sequence<int, 4>{}, [&](auto jc) {
    constexpr int J = jc;
    double r[4], l[4][4], s[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = q; p < 4; ++p) s[p][q] = lane_f64(a[J], 4 * J + p + 16 * q);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      // the hardware's estimate y (24 bits) times 1 + g + g^2, g = 1 - d y
      double y = __builtin_amdgcn_rcp(s[p][p]);
      if constexpr (CHECK) y = s[p][p] < lane_f64(least[J], 16 * p) ? 0.0 : y;
      const double g = fma(-s[p][p], y, 1.0), h = fma(g, g, g);
      r[p] = fma(y, h, y);
#pragma unroll
      for (int i = p + 1; i < 4; ++i) {
        const double t = s[i][p] * y;
        l[i][p] = fma(t, h, t);
#pragma unroll
        for (int q = p + 1; q <= i; ++q) s[i][q] = fma(-l[i][p], s[q][p], s[i][q]);
      }
    }
    // (computed by all lanes: not to be drawn into branches of the selections below)
    asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
    const double n10 = -l[1][0], n21 = -l[2][1], n32 = -l[3][2];
    const double n20 = fma(n21, n10, -l[2][0]), n31 = fma(n32, n21, -l[3][1]);
    const double n30 = fma(n32, n20, fma(-l[3][1], n10, -l[3][0]));
    // N as the left operand of four 4 x 4 x 4 products side by side (lane: row sub % 4, column kq)
    double nv = (sub & 3) == kq ? 1.0 : 0.0;
    nv = at == 4 ? n10 : nv; nv = at == 9 ? n21 : nv; nv = at == 8 ? n20 : nv;
    nv = at == 14 ? n32 : nv; nv = at == 13 ? n31 : nv; nv = at == 12 ? n30 : nv;
    d[J] = k1 ? s[1][1] : s[0][0];
    d[J] = k2 ? s[2][2] : d[J];
    d[J] = k3 ? s[3][3] : d[J];
    if constexpr (J < 3) {
      double rk = k1 ? r[1] : r[0];
      rk = k2 ? r[2] : rk;
      rk = k3 ? r[3] : rk;
      rk = sub >= 4 * (J + 1) ? -rk : 0.0;   // rows below the panel
      const double u = __builtin_amdgcn_mfma_f64_4x4x4f64(nv, a[J], 0.0, 0, 0, 0);   // row kq, column sub
      const double w = rk * u;
      a = __builtin_amdgcn_mfma_f64_16x16x4f64(w, u, a, 0, 0, 0);
      f[J] = __builtin_amdgcn_mfma_f64_4x4x4f64(nv, e[J], 0.0, 0, 0, 0);
      e = __builtin_amdgcn_mfma_f64_16x16x4f64(w, f[J], e, 0, 0, 0);
    } else {
      f[J] = __builtin_amdgcn_mfma_f64_4x4x4f64(nv, e[J], 0.0, 0, 0, 0);
    }
  });
}

// The block's inverse factor.  Pivots below kPivotFloor times their vector's square (e0[j], row 4 j + kq) project nothing and
// count as that (see chol_kernel); a block that has one is taken again with the checks.
// out: the inverse in operand order; inv: the same, rows of floored pivots zero; smallest: the least pivot of the lane's rows and
// what it was before, 0 if one of them was floored, infinity for zero vectors; wanted: the same of the block's first n_wanted rows.
__device__ __forceinline__ void factor_block(f64x4 a, const double (&e0)[4], double* __restrict__ out, double* __restrict__ inv,
                                             int n_wanted, double& smallest, double& wanted) {
  const int lane = threadIdx.x & (kWave - 1), sub = lane & 15, kq = lane >> 4;
  double f[4], d[4], least[4];
  bool bad = false;
  factor_panels<false>(a, least, f, d);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    least[j] = e0[j] > 1e-280 ? kPivotFloor * e0[j] : INFINITY;
    bad |= d[j] < least[j];
  }
  if (__builtin_expect(__any(bad), 0)) factor_panels<true>(a, least, f, d);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool none = least[j] == INFINITY, floored = d[j] < least[j];
    const double piv = none ? 1.0 : (floored ? least[j] : d[j]), x = f[j] * rsqrt_f64(piv);
    const double p = none ? INFINITY : floored ? 0.0 : piv;
    smallest = fmin(smallest, p);
    wanted = 4 * j + kq < n_wanted ? fmin(wanted, p) : wanted;
    out[op_index(4 * j + kq, sub)] = x;
    inv[op_index(4 * j + kq, sub)] = floored ? 0.0 : x;
  }
}

// Cholesky factor of S [16 nb][16 nb] (lower triangle read; zero beyond the vectors), one workgroup of eight waves per
// sequence.  Lp: packed blocks in operand order, off the diagonal -L, on it the inverse of L's block (what trsm_kernel
// multiplies by).
// Wave 0 has the chain: it takes block (k + 1, k) of column k, the next diagonal block and that block's pivots, while the
// others finish column k and keep the trailing blocks in their accumulators (dealt out in turn by columns, NBW per wave) up
// to date; of those, the next block column and the diagonal block after the next go through LDS.
// What bounds it is that chain: for 192 vectors a step takes 5,000 cycles, 3,300 of them the pivots (panels of four on the
// matrix instruction; a column at a time with broadcasts along the rows 5,000) and 750 the next block, the first three steps
// half as much again for the others' matrix instructions; the start 6,000.  33 us in all, where one wave after the other,
// pivots, column, trailing blocks with four barriers a step, took 49.  Above 192 vectors a wave's blocks fill its registers.
// A pivot below kPivotFloor of the vector's own square is rounding: it is set to that floor, which leaves the vector's
// remainder at a size that the next pass can work on, and nothing is projected on it; a zero vector stays zero.
// shift (may be NULL): of each sequence b, the least entry of L's diagonal, 0 where a pivot was set to its floor or where one of
// the first r entries is less than kShiftRatio times the least (see launch_factorize), and the power of two that brings the
// longest vector between 1/2 and 1; and `pause`: how many of the steps that follow may go without an orthonormalisation in
// between, one more than that, and kMoreSteps where b is 0.  What an earlier vector leaves in a later one by rounding (1e-16) grows by
// the ratio of their eigenvalues in every step; up to three steps, as long as the largest ratio (that of the longest vector and
// the least entry) to their number is below 1e13.  The products of vectors three steps apart from orthonormal ones are sixth
// powers of eigenvalues, twelfth powers of singular values: without the power of two those of keys beyond 2^82 leave fp64, and
// those of keys below 2^-82 fall under what counts as a zero vector.
template <int NBW>
__global__ __launch_bounds__(512) void chol_kernel(const double* __restrict__ S, double* __restrict__ Lp, int nb,
                                                   int r, Shift* __restrict__ shift, int32_t* __restrict__ pause,
                                                   Every every) {
  if (step_left_out(every, blockIdx.x)) return;
  __shared__ double col[kMaxFactorBlocks][272];   // current block column, rows at a pitch of 17
  __shared__ double sol[kMaxFactorBlocks][256];   // the same times the diagonal block's inverse, operand order
  __shared__ double inv[256];                     // inverse of the diagonal block, rows of floored pivots zero
  __shared__ double next[4][kWave];               // the diagonal block after the next, as in the accumulators
  __shared__ uint16_t place[7][NBW];              // block row and column of the blocks of waves 1 .. 7 (column nb: no block)
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int sub = lane & 15, kq = lane >> 4;
  const int ld = 16 * nb;
  S += (size_t)blockIdx.x * ld * ld;
  Lp += (size_t)blockIdx.x * (nb * (nb + 1) / 2) * 256;
  const double* Sl = S + (size_t)kq * ld + sub;
  // trailing blocks: columns 1 .. nb - 1 from the diagonal down, without (1, 1); wave 4, which shares wave 0's SIMD, takes part
  // in the first quarter of the columns only
  const int c7 = NBW == 11 ? nb / 4 : nb, n7 = c7 * nb - c7 * (c7 + 1) / 2 - 1, t7 = (max(n7, 0) + 6) / 7;
  for (int x = threadIdx.x; x < 7 * NBW; x += 512) {
    const int w = x % 7, t = x / 7;
    int idx = t < t7 ? (x < n7 ? x + 1 : 1 << 20) : w == 3 ? 1 << 20 : n7 + 1 + (t - t7) * 6 + w - (w > 3 ? 1 : 0), k = 1;
    while (k < nb && idx >= nb - k) { idx -= nb - k; ++k; }
    place[w][t] = k < nb ? (uint16_t)((k + idx) << 8 | k) : (uint16_t)nb;
  }
  for (int x = threadIdx.x; x < (nb - 1) * 256; x += 512) {
    const int i = 1 + (x >> 8), r = (x >> 4) & 15, c = x & 15;
    col[i][r * 17 + c] = S[(size_t)(16 * i + r) * ld + c];
  }
  __syncthreads();
  if (wave == 0) {
    f64x4 d;
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = Sl[4 * j * ld];
    f64x4 a = d;
    if (nb > 1)
#pragma unroll
      for (int j = 0; j < 4; ++j) d[j] = -Sl[(16 + 4 * j) * ld + 16];
    __builtin_amdgcn_s_setprio(3);
    double least = INFINITY, least_wanted = INFINITY;
    double e1[4];   // squares of the next block's vectors 4 j + kq, ahead of their use
#pragma unroll
    for (int j = 0; j < 4; ++j) e1[j] = S[(size_t)(4 * j + kq) * (ld + 1)];
    for (int k = 0;; ++k) {
      double e0[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        e0[j] = e1[j];
        e1[j] = S[(size_t)(16 * min(k + 1, nb - 1) + 4 * j + kq) * (ld + 1)];
      }
      factor_block(a, e0, Lp + (size_t)tri_block(nb, k, k) * 256, inv, r - 16 * k, least, least_wanted);
      __syncthreads();   // B: the inverse, column k and the next diagonal block are in LDS
      if (k + 1 >= nb) break;
      if (k > 0)
#pragma unroll
        for (int j = 0; j < 4; ++j) d[j] = next[j][lane];
      double x4[4], iv[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) { x4[t] = col[k + 1][sub * 17 + 4 * t + kq]; iv[t] = inv[lane * 4 + t]; }
      f64x4 x = {0.0, 0.0, 0.0, 0.0}, y = {0.0, 0.0, 0.0, 0.0};
      x = __builtin_amdgcn_mfma_f64_16x16x4f64(x4[0], iv[0], x, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f64_16x16x4f64(x4[1], iv[1], y, 0, 0, 0);
      x = __builtin_amdgcn_mfma_f64_16x16x4f64(x4[2], iv[2], x, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f64_16x16x4f64(x4[3], iv[3], y, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) sol[k + 1][op_index(4 * j + kq, sub)] = x[j] + y[j];
      __syncthreads();   // A: column k times the inverse is in LDS
      double l4[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) l4[t] = sol[k + 1][lane * 4 + t];
      y = f64x4{0.0, 0.0, 0.0, 0.0};
      d = __builtin_amdgcn_mfma_f64_16x16x4f64(l4[0], l4[0], d, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f64_16x16x4f64(l4[1], l4[1], y, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f64_16x16x4f64(l4[2], l4[2], d, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f64_16x16x4f64(l4[3], l4[3], y, 0, 0, 0);
      double* dst = Lp + (size_t)tri_block(nb, k + 1, k) * 256 + lane * 4;
#pragma unroll
      for (int t = 0; t < 4; ++t) dst[t] = -l4[t];
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = -(d[j] + y[j]);
    }
    if (shift) {
      least = fmin(least, shfl_xor_f64(least, 16));
      least = fmin(least, shfl_xor_f64(least, 32));
      least_wanted = fmin(least_wanted, shfl_xor_f64(least_wanted, 16));
      least_wanted = fmin(least_wanted, shfl_xor_f64(least_wanted, 32));
      double longest = 0.0;
      for (int i = lane; i < ld; i += kWave) longest = fmax(longest, S[(size_t)i * (ld + 1)]);
      longest = wave_max_f64(longest);
      if (lane == 0) {
        // (the root first: its exponent is the vector's; zeros and what is not finite are left as they are)
        const bool finite = longest > 0.0 && longest < INFINITY;
        // (squares of entries; infinity: no vector but zeros)
        const bool shifts = least > 0.0 && least < INFINITY && least_wanted >= kShiftRatio * kShiftRatio * least;
        shift[blockIdx.x] = {shifts ? sqrt(least) : 0.0,
                             finite ? ldexp(1.0, -__builtin_amdgcn_frexp_exp(sqrt(longest))) : 1.0};
        const double x = longest / least;   // squared ratio
        const int steps = !(least > 0.0 && least < INFINITY) ? 1 : x * x * x <= 1e26 ? 3 : x * x <= 1e26 ? 2 : 1;
        pause[blockIdx.x] = steps | (shifts ? 0 : kMoreSteps);
      }
    }
    return;
  }
  f64x4 acc[NBW];   // the negatives of the trailing blocks
  int bi[NBW], bk[NBW];
  // (few instructions per load: this runs once, and fetching the code is what it waits for)
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int x = __builtin_amdgcn_readfirstlane(place[wave - 1][t]);
    bi[t] = x >> 8; bk[t] = x & 255;
    const double* p = Sl + (bk[t] < nb ? 16 * (bi[t] * ld + bk[t]) : 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[t][j] = -p[4 * j * ld];
  }
  for (int k = 0;; ++k) {
    __syncthreads();   // B
    if (k + 1 >= nb) break;
    // L(i, k) = A(i, k) inv^T
    for (int i = k + 1 + wave; i < nb; i += 7) {
      double a[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) a[t] = col[i][sub * 17 + 4 * t + kq];
      f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int t = 0; t < 4; ++t) x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], inv[lane * 4 + t], x, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) sol[i][op_index(4 * j + kq, sub)] = x[j];
      double* dst = Lp + (size_t)tri_block(nb, i, k) * 256;
#pragma unroll
      for (int t = 0; t < 4; ++t) dst[lane * 4 + t] = -sol[i][lane * 4 + t];
    }
    __syncthreads();   // A
#pragma unroll
    for (int t = 0; t < NBW; ++t)
      if (bk[t] > k && bk[t] < nb) {
#pragma unroll
        for (int x = 0; x < 4; ++x)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(sol[bi[t]][lane * 4 + x], sol[bk[t]][lane * 4 + x], acc[t], 0, 0, 0);
        if (bk[t] == k + 1 && bi[t] > k + 1)
#pragma unroll
          for (int j = 0; j < 4; ++j) col[bi[t]][(4 * j + kq) * 17 + sub] = -acc[t][j];
        if (bk[t] == k + 2 && bi[t] == k + 2)
#pragma unroll
          for (int j = 0; j < 4; ++j) next[j][lane] = acc[t][j];
      }
  }
}

// X = L^-1 Y, rows of length D: four waves per 16 columns, wave w with the block rows w, w + 4, ... in accumulators.  Down the
// block rows: the owner of row k multiplies it by the inverse of the diagonal block and leaves the result in LDS -- in the
// operand layout it is in already (result register t of a lane is the row of contraction step t) --, then every wave takes
// it out of its later rows.  The blocks of the next block column are requested while the current one's instructions run.
// 192 vectors of 1024 columns: 12.5 us (one wave for all rows, 312 matrix instructions in a row: 18.5 us).
template <int NB>
__global__ __launch_bounds__(256) void trsm_kernel(const double* __restrict__ Lp, const double* __restrict__ Y,
                                                   double* __restrict__ X, int m, int nb, int D, Every every) {
  if (sequence_done(every, blockIdx.y)) return;
  if (step_left_out(every, blockIdx.y)) {   // X <- Y
    const size_t at = (size_t)blockIdx.y * m * D + blockIdx.x * 16 + (threadIdx.x & 15);
#pragma unroll 8
    for (int r = threadIdx.x >> 4; r < m; r += 16) X[at + (size_t)r * D] = Y[at + (size_t)r * D];
    return;
  }
  constexpr int NR = (NB + 3) / 4;           // block rows per wave
  __shared__ double xs[2][kWave][4];
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int sub = lane & 15, kq = lane >> 4;
  const size_t base = (size_t)blockIdx.y * m * D + blockIdx.x * 16 + sub;
  Lp += (size_t)blockIdx.y * (nb * (nb + 1) / 2) * 256 + lane * 4;
  double next[NR][4];
  auto request = [&](int k) {   // this wave's blocks of block column k (rows above it: nothing; clamped, not guarded)
#pragma unroll
    for (int x = 0; x < NR; ++x) {
      const int i = min(max(wave + 4 * x, k), nb - 1);
      const double2* p = reinterpret_cast<const double2*>(Lp + (size_t)tri_block(nb, i, k) * 256);
      const double2 lo = p[0], hi = p[1];
      next[x][0] = lo.x; next[x][1] = lo.y; next[x][2] = hi.x; next[x][3] = hi.y;
    }
  };
  request(0);
  f64x4 acc[NR];
#pragma unroll
  for (int x = 0; x < NR; ++x)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = 16 * (wave + 4 * x) + 4 * j + kq;
      const double y = Y[base + (size_t)min(r, m - 1) * D];
      acc[x][j] = r < m ? y : 0.0;
    }
  // (written out for up to 12 block rows; beyond, the code is 30 KB, which each launch fetches anew: a loop over four rows each.
  // 16 x 8K, rank 192: the call 9.59 -> 9.26 ms; as a loop with 12 rows 4 x 32K x 3072 went from 17.63 to 17.85)
  constexpr int kWritten = NB > 12 ? 1 : 4;
#pragma unroll
  for (int x0 = 0; x0 < NR; ++x0) {
#pragma unroll kWritten
    for (int w = 0; w < 4; ++w) {
      const int k = 4 * x0 + w;
      if (k >= nb) break;
      double cur[NR][4];
#pragma unroll
      for (int x = x0; x < NR; ++x)
#pragma unroll
        for (int t = 0; t < 4; ++t) cur[x][t] = next[x][t];
      request(min(k + 1, nb - 1));
      if (wave == w) {
        f64x4 v = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < 4; ++t) v = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[x0][t], acc[x0][t], v, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = 16 * k + 4 * j + kq;
          xs[k & 1][lane][j] = v[j];
          if (r < m) X[base + (size_t)r * D] = v[j];
        }
      }
      __syncthreads();   // (two buffers: the next owner writes the other one while late waves still read this one)
      double xk[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) xk[t] = xs[k & 1][lane][t];
#pragma unroll
      for (int x = x0; x < NR; ++x)
        if (wave + 4 * x > k && wave + 4 * x < nb)
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[x][t], xk[t], acc[x], 0, 0, 0);
    }
  }
}

// ---- eigenvectors of a small symmetric matrix: one-sided Jacobi in blocks ----------------------------------
// Columns of W (initially T; column p is the row W[p*mp ...] in memory) are rotated until they are orthogonal, the same
// rotations accumulated in V: then the norms of W's columns are the eigenvalues of T and the columns of V its eigenvectors.
// The columns are taken as nb = mp / 16 blocks; a step pairs the blocks up (circle method: (nb-1, st), ((st+i) mod (nb-1),
// (st-i) mod (nb-1))), and a workgroup makes the 16 x 16 pairs of columns between its two blocks orthogonal (in the first
// step of a sweep and ahead of the sweeps all pairs of its 32 columns): it forms the 32 x 32 products of the columns on the
// matrix instruction, rotates those (two-sided, in LDS, 16 disjoint rotations at a time, accumulated in J) and applies J to
// its columns as one product.  A rotation's angle thus costs two rounds of LDS and a barrier, not a pass over the columns and
// a launch: a sweep of 192 columns is 11 launches of 15 us (the first 22, those without a rotation 6) where a launch per set of
// 96 single rotations took 191 of 4.5 us.  In all 0.68 ms for one sequence, 1.0 with six sweeps and no passes ahead of them, 8.1
// with single rotations.
// V is not needed before the end: its product with J is done by other workgroups of the next step's launch.
// A sweep in which every cosine met was below kJacobiDone needs no successor (what is left is its square): the launches of
// the later ones end at once.  sweep_max [batch][sweeps]: the largest cosine of each sweep (its bits; cosines are >= 0).
constexpr float kJacobiDone = 1e-10f;
__device__ __forceinline__ bool jacobi_active(const int32_t* sweep_max, int sweep) {
  // (a stored cosine that is not a number counts as not done)
  return sweep == 0 || !(__int_as_float(sweep_max[sweep - 1]) < kJacobiDone);
}
// (c, s) of the rotation that makes two columns with squares al, be and product ga orthogonal: tan 2 theta = 2 ga / (be - al),
// |theta| <= pi / 4, through cos 2 theta and two reciprocal square roots; the exponent is taken out first.
__device__ __forceinline__ void rotation(double al, double be, double ga, double& c, double& s) {
  double d = be - al, g = 2.0 * ga;
  const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(d), fabs(g)));
  d = __builtin_amdgcn_ldexp(d, ex); g = __builtin_amdgcn_ldexp(g, ex);   // the larger in [1/2, 1], or both 0
  const double h2 = fma(d, d, g * g), r = rsqrt_f64(h2);
  const double c2 = fma(0.5 * fabs(d), r, 0.5), rc = rsqrt_f64(c2), sn = 0.5 * g * r * rc;
  c = h2 == 0.0 ? 1.0 : c2 * rc;
  s = h2 == 0.0 ? 0.0 : d < 0.0 ? -sn : sn;
}
// lane J of each row of 16 in all lanes of the row
template <int J>
__device__ __forceinline__ double row_lane_f64(double x) {
  return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(x), 0x150 + J, 0xf, 0xf, true));
}
// Ahead of the sweeps come passes over neighbouring blocks only, all pairs of 32 columns each, in two steps a pass: after
// the subspace iteration T is a matrix whose entries fall off fast from the diagonal, so these settle most of it and spare more
// sweeps (of nb - 1 steps) than they cost.  Whole calls, 1 x 8K x 1024, us without and with one, two, three, four passes:
//   exp(-i / 40): 56 vectors 962 / 970 / 973 / 991 / 1018, 96 1180 / 1164 / 1146 / 1143 / 1181, 120 1407 / 1362 / 1321 / 1313 /
//     1349, 160 1657 / 1593 / 1522 / 1499 / 1531, 192 1911 / 1833 / 1726 / 1686 / 1732, 288 3973 / 3758 / 3566 / 3401 / 3446
//   exp(-i / 100): 96 1300 / 1291 / 1270 / 1289 / 1331, 128 1530 / 1485 / 1452 / 1473 / 1503, 192 2172 / 2020 / 1938 / 1952 / 1981
//   flat: 96 1436 / 1479 / 1476 / 1519 / 1555, 128 1767 / 1757 / 1791 / 1771 / 1819, 192 2571 / 2526 / 2573 / 2617 / 2623
// After a first pass without a cosine above kLocalWorth (flat spectra, which take nine sweeps either way) the others are left out.
constexpr float kLocalWorth = 1e-3f;
__host__ __device__ __forceinline__ int local_steps(int nb) { return nb >= 10 ? 6 : nb >= 8 ? 4 : 0; }
// local_max [batch]: the largest cosine of the first of them, as in sweep_max.
// step = local step, then local_steps(nb) + sweep * (nb - 1) + st.  Workgroups [0, nb/2): step `step` on W (none when step ==
// n_steps); [nb/2, nb): the step before, on V.  J and idle (whether its J is the identity) alternate between two halves from step to step.
// A round in which every pair is orthogonal to rounding at the start of the step is left out.
__global__ __launch_bounds__(512) void jacobi_block_kernel(double* __restrict__ W, double* __restrict__ V,
                                                           double* __restrict__ Jbuf, int32_t* __restrict__ idle,
                                                           int32_t* __restrict__ sweep_max, int32_t* __restrict__ local_max,
                                                           int mp, int step, int n_steps, int n_sweeps) {
  constexpr int P = 33;                     // pitch of the 32 x 32 matrices in LDS
  __shared__ double red[8 * 3 * 256];       // partial products of the waves; then the second copy of S, and J
  __shared__ double S0[32 * P];
  __shared__ uint2 found[8];                // largest cosine and rounds of each wave's pairs
  __shared__ double2 cs[2][16];             // rotations of the last two rounds
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int sub = lane & 15, kq = lane >> 4;
  const int nb = mp / 16, np = nb / 2, b = blockIdx.y, batch = gridDim.y;
  const bool on_v = (int)blockIdx.x >= np;
  const int mine = on_v ? step - 1 : step, pair = on_v ? blockIdx.x - np : blockIdx.x;
  if (mine < 0 || mine >= n_steps) return;
  const int n_local = local_steps(nb);
  const bool local = mine < n_local;
  const int sweep = local ? 0 : (mine - n_local) / (nb - 1), st = local ? 0 : mine - n_local - sweep * (nb - 1);
  sweep_max += (size_t)b * n_sweeps;
  if (local) {
    // (a stored cosine that is not a number counts as worth it)
    if (mine >= 2 && __int_as_float(local_max[b]) <= kLocalWorth) return;
    if (2 * pair + (mine & 1) + 1 >= nb) return;
  } else if (!jacobi_active(sweep_max, sweep)) {
    return;
  }
  const int slot = ((mine & 1) * batch + b) * np + pair;
  double* Jg = Jbuf + (size_t)slot * 1024;
  int pb, qb;
  if (local) { pb = 2 * pair + (mine & 1); qb = pb + 1; }
  else if (pair == 0) { pb = nb - 1; qb = st; }
  else { pb = (st + pair) % (nb - 1); qb = (st - pair + (nb - 1)) % (nb - 1); }
  double* M = (on_v ? V : W) + (size_t)b * mp * mp;
  auto row = [&](int i) { return M + (size_t)((i < 16 ? pb * 16 : qb * 16 - 16) + i) * mp; };
  if (on_v && idle[slot]) return;
  // what J will be applied to: 16 entries of the 32 columns per wave at a time, the first two pieces requested ahead
  double xa[2][8];
  auto request = [&](double (&x)[8], int c0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = row(4 * t + kq)[c0 + sub];
  };
  const double* Js = Jg;                    // J, row p, column q at Js[p * pitch + q]
  int pitch = 32;
  if (!on_v) {
    // products of the 32 columns: tiles (0,0), (0,1), (1,1), the contraction dealt to the waves 8 at a time, all requested at once
    constexpr int NP = (kMaxFactorBlocks * 2 + 7) / 8;
    f64x4 g[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) g[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    const double* r0 = row(sub) + 2 * kq + 8 * wave;
    const double* r1 = row(16 + sub) + 2 * kq + 8 * wave;
    double2 x[NP], y[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (8 * (wave + 8 * i) < mp) {
        x[i] = *reinterpret_cast<const double2*>(r0 + 64 * i);
        y[i] = *reinterpret_cast<const double2*>(r1 + 64 * i);
      }
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (8 * (wave + 8 * i) < mp) {
        g[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i].x, x[i].x, g[0], 0, 0, 0);
        g[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i].x, y[i].x, g[1], 0, 0, 0);
        g[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[i].x, y[i].x, g[2], 0, 0, 0);
        g[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i].y, x[i].y, g[0], 0, 0, 0);
        g[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i].y, y[i].y, g[1], 0, 0, 0);
        g[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[i].y, y[i].y, g[2], 0, 0, 0);
      }
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) red[(wave * 3 + t) * 256 + (4 * j + kq) * 16 + sub] = g[t][j];
    if (16 * wave < mp) request(xa[0], 16 * wave);
    if (16 * (wave + 8) < mp) request(xa[1], 16 * (wave + 8));
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * 256; i += 512) {
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < 8; ++w) v += red[w * 768 + i];
      const int t = i >> 8, r = (i >> 4) & 15, c = i & 15;
      if (t == 0) S0[r * P + c] = v;
      if (t == 1) { S0[r * P + 16 + c] = v; S0[(16 + c) * P + r] = v; }
      if (t == 2) S0[(16 + r) * P + 16 + c] = v;
    }
    __syncthreads();
    // largest cosine among the pairs this step is about, and the rounds in which there is something to rotate
    uint32_t big = 0, rounds = 0;           // (cosines are >= 0: their bits are in their order, not-a-numbers above all)
    for (int i = threadIdx.x; i < 1024; i += 512) {
      const int r = i >> 5, c = i & 31;
      const double ga = fabs(S0[r * P + c]), al = S0[r * P + r], be = S0[c * P + c];
      if (r < c && (st == 0 || (r < 16 && c >= 16)) && !(ga <= 1e-300)) {
        const float x = (float)(ga * rsqrt_f64(al) * rsqrt_f64(be));
        big = max(big, __float_as_uint(x));
        // (the round of a pair, see members below: (c - r) mod 16, or with 31 the other one, else half the sum mod 31)
        if (!(x <= 2e-16f)) rounds |= 1u << (st != 0 ? (c - r) & 15 : c == 31 ? r : (r + c) * 16 % 31);
      }
    }
    big = wave_max_u32(big);
    rounds = wave_or_u32(rounds);
    if (lane == 0) found[wave] = make_uint2(big, rounds);
    double* S1 = red;                      // (the partial products have been read)
    double* J = red + 32 * P;
    for (int i = threadIdx.x; i < 32 * P; i += 512) J[i] = i / P == i % P ? 1.0 : 0.0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 8; ++w) { const uint2 f = found[w]; big = max(big, f.x); rounds |= f.y; }
    rounds = (uint32_t)__builtin_amdgcn_readfirstlane((int)rounds);
    if (threadIdx.x == 0) {
      if (!local) atomicMax(&sweep_max[sweep], (int)big);
      else if (mine < 2) atomicMax(&local_max[b], (int)big);
      idle[slot] = rounds ? 0 : 1;
    }
    if (!rounds) return;
    // the 16 disjoint pairs of round u: across the two blocks, or the circle method over all 32 columns
    auto members = [&](int u, int i, int& p, int& q) {
      if (st != 0) { p = i; q = 16 + ((i + u) & 15); }
      else if (i == 0) { p = 31; q = u; }
      else { p = u + i; p -= p >= 31 ? 31 : 0; q = u - i; q += q < 0 ? 31 : 0; }
    };
    if (wave < 4) {
      // waves 0-3 (one per SIMD) rotate S: 16 lanes take the rows of pair pu, each with the columns of another pair, the first
      // with its own, so that the rows' rotation is what lane 0 of the 16 has formed for its columns
      const int pu = wave * 4 + kq, pc = (pu + sub) & 15;
      int o[7];   // places of the pair's three products and of the four entries
      auto places = [&](int u) {
        int p, q, r, t;
        members(u, pc, p, q);
        members(u, pu, r, t);
        o[0] = p * P + p; o[1] = q * P + q; o[2] = p * P + q;
        o[3] = r * P + p; o[4] = r * P + q; o[5] = t * P + p; o[6] = t * P + q;
      };
      places(__ffs(rounds) - 1);
      const double* Sa = S0;
      double* Sb = S1;
      for (int t = 0; rounds; ++t) {
        rounds &= rounds - 1;
        const double al = Sa[o[0]], be = Sa[o[1]], ga = Sa[o[2]];
        const double pp = Sa[o[3]], pq = Sa[o[4]], qp = Sa[o[5]], qq = Sa[o[6]];
        double c, sn;
        rotation(al, be, ga, c, sn);
        if (wave == 0 && kq == 0) cs[t & 1][pc] = make_double2(c, sn);
        const double cu = row_lane_f64<0>(c), su = row_lane_f64<0>(sn);
        const double tp = cu * pp - su * qp, tq = cu * pq - su * qq, bp = su * pp + cu * qp, bq = su * pq + cu * qq;
        Sb[o[3]] = c * tp - sn * tq; Sb[o[4]] = sn * tp + c * tq;
        Sb[o[5]] = c * bp - sn * bq; Sb[o[6]] = sn * bp + c * bq;
        places((__ffs(rounds) - 1) & 31);
        __syncthreads();
        double* tmp = const_cast<double*>(Sa); Sa = Sb; Sb = tmp;
      }
    } else {
      // waves 4-7 apply the rotations of the round before to J: columns of pair sub, eight rows per wave
      double* jr = J + ((wave - 4) * 8 + kq * 2) * P;
      __syncthreads();
      for (int t = 0; rounds; ++t) {
        int p, q;
        members(__ffs(rounds) - 1, sub, p, q);
        rounds &= rounds - 1;
        const double2 r = cs[t & 1][sub];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const double x = jr[e * P + p], y = jr[e * P + q];
          jr[e * P + p] = r.x * x - r.y * y; jr[e * P + q] = r.y * x + r.x * y;
        }
        if (rounds) __syncthreads();
      }
    }
    __syncthreads();
    Js = J; pitch = P;
  } else {
    if (16 * wave < mp) request(xa[0], 16 * wave);
    if (16 * (wave + 8) < mp) request(xa[1], 16 * (wave + 8));
  }
  // new column q = sum_p J[p][q] column p
  double ja[2][8];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int t = 0; t < 8; ++t) ja[mt][t] = Js[(4 * t + kq) * pitch + 16 * mt + sub];
  auto apply = [&](int c0, bool two) {      // one piece, or two, 128 entries apart
    f64x4 y[2][2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) y[0][mt] = y[1][mt] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        y[0][mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ja[mt][t], xa[0][t], y[0][mt], 0, 0, 0);
        if (two) y[1][mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ja[mt][t], xa[1][t], y[1][mt], 0, 0, 0);
      }
#pragma unroll
    for (int x = 0; x < 2; ++x)
      if (x == 0 || two)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int j = 0; j < 4; ++j) row(16 * mt + 4 * j + kq)[c0 + 128 * x + sub] = y[x][mt][j];
  };
  if (16 * (wave + 8) < mp) apply(16 * wave, true);
  else if (16 * wave < mp) apply(16 * wave, false);
  if (16 * (wave + 16) < mp) {              // more than 256 vectors
    request(xa[0], 16 * (wave + 16));
    apply(16 * (wave + 16), false);
  }
  if (!on_v)
    for (int i = threadIdx.x; i < 1024; i += 512) Jg[i] = Js[(i >> 5) * P + (i & 31)];
}

}  // namespace skv
