// First line of the pre-filling algorithm: A, B <- SVD(K) of the pre-RoPE keys K [s, D = h_kv*d]
// of every sequence, truncated to rank r: B = Psi^T (the r leading right singular vectors), A = K Psi
// (section "High-throughput Decoding", footnote: keys are stored as K Psi and projected back with Psi^T).
//
// On the GPU the right singular vectors are the leading eigenvectors of the Gram matrix G = K^T K:
//   1. G from 8-bit digits of the keys on the integer matrix instruction, products exact (factorize_gram.hpp), or, for
//      sequences whose keys' magnitudes are too far apart for that, gram_kernel: fp64 on the fp64 matrix pipe (v_mfma_f64_16x16x4f64; the
//      products of stored elements are exact) -- the dense contraction, 2 s D^2 operations; only blocks on and above the
//      diagonal are formed, gram_finish sums the token splits and mirrors;
//   2. subspace iteration on m = r + oversample vectors (X <- orth(G X), by Cholesky factorisation of the vectors'
//      products), then one Rayleigh-Ritz step: T = X^T G X, eigenvectors of the small T by one-sided Jacobi rotations in
//      blocks, the r largest kept -- all fp64, small, one launch per dependent step (factorize_small.hpp);
//   3. sign convention (largest-magnitude component positive), B written, and A = K Psi, from digits again, entries that
//      these do not hold to 24 bits in fp64 (factorize_project.hpp), or all of a sequence in fp64 (project_kernel).
// Operand layout of v_mfma_f64_16x16x4f64 as measured on gfx950: A lane l holds (m = l % 16, k = l / 16),
// B lane l holds (n = l % 16, k = l / 16), result register j of lane l is (m = 4 j + l / 16, n = l % 16).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "factorize_project.hpp"
#include "factorize_small.hpp"
#include "kernels.hpp"

namespace skv {

// four consecutive stored elements, kept as stored and widened to fp64 when they are used: what a prefetch holds.
// Loads are never predicated here and in the loops below (indices are clamped instead): a load under a lane mask made the
// compiler wait for it before the matrix instructions it was meant to overlap.
template <int EB>
struct Raw4 {
  uint32_t w[EB == 2 ? 2 : 1];
  __device__ __forceinline__ void load(const uint8_t* p) {
    if constexpr (EB == 2) {
      const uint2 v = *reinterpret_cast<const uint2*>(p);
      w[0] = v.x; w[1] = v.y;
    } else {
      w[0] = *reinterpret_cast<const uint32_t*>(p);
    }
  }
  __device__ __forceinline__ void widen(double (&x)[4]) const {
    float f[4];
    if constexpr (EB == 2) { f[0] = bf16_lo(w[0]); f[1] = bf16_hi(w[0]); f[2] = bf16_lo(w[1]); f[3] = bf16_hi(w[1]); }
    else e5m2x4_to_f32(w[0], f);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = (double)f[e];
  }
};

// ---- 1. Gram matrix ---------------------------------------------------------------------------------
// WK waves per (pair of 64-column blocks bi <= bj, token split, sequence), which take 16 tokens in turn and add their sums up
// through LDS: the splits suit the digits' products, a sequence of these needs more waves.  Tile (mt, nt) of the 64 x 64
// block holds columns i0 + 4 m + mt against j0 + 4 n + nt, so that a lane's four consecutive columns feed
// four tiles and every load is 8 (or 4) contiguous bytes.  part [split][b][pair][64][64] fp64: the blocks bi <= bj packed,
// a little over half of D x D.
// Only for sequences whose flag is raised (gram_digits_kernel forms the others' sums).
// Bound by the matrix pipe: 67 TFLOP/s at 16 x 128K x 1024 (a large library product reaches 73; 61 with loads under lane
// masks, whose results the matrix instructions then waited for).
template <int EB, int WK>
__global__ __launch_bounds__(64 * WK, 2) void gram_kernel(const void* __restrict__ K, double* __restrict__ part,
                                                     const int32_t* __restrict__ flags, int s, int D, int nb,
                                                     int tokens_per_split, int batch) {
  __shared__ double red[WK > 1 ? WK / 2 : 1][WK > 1 ? 64 : 1][64];   // [wave][register][lane]
  if (!flags[blockIdx.z]) return;
  const int wk = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x & (kWave - 1), mrow = lane & 15, kq = lane >> 4;
  // pair index -> (bi, bj), bi <= bj, row by row of the upper triangle (upper_block the other way round)
  int p = blockIdx.x, bi = 0;
  while (p >= nb - bi) { p -= nb - bi; ++bi; }
  const int bj = bi + p;
  const int split = blockIdx.y, b = blockIdx.z;
  const int t_begin = split * tokens_per_split, t_end = min(s, t_begin + tokens_per_split);
  // columns past the end repeat the last four; their results are not written
  const int ci = min(bi * 64 + 4 * mrow, D - 4), cj = min(bj * 64 + 4 * mrow, D - 4);
  const uint8_t* Kb = static_cast<const uint8_t*>(K) + (size_t)b * s * D * EB;

  f64x4 acc[4][4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = f64x4{0.0, 0.0, 0.0, 0.0};

  // 16 tokens (four matrix steps) per iteration; the next iteration's rows are requested before this one's 64
  // matrix instructions, which is longer than a load takes
  constexpr int PF = 4;
  Raw4<EB> an[PF], bn[PF];
  auto request = [&](int t0) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const uint8_t* row = Kb + (size_t)min(t0 + 4 * u + kq, s - 1) * D * EB;
      an[u].load(row + ci * EB);
      bn[u].load(row + cj * EB);
    }
  };
  request(t_begin + 4 * PF * wk);
  for (int t0 = t_begin + 4 * PF * wk; t0 < t_end; t0 += 4 * PF * WK) {
    Raw4<EB> ac[PF], bc[PF];
#pragma unroll
    for (int u = 0; u < PF; ++u) { ac[u] = an[u]; bc[u] = bn[u]; }
    request(t0 + 4 * PF * WK);
    if (t0 + 4 * PF > t_end) {   // fewer than 16 tokens left: the ones past the end count as zero
#pragma unroll
      for (int u = 0; u < PF; ++u)
        if (t0 + 4 * u + kq >= t_end)
#pragma unroll
          for (int x = 0; x < (EB == 2 ? 2 : 1); ++x) { ac[u].w[x] = 0u; bc[u].w[x] = 0u; }
    }
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      double a[4], bb[4];
      ac[u].widen(a);
      bc[u].widen(bb);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[mt], bb[nt], acc[mt][nt], 0, 0, 0);
    }
  }
  // the upper half of the waves hands its sums to the lower half, until one is left
#pragma unroll
  for (int w = WK / 2; w >= 1; w /= 2) {
    if (wk >= w && wk < 2 * w)
#pragma unroll
      for (int x = 0; x < 64; ++x) red[wk - w][x][lane] = acc[x >> 4][x >> 2 & 3][x & 3];
    __syncthreads();
    if (wk < w)
#pragma unroll
      for (int x = 0; x < 64; ++x) acc[x >> 4][x >> 2 & 3][x & 3] += red[wk][x][lane];
    if (w > 1) __syncthreads();
  }
  if (wk > 0) return;
  double* out = part + (((size_t)split * batch + b) * gridDim.x + blockIdx.x) * 4096;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = 4 * (4 * j + kq) + mt, x = 4 * mrow + nt;
        if (bi * 64 + i < D && bj * 64 + x < D) out[i * 64 + x] = acc[mt][nt][j];
      }
}

// ---- 2. small fp64 linear algebra --------------------------------------------------------------------
// start vectors: Xt[b][i][x] uniform in (-1, 1) from a counter-based hash (same numbers on every run)
__global__ __launch_bounds__(256) void subspace_init_kernel(double* __restrict__ Xt, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  uint64_t z = (i + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  Xt[i] = (double)(int64_t)(z >> 11) * (1.0 / 4503599627370496.0) - 1.0;  // 53 bits -> [-1, 1)
}

// before the Jacobi sweeps: V <- identity (mp x mp per sequence), the largest cosine of every sweep <- 0
__global__ __launch_bounds__(256) void jacobi_init_kernel(double* __restrict__ V, int32_t* __restrict__ sweep_max,
                                                          int32_t* __restrict__ local_max, int mp, int n_sweeps) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < (size_t)n_sweeps) sweep_max[(size_t)blockIdx.y * n_sweeps + i] = 0;
  if (i == 0) local_max[blockIdx.y] = 0;
  if (i >= (size_t)mp * mp) return;
  V[(size_t)blockIdx.y * mp * mp + i] = (i / mp == i % mp) ? 1.0 : 0.0;
}

// order [r]: the columns of W with the largest norms (ties: lower index), strongest first.  A wave per column for the
// norms, then every column counts the ones before it.
__global__ __launch_bounds__(1024) void ritz_select_kernel(const double* __restrict__ W, int32_t* __restrict__ order,
                                                           double* __restrict__ sigma_out, int mp, int m, int r) {
  extern __shared__ double nrm[];  // [m]
  const int b = blockIdx.x, lane = threadIdx.x & (kWave - 1);
  for (int p = threadIdx.x / kWave; p < m; p += 1024 / kWave) {
    const double* w = W + ((size_t)b * mp + p) * mp;
    double n = 0.0;
    for (int x = lane; x < mp; x += kWave) n = fma(w[x], w[x], n);
    n = wave_sum_f64(n);
    if (lane == 0) nrm[p] = n;
  }
  // (norms that are not numbers have no place in the order: every entry is a valid column whatever the input)
  for (int p = threadIdx.x; p < r; p += 1024) order[(size_t)b * r + p] = p;
  __syncthreads();
  for (int p = threadIdx.x; p < m; p += 1024) {
    int rank = 0;
    for (int o = 0; o < m; ++o) rank += (nrm[o] > nrm[p]) || (nrm[o] == nrm[p] && o < p);
    if (rank < r) {
      order[(size_t)b * r + rank] = p;
      if (sigma_out) sigma_out[(size_t)b * r + rank] = sqrt(sqrt(nrm[p]));  // |column| = eigenvalue of G = sigma^2
    }
  }
}

// sign convention and B: the component of largest magnitude of every right singular vector is made positive
// (ties: lowest index); Psi_t [b][r][D] is updated in place, B [b][h_kv][r][d] is its rounding to storage
template <int EB>
__global__ __launch_bounds__(256) void emit_b_kernel(double* __restrict__ Psi_t, void* __restrict__ Bout, int D, int r,
                                                     int hkv, int d) {
  __shared__ double sv[4];
  __shared__ int si[4];
  const int rho = blockIdx.x, b = blockIdx.y;
  double* v = Psi_t + ((size_t)b * r + rho) * D;
  double best = -1.0;
  int at = 0;
  for (int x = threadIdx.x; x < D; x += 256) { const double a = fabs(v[x]); if (a > best) { best = a; at = x; } }
#pragma unroll
  for (int msk = 32; msk >= 1; msk >>= 1) {
    const double ob = shfl_xor_f64(best, msk);
    const int oa = __shfl_xor(at, msk, kWave);
    if (ob > best || (ob == best && oa < at)) { best = ob; at = oa; }
  }
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = best; si[threadIdx.x >> 6] = at; }
  __syncthreads();
  best = sv[0]; at = si[0];
  for (int w = 1; w < 4; ++w) if (sv[w] > best || (sv[w] == best && si[w] < at)) { best = sv[w]; at = si[w]; }
  const double sign = v[at] < 0.0 ? -1.0 : 1.0;
  __syncthreads();
  for (int x = threadIdx.x; x < D; x += 256) {
    const double val = sign * v[x];
    v[x] = val;
    const int h = x / d, xx = x - h * d;
    kv_store_elem<EB>(Bout, (((size_t)b * hkv + h) * r + rho) * d + xx, val);
  }
}

// ---- 3. A = K Psi -----------------------------------------------------------------------------------------
// For sequences whose flag is raised (project_digits_kernel takes the others), and keys wider than 32768.
// One wave per (32 tokens, 16 NT rank columns, sequence): M = tokens (two 16-row tiles), N = rank index, contraction over
// the key columns (a lane's four consecutive stored elements are four contraction steps).  Every fragment of Psi read
// from L2 serves both token tiles; two tiles and not three so that two waves share a SIMD and one widens while the
// other's matrix instructions run.  16 x 128K x 1024, rank 160: 13.4 ms with three tiles and a lane's columns in one
// 32-byte piece (a quarter of each line of Psi used per step, the rest evicted before its turn), 12.2 ms with loads under lane
// masks, 11.4 ms now (60 TFLOP/s); one sequence of 32K 307 -> 195 us.
template <int EB, int NT>
__global__ __launch_bounds__(64, 2) void project_kernel(const void* __restrict__ K, const double* __restrict__ Psi_t,
                                                     void* __restrict__ Aout, const int32_t* __restrict__ flags, int s,
                                                     int s_cap, int D, int r) {
  if (flags && !flags[blockIdx.z]) return;
  constexpr int MT = 2;
  const int lane = threadIdx.x, mrow = lane & 15, kq = lane >> 4;
  const int tok0 = blockIdx.x * (16 * MT), n0 = blockIdx.y * (16 * NT), b = blockIdx.z;
  const uint8_t* krow[MT];   // tokens and ranks past the end repeat the last real one; their results are not written
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    krow[mt] = static_cast<const uint8_t*>(K) + ((size_t)b * s + min(tok0 + 16 * mt + mrow, s - 1)) * D * EB;
  f64x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f64x4{0.0, 0.0, 0.0, 0.0};
  const double* prow[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) prow[nt] = Psi_t + ((size_t)b * r + min(n0 + 16 * nt + mrow, r - 1)) * D;
  // The contraction runs over 64 key columns per outer step, 16 per inner step: lane group kq takes columns 4 kq .. + 3 of the
  // 16, so that what a wave reads of a row of Psi in one step is one whole cache line.  The token rows are requested a
  // whole outer step ahead (they come from HBM), the Psi fragments of the next inner step (from L2) before the matrix
  // instructions of the current one.
  Raw4<EB> kn[MT][4];
  double pn[NT][4];
  auto request_k = [&](int c0) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        kn[mt][u].load(krow[mt] + min(c0 + 16 * u + 4 * kq, D - 4) * EB);
      }
  };
  auto request_psi = [&](int col) {   // col = first of this lane group's four columns
    col = min(col, D - 4);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const double2 lo = *reinterpret_cast<const double2*>(prow[nt] + col), hi = *reinterpret_cast<const double2*>(prow[nt] + col + 2);
      pn[nt][0] = lo.x; pn[nt][1] = lo.y; pn[nt][2] = hi.x; pn[nt][3] = hi.y;
    }
  };
  request_k(0);
  request_psi(4 * kq);
#pragma unroll 1
  for (int c0 = 0; c0 < D; c0 += 64) {
    Raw4<EB> kc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int u = 0; u < 4; ++u) kc[mt][u] = kn[mt][u];
    request_k(c0 + 64);
    auto inner = [&](auto u_tag, int next_col) {
      constexpr int U = decltype(u_tag)::value;
      double a[MT][4], pb[NT][4];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) kc[mt][U].widen(a[mt]);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e) pb[nt][e] = pn[nt][e];
      request_psi(next_col);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[mt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[mt][e], pb[nt][e], acc[mt][nt], 0, 0, 0);
    };
    const int cb = c0 + 4 * kq;
    inner(std::integral_constant<int, 0>{}, cb + 16);
    inner(std::integral_constant<int, 1>{}, cb + 32);
    if (c0 + 32 < D) {   // (the key width is a multiple of 32)
      inner(std::integral_constant<int, 2>{}, cb + 48);
      inner(std::integral_constant<int, 3>{}, cb + 64);
    }
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = tok0 + 16 * mt + 4 * j + kq, rho = n0 + 16 * nt + mrow;
        if (t < s && rho < r) kv_store_elem<EB>(Aout, ((size_t)b * s_cap + t) * r + rho, acc[mt][nt][j]);
      }
}

// ---- launch sequence ----------------------------------------------------------------------------------------
// C (Mw x Nw, zero outside M x N) = A B, see gemm64_kernel; ?.ld = elements from row to row, ?.stride = from sequence to
// sequence.  Fewer than 64 tiles of 32 x 32 (the m x m products of one sequence): 16 x 16 tiles, the contraction cut in
// 16 (192 x 192 x 1024: 9.9 us, cut in four 11.7, 18.5 us on 36 tiles of 32 x 32).  Up to 1024: 32 x 32 tiles with the
// contraction cut eight ways (192 x 1024 x 1024 takes 19.6 us for one sequence, 211 us with a tile per workgroup on the vector
// unit).  More: 64 x 64 blocks, the contraction cut in four, a wave's 16 tiles of 16 x 16 in 413 registers: half the reads
// from L2 of 2 x 2 waves of 32 x 32 (16 sequences: 155 us, 185 with those; the call 25.5 -> 25.0 ms, 6 x 20K 6.0 -> 5.7,
// 4 x 32K x 3072 19.6 -> 17.9).  B by rows (one product per call) keeps the 2 x 2 waves: 34 us against 44.  The limits lie
// between shapes that were measured on both sides, 192 vectors of 1 and 16 sequences; those in between were not searched.
struct Mat { const double* p; int ld; size_t stride; };
template <bool BT>
static hipError_t gemm64(Mat A, Mat B, double* C, int ldc, size_t strideC, int M, int N, int K, int Kb, int Mw, int Nw,
                         int batch, hipStream_t st, const int32_t* a_rows = nullptr, int a_rows_stride = 0,
                         const Shift* shift = nullptr, double node = 0.0, Every every = {nullptr, 0, false}, bool lower = false) {
  const long tiles = (long)((Mw + 31) / 32) * ((Nw + 31) / 32) * batch;
#define SKV_GEMM(T_, WM_, WN_, WK_)                                                                                       \
  hipLaunchKernelGGL((gemm64_kernel<T_, WM_, WN_, WK_, BT>), dim3((Nw + 16 * T_ * WN_ - 1) / (16 * T_ * WN_),             \
                     (Mw + 16 * T_ * WM_ - 1) / (16 * T_ * WM_), batch), dim3(64 * WM_ * WN_ * WK_), 0, st, A.p, B.p, C, M, N, \
                     K, Kb, A.ld, B.ld, ldc, Mw, Nw, A.stride, B.stride, strideC, a_rows, a_rows_stride, \
                     shift, node, every, lower)
  if (tiles < 64) SKV_GEMM(1, 1, 1, 16);
  else if (tiles < 1024) SKV_GEMM(2, 1, 1, 8);
  else if constexpr (BT) SKV_GEMM(4, 1, 1, 4);
  else SKV_GEMM(2, 2, 2, 2);
#undef SKV_GEMM
  return hipGetLastError();
}

static RestLists rest_lists(char* ws, const FactorizePlan& pl) {
  return {reinterpret_cast<uint32_t*>(ws + pl.rest_where), reinterpret_cast<uint16_t*>(ws + pl.rest)};
}

// 1. G = K^T K: the digits' products, or the fp64 kernel for sequences whose flag is raised, and the sum over the splits
template <int EB>
static hipError_t launch_gram(const void* K, double* part, double* G, float* scale, int32_t* flags, uint16_t* chunk_max,
                              RestLists rest, int32_t* rest_count, int32_t* marks, uint32_t* by_col, int32_t* col_begin,
                              const FactorizePlan& pl, int batch, int s, int D, hipStream_t st) {
  const int pieces = D * EB / 16;
  hipLaunchKernelGGL(column_max_kernel<EB>, dim3(pl.n_chunks, batch, (pieces + pl.max_lv - 1) / pl.max_lv), dim3(256), 0, st, K,
                     chunk_max, flags, s, D, pl.max_lv, pl.max_chunk, pl.n_chunks);
  hipLaunchKernelGGL(column_scale_kernel<EB>, dim3(pl.nb, batch), dim3(1024), 0, st, K, chunk_max, scale, flags, s, D,
                     pl.n_chunks, pl.tokens_per_split, ((uint64_t)s << 32) / (uint32_t)std::min(s, kSample), pl.rest_share);
  constexpr int kLds = 2 * 2 * 3 * 128 * 64;   // two stages of two column blocks of three digits
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gram_digits_kernel<EB>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gram_digits_kernel<EB>, dim3((unsigned)((long)batch * pl.n_splits * (pl.nb2 * (pl.nb2 + 1) / 2))), dim3(512),
                     kLds, st, K, scale, part, rest, rest_count, marks, flags, s, D, pl.nb, pl.nb2, pl.tokens_per_split, pl.n_splits,
                     batch, pl.rest_cap, pl.n_marks);
#define SKV_GRAM64(WK_)                                                                                                  \
  hipLaunchKernelGGL((gram_kernel<EB, WK_>), dim3(pl.nb * (pl.nb + 1) / 2, pl.n_splits, batch), dim3(64 * WK_), 0, st, K, part, \
                     flags, s, D, pl.nb, pl.tokens_per_split, batch)
  if (pl.waves64 == 8) SKV_GRAM64(8); else if (pl.waves64 == 4) SKV_GRAM64(4); else if (pl.waves64 == 2) SKV_GRAM64(2); else SKV_GRAM64(1);
#undef SKV_GRAM64
  hipLaunchKernelGGL(rest_by_column_kernel, dim3(pl.nb2, batch), dim3(1024), 0, st, rest.where, rest_count, flags, by_col, col_begin, pl.nb2,
                     pl.n_splits, pl.rest_cap);
  const int nt = D / 32;   // (the key width is a multiple of 32)
  hipLaunchKernelGGL(gram_finish_kernel<EB>, dim3(nt * (nt + 1) / 2, batch), dim3(256), 0, st, part, G, K, scale, rest, by_col, col_begin,
                     flags, s, D, nt, pl.nb, pl.nb2, pl.n_splits, batch, pl.rest_cap);
  return hipGetLastError();
}

// 3. A = K Psi: digits, or the fp64 kernel for sequences whose flag is raised
template <int EB>
static hipError_t launch_project(const void* K, const double* Psi_t, void* A, char* ws, const FactorizePlan& pl, int batch, int s,
                                 int s_cap, int D, int r, hipStream_t st) {
  int32_t* flags = reinterpret_cast<int32_t*>(ws + pl.flags);
  // 32-bit sums of digits: at most 3 * 2^14 per column; and a launch has fewer than 2^32 threads, which some 4e8 tokens of
  // rank 160 would pass (project_kernel counts sequences in a dimension of their own)
  const int nt = (r + 31) / 32;
  const long blocks = (long)batch * pl.n_splits * (pl.n_marks - 1), workgroups = (blocks + 7) / 8 * 8 * nt;
  const bool digits = D <= 32768 && workgroups < 1l << 23;
  if (digits) {
    const float* scale = reinterpret_cast<const float*>(ws + pl.scale);
    uint8_t* psi_digits = reinterpret_cast<uint8_t*>(ws + pl.psi_digits);
    int32_t* exps = reinterpret_cast<int32_t*>(ws + pl.psi_exps);
    hipLaunchKernelGGL(psi_digits_kernel<EB>, dim3(32 * nt, batch), dim3(256), 0, st, Psi_t, scale, psi_digits, exps, D, r, nt);
    constexpr int kLds = 2 * kPsiDeep * kPsiStage;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&project_digits_kernel<EB>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(project_digits_kernel<EB>, dim3((unsigned)workgroups), dim3(512), kLds, st, K, psi_digits, exps,
                       Psi_t, rest_lists(ws, pl), reinterpret_cast<const int32_t*>(ws + pl.marks),
                       flags, scale, A, s, s_cap, D, r, nt, pl.nb2, pl.tokens_per_split, pl.n_splits, batch, pl.rest_cap, pl.n_marks);
  }
  // up to five 16-rank tiles per wave, the tiles dealt evenly to as few waves as that takes (rank 96: 2 x 3, not 5 + 1)
  const int tiles = (r + 15) / 16, waves = (tiles + 4) / 5, per_wave = (tiles + waves - 1) / waves;
  const dim3 grid((s + 31) / 32, waves, batch);
#define SKV_PROJECT(NT_) hipLaunchKernelGGL((project_kernel<EB, NT_>), grid, dim3(64), 0, st, K, Psi_t, A, digits ? flags : nullptr, s, s_cap, D, r)
  if (per_wave == 5) SKV_PROJECT(5); else if (per_wave == 4) SKV_PROJECT(4); else SKV_PROJECT(3);
#undef SKV_PROJECT
  return hipGetLastError();
}

FactorizePlan plan_factorize(int batch, int s, int D, int r, int oversample, int n_sweeps, int kv_bytes) {
  FactorizePlan p{};
  p.m = std::min(D, r + oversample);
  p.mp = (p.m + 31) / 32 * 32;
  p.nb = (D + 63) / 64;
  const long pairs = (long)p.nb * (p.nb + 1) / 2;
  const long blocks = pairs * batch;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  auto doubles = [&](size_t per_sequence) { return up(per_sequence * batch * 8); };
  auto split_tokens = [&](long splits) {
    p.tokens_per_split = (int)(((s + splits - 1) / splits + 15) / 16 * 16);
    p.n_splits = (s + p.tokens_per_split - 1) / p.tokens_per_split;
  };
  const size_t m = p.m, mp = p.mp, DD = (size_t)D * D, nbc = (m + 15) / 16;

  // Workspace: G, then one region that first holds the partial sums of the Gram matrix and, once G is formed, everything
  // else.  V takes G's place (G is last read by the product that forms T; mp <= D), S is W's place (last read before T is
  // written), J and Psi_t that of Lp and Yt (last read by T's products; r <= m).
  p.G = p.V = 0;
  size_t off = doubles(DD);
  p.part = p.Xt = p.psi_digits = off;
  const size_t vectors = (size_t)(r + 31) / 32 * 32;
  size_t end = off + std::max(doubles(m * D), up((size_t)batch * (vectors / 32) * ((D + 63) / 64) * kPsiStage));
  p.W = p.S = end; end += doubles(mp * mp);
  // (the shifts are last read before the sweeps)
  p.idle = p.shift = end; end += up(std::max((size_t)2 * batch * (mp / 32) * 4, m < (size_t)D ? batch * sizeof(Shift) : 0));
  p.sweep_max = end; end += up((size_t)batch * n_sweeps * 4);
  p.order = end; end += up((size_t)batch * r * 4);
  p.psi_exps = end; end += up((size_t)batch * vectors * 4);
  p.Lp = p.Jbuf = p.Psi_t = end;
  p.Yt = end + doubles(nbc * (nbc + 1) / 2 * 256);
  end = std::max(p.Yt + doubles(m * D), end + doubles(2 * (mp / 32) * 1024));
  const size_t split_bytes = (size_t)blocks * 4096 * 8;

  // What a workspace may take: programs that keep one were given room for D x D partial sums of every split, the tokens
  // split for 8192 waves, and all other arrays side by side.  That room holds about twice as many packed ones.
  // (SHADOWKV_GRAM_WAVES, a tuning override: waves aimed at)
  static const long target = [] { const char* e = getenv("SHADOWKV_GRAM_WAVES"); return e ? atol(e) : 0l; }();
  const long aim = target > 0 ? target : 8192l;
  const long aim_splits = std::max(1l, std::min((s + 1023l) / 1024, (aim + blocks - 1) / blocks));
  split_tokens(aim_splits);
  const size_t even = (m + 1) / 2 * 2;
  const size_t room = doubles(p.n_splits * DD) + doubles(DD) + 2 * doubles(m * D) + 2 * doubles(even * even) + doubles(r * m) +
                      doubles((size_t)r * D);
  // Behind these lies what the digits need: the columns' scales, the sequences' flags and the lists of what the
  // digits miss, in token order and by column, with room for three elements in 2048 (96 at least, or what the room leaves).
  p.nb2 = (D + 127) / 128;
  const long tiles = (long)p.nb2 * (p.nb2 + 1) / 2;
  auto rest_room = [&] { return std::max(64, p.tokens_per_split / 32) * 3 / 2; };   // of 32 elements a token: 128 columns, 16 of 64 tokens
  auto place = [&](long splits) {
    split_tokens(splits);
    size_t at = std::max(off + up(p.n_splits * split_bytes), end);
    const size_t lists = (size_t)batch * p.n_splits * p.nb2 * 4;
    p.scale = at; at += up((size_t)batch * D * 4);
    p.flags = at; at += up((size_t)batch * 4);
    p.col_begin = at; at += up((size_t)batch * p.nb2 * 129 * 4);
    p.rest_count = at; at += up(lists * 4);
    p.n_marks = (p.tokens_per_split + 255) / 256 + 1;
    p.marks = at; at += up(lists * p.n_marks * 4);
    const size_t left = room > at + 512 ? room - at - 512 : 0;
    // (10 bytes an entry, four of them its place in the order by column; 16 of what is left for three halves of one)
    p.rest_cap = (int)std::min<size_t>(std::max(64, p.tokens_per_split / 32), left / (lists * 16)) * 3 / 2;
    p.rest_where = at; p.by_col = p.rest_where + lists * p.rest_cap * 4; p.rest = p.by_col + lists * p.rest_cap * 4;
    at += up(lists * p.rest_cap * 10);
    return at;
  };
  // rounds of fp64 workgroups of so many waves: two waves a SIMD, or one, which takes 0.6 of the time
  auto rounds64 = [](long workgroups, int waves) {
    const long resident = 2048 / waves, rest = workgroups % resident;
    return (double)(workgroups / resident) + (rest == 0 ? 0.0 : rest <= resident / 2 && waves < 8 ? 0.6 : 1.0);
  };
  long splits = 1;
  if (target > 0) {
    splits = std::max(1l, std::min(aim_splits, (long)((room - off) / split_bytes)));
  } else {
    // The token splits that cost least: a workgroup fills a compute unit and takes 20 ns per token; where the groups of
    // tiles go round the XCDs evenly each XCD has 32 compute units for its share, otherwise all 256 share.  Every split
    // costs its partial sums once written and once read (1.06 x 8 bytes D^2 per sequence at 4.6 TB/s).  A tenth of what the
    // fp64 sums would take counts as well, so that sequences that go that way do not pay for a split that suits only the
    // others: 2048 of their waves are resident, two per SIMD, a wave takes 245 us for 1024 tokens, a round of at most one
    // wave per SIMD 0.6 of that.  More splits have to be worth half a per cent, and leave the lists their size.
    // 16 x 128K x 1024: 8 splits (digits 18 rounds, fp64 8.5; with 4 splits 9 and 4.25 rounds, the latter 40.6 against
    // 38.1 ms); 1 x 32K: 7 splits, 252 workgroups.
    double best = 0.0;
    for (long sp = 1; sp <= std::min((s + 511l) / 512, 512l); ++sp) {
      if (sp > 1 && (place(sp) > room || p.rest_cap < rest_room())) break;
      const long groups = sp * batch;
      const long rounds = groups % 8 == 0 ? (groups / 8 * tiles + 31) / 32 : (groups * tiles + 255) / 256;
      const double tokens = (double)((s + sp - 1) / sp);
      const double cost = ((double)rounds * 0.02 + 0.1 * rounds64(blocks * sp, 1) * (245.0 / 1024.0)) * tokens + (double)sp * batch * D * D * (1.06 * 8.0 / 4.6e6);
      if (sp == 1 || cost < best * 0.995) { best = cost; splits = sp; }
    }
  }
  p.total = place(splits);
  // Waves that share an fp64 block of a part, for the least rounds times tokens of a wave.  With one wave each, as many splits as
  // suit the digits left half of the chip idle: 1 x 32K x 1024 624 us with the 15 splits that the fp64 sums would choose, 1,214
  // with 7 splits and one wave, 648 with two, 636 with four; 2 x 32K x 512 344, 717, 379 and 376; 3 x 8K x 1024 460, 566, 549 and
  // 543.  Four rather than fewer where they are equal: a few sequences of a batch fill more of the chip (two of which one is
  // summed in fp64, 2 x 32K x 512: the call 4.21 ms with two waves, 4.04 with four).
  p.waves64 = 1;
  auto time64 = [&](int w) { return rounds64(blocks * p.n_splits, w) * ((p.tokens_per_split + 16 * w - 1) / (16 * w)); };
  for (int w = 2; w <= 8; w *= 2)
    if (time64(w) < (w < 8 ? 1.02 : 0.95) * time64(p.waves64)) p.waves64 = w;
  p.rest_share = std::min(1.0f / 512.0f, std::max(0.0f, (float)p.rest_cap - 4.0f * std::sqrt((float)p.rest_cap)) / (32.0f * (float)p.tokens_per_split));
  // the columns' largest elements by chunk of tokens lie where G will
  const int ne = 16 / kv_bytes, pieces = D / ne;
  p.max_lv = 1;
  while (2 * p.max_lv <= std::min(pieces, 128)) p.max_lv *= 2;
  const long column_groups = (pieces + p.max_lv - 1) / p.max_lv;
  const long chunks = std::max(1l, std::min({(2048 + batch * column_groups - 1) / (batch * column_groups), (long)(s + 63) / 64, 4l * D}));
  p.max_chunk = (int)((s + chunks - 1) / chunks);
  p.n_chunks = (s + p.max_chunk - 1) / p.max_chunk;
  return p;
}

hipError_t launch_factorize(const void* k_pre, int kv_bytes, void* A, void* B, double* psi_out, double* sigma_out,
                            char* ws, const FactorizePlan& pl, int batch, int hkv, int d, int s, int s_cap, int r,
                            int n_iter, int n_sweeps, hipStream_t st) {
  const int D = hkv * d, m = pl.m, mp = pl.mp;
  double* part = reinterpret_cast<double*>(ws + pl.part);
  double* G = reinterpret_cast<double*>(ws + pl.G);
  double* Xt = reinterpret_cast<double*>(ws + pl.Xt);
  double* Yt = reinterpret_cast<double*>(ws + pl.Yt);
  double* S = reinterpret_cast<double*>(ws + pl.S);
  double* Lp = reinterpret_cast<double*>(ws + pl.Lp);
  double* W = reinterpret_cast<double*>(ws + pl.W);
  double* V = reinterpret_cast<double*>(ws + pl.V);
  double* Jbuf = reinterpret_cast<double*>(ws + pl.Jbuf);
  int32_t* idle = reinterpret_cast<int32_t*>(ws + pl.idle);
  int32_t* sweep_max = reinterpret_cast<int32_t*>(ws + pl.sweep_max);
  int32_t* order = reinterpret_cast<int32_t*>(ws + pl.order);
  double* Psi_t = psi_out ? psi_out : reinterpret_cast<double*>(ws + pl.Psi_t);
  hipError_t e;
#define SKV_CHECK() do { e = hipGetLastError(); if (e != hipSuccess) return e; } while (0)
  // 1. G = K^T K
  {
    float* scale = reinterpret_cast<float*>(ws + pl.scale);
    int32_t* flags = reinterpret_cast<int32_t*>(ws + pl.flags);
    uint16_t* chunk_max = reinterpret_cast<uint16_t*>(ws + pl.G);
    const RestLists rest = rest_lists(ws, pl);
    int32_t* rest_count = reinterpret_cast<int32_t*>(ws + pl.rest_count);
    int32_t* marks = reinterpret_cast<int32_t*>(ws + pl.marks);
    uint32_t* by_col = reinterpret_cast<uint32_t*>(ws + pl.by_col);
    int32_t* col_begin = reinterpret_cast<int32_t*>(ws + pl.col_begin);
    e = kv_bytes == 1 ? launch_gram<1>(k_pre, part, G, scale, flags, chunk_max, rest, rest_count, marks, by_col, col_begin, pl, batch, s, D, st)
                      : launch_gram<2>(k_pre, part, G, scale, flags, chunk_max, rest, rest_count, marks, by_col, col_begin, pl, batch, s, D, st);
    if (e != hipSuccess) return e;
  }
  // 2. subspace iteration: X <- orth(G X); rows of Xt are the vectors
  const size_t nx = (size_t)batch * m * D;
  hipLaunchKernelGGL(subspace_init_kernel, dim3((unsigned)((nx + 255) / 256)), dim3(256), 0, st, Xt, nx);
  SKV_CHECK();
  // X <- orthonormal basis of the rows of Y, each row from the ones before it (see chol_kernel)
  const int nbc = (m + 15) / 16;
  // (with `every` for those sequences whose turn it is, X <- Y for the others)
  auto orthonormalise = [&](const double* Y, double* X, Shift* shift = nullptr, int32_t* pause = nullptr,
                            Every every = {nullptr, 0, false}) -> hipError_t {
    hipError_t err = gemm64<true>({Y, D, (size_t)m * D}, {Y, D, (size_t)m * D}, S, 16 * nbc, (size_t)256 * nbc * nbc, m, m, D, D, 16 * nbc, 16 * nbc, batch, st,
                                  nullptr, 0, nullptr, 0.0, every, true);
    if (err != hipSuccess) return err;
#define SKV_ORTH(NBW_, NB_)                                                                                       \
  do {                                                                                                            \
    hipLaunchKernelGGL(chol_kernel<NBW_>, dim3(batch), dim3(512), 0, st, S, Lp, nbc, r, shift, pause, every); \
    hipLaunchKernelGGL(trsm_kernel<NB_>, dim3(D / 16, batch), dim3(256), 0, st, Lp, Y, X, m, nbc, D, every);         \
  } while (0)
    // (trailing blocks per wave of seven, block rows held): up to 80, 192, 224, 288 vectors
    if (nbc <= 5) SKV_ORTH(2, 5);
    else if (nbc <= 12) SKV_ORTH(11, 12);
    else if (nbc <= 14) SKV_ORTH(14, 14);
    else SKV_ORTH(22, kMaxFactorBlocks);
#undef SKV_ORTH
    return hipGetLastError();
  };
  // Y = X (G - node shift); G is symmetric, so its rows are its columns
  auto times_gram = [&](const double* X, double* Y, const Shift* by = nullptr, double node = 0.0, Every every = {nullptr, 0, false}) {
    return gemm64<true>({X, D, (size_t)m * D}, {G, D, (size_t)D * D}, Y, D, (size_t)m * D, m, D, D, D, m, D, batch, st, nullptr, 0, by,
                        node, every);
  };
  // Steps of G alone damp what lies beyond the m vectors by lam_(m+1) / lam_r each.  By default four of these are followed by
  // nine of G - theta_j with theta_j the Chebyshev points of [0, b], b the least entry of the fourth factor's diagonal: 0.8 to
  // 1.2 lam_m on every spectrum tried, at which the nine damp like 1 / T_9(2 lam_r / b - 1).  They do so where the least of the
  // diagonal's first r entries is at least kShiftRatio = 4 times b: everything up to b is then damped by 1e-10 on top of its
  // fourth power, whatever comes after the m vectors (numpy model, 125 spectra of 256, 512 and 1024 columns, ramps and plateaus
  // that drop at any place among them: residuals up to 300 times smaller than after sixteen steps of G, or within 5e-14 lam_1 per
  // vector, which is D rounding units).  With the r-th eigenvalue closer to b the points' polynomial is not small on [0, b], and a
  // spectrum that drops there loses: 64 equal eigenvalues and the rest 0.117 of these, r = 32, residual 1.8e-4 against 1e-13.
  // Such sequences, and those where a pivot was rounding, have b = 0: nothing is shifted, and three steps more (four launches of
  // 2 us each for the others) make sixteen.  Of the nine, or twelve, every third, or second, is followed by an orthonormalisation
  // where the eigenvalues lie close enough (see chol_kernel), and the last: after four steps the vectors are near enough to single
  // eigenvectors that another step mostly scales them, so the order of the points matters to rounding only; large and small ones
  // take turns.  (Same model: the same residuals to two digits, eigenvalues from alike to 1e30 apart.  1 x 32K: 56 us for an
  // orthonormalisation, 10 for one left out.)
  constexpr int kPlain = 4, kPoints = 9, kMost = 16;
  const bool shifted = n_iter == 0 && m < D;
  Shift* shift = reinterpret_cast<Shift*>(ws + pl.shift);
  int32_t* pause = order;   // (the order is found after these steps)
  const int steps = n_iter ? n_iter : shifted ? kPlain + kPoints : kMost;
  for (int it = 0; it < steps; ++it) {
    const int j = shifted ? it - kPlain : -1;
    const double node = 0.5 - 0.5 * std::cos(3.14159265358979323846 * (2 * (4 * j % kPoints) + 1) / (2 * kPoints));
    if ((e = j < 0 ? times_gram(Xt, Yt) : times_gram(Xt, Yt, shift, node)) != hipSuccess) return e;
    const bool pauses = j >= 0 && it + 1 < steps;
    if ((e = orthonormalise(Yt, Xt, j == -1 && shifted ? shift : nullptr, pause, {pauses ? pause : nullptr, j + 1, false})) != hipSuccess) return e;
  }
  for (int it = steps; shifted && it < kMost; ++it) {   // sequences without a shift
    if ((e = times_gram(Xt, Yt, shift, 0.0, {pause, 0, true})) != hipSuccess) return e;
    if ((e = orthonormalise(Yt, Xt, nullptr, nullptr, {pause, it - kPlain + 1, true})) != hipSuccess) return e;
  }
  // twice more before the Ritz step: the first brings the basis to the rounding unit, the second does the same for
  // vectors whose pivots were rounding in the one before
  if ((e = orthonormalise(Xt, Yt)) != hipSuccess) return e;
  if ((e = orthonormalise(Yt, Xt)) != hipSuccess) return e;
  // Rayleigh-Ritz: T = X^T G X = Xt (Xt G)^T
  if ((e = times_gram(Xt, Yt)) != hipSuccess) return e;
  {
    // W [mp x mp]: T(i, j) = sum_x Xt[i][x] Yt[j][x], zero outside the leading m x m block
    if ((e = gemm64<true>({Xt, D, (size_t)m * D}, {Yt, D, (size_t)m * D}, W, mp, (size_t)mp * mp, m, m, D, D, mp, mp, batch, st)) != hipSuccess)
      return e;
    int32_t* local_max = order;   // (the order is found after the sweeps)
    hipLaunchKernelGGL(jacobi_init_kernel, dim3((unsigned)(((size_t)mp * mp + 255) / 256), batch), dim3(256), 0, st, V, sweep_max,
                       local_max, mp, n_sweeps);
    SKV_CHECK();
    const int nbj = mp / 16, n_steps = local_steps(nbj) + n_sweeps * (nbj - 1);
    for (int step = 0; step <= n_steps; ++step)   // (the last launch only brings V up to date)
      hipLaunchKernelGGL(jacobi_block_kernel, dim3(nbj, batch), dim3(512), 0, st, W, V, Jbuf, idle, sweep_max, local_max, mp, step,
                         n_steps, n_sweeps);
    SKV_CHECK();
    hipLaunchKernelGGL(ritz_select_kernel, dim3(batch), dim3(1024), (size_t)m * sizeof(double), st, W, order, sigma_out, mp, m, r);
    SKV_CHECK();
  }
  // Psi_t [r x D] = (the chosen columns of V)^T [r x mp] Xt [m x D]; V is zero in those rows beyond m
  if ((e = gemm64<false>({V, mp, (size_t)mp * mp}, {Xt, D, (size_t)m * D}, Psi_t, D, (size_t)r * D, r, D, mp, m, r, D, batch, st,
                         order, r)) != hipSuccess)
    return e;
  // 3. sign convention, B, A = K Psi
  if (kv_bytes == 1) hipLaunchKernelGGL(emit_b_kernel<1>, dim3(r, batch), dim3(256), 0, st, Psi_t, B, D, r, hkv, d);
  else hipLaunchKernelGGL(emit_b_kernel<2>, dim3(r, batch), dim3(256), 0, st, Psi_t, B, D, r, hkv, d);
  SKV_CHECK();
  e = kv_bytes == 1 ? launch_project<1>(k_pre, Psi_t, A, ws, pl, batch, s, s_cap, D, r, st)
                    : launch_project<2>(k_pre, Psi_t, A, ws, pl, batch, s, s_cap, D, r, st);
  if (e != hipSuccess) return e;
#undef SKV_CHECK
  return hipSuccess;
}

}  // namespace skv
