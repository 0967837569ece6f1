// Landmark scoring: P = Q L^T * scale for every landmark slot (first line of the
// decoding algorithm), streamed once from HBM for the heads of a KV group (up to four here, up to 16 per pass in
// score_kernel_g16 further down).
//
// The scores decide an index set that has to match an fp64 reference: the logit is the
// plain dot product of the bf16 inputs, so the inputs are widened to fp64 and contracted on
// the fp64 matrix pipe (v_mfma_f64_4x4x4f64: four independent 4x4x4 blocks per wave, 256 FMAs
// per issue, no cross-lane reduction needed); the products are exact and the fp64 sum does
// not depend on the order of summation beyond its last bit.  The per-tile softmax statistics
// are formed from the fp64 logits.  What is stored for the selection is the logit rounded once
// to fp32 (half the bytes): the selection searches on those and settles its boundary on logits
// it forms again in fp64, so the rounding never decides a rank.  The vector ALU only unpacks
// and converts, which leaves the kernel bound by the HBM read of L.
//
// Operand layout of the instruction, as measured on gfx950: input lane
// = 16*k + 4*block + (i for A | j for B), result lane = 16*i + 4*block + j.
// Here i = query head (4), j = landmark row inside the block (4 blocks = 16 rows),
// k = which 16-byte piece of each 64-byte row segment the lane loads.  A wave covers
// NT 16-row tiles (one, two or four, see score_tiles; all loads issued before the first MFMA), a workgroup
// four times as many.
// Result lane 16*i + r holds the logit of head i, row r of the tile: it stores it
// (16 consecutive floats per head) and keeps the fp64 value until the wave's tiles are
// done, when its rows' (max, sum exp) are formed at once (row16_lse) and merged over the
// workgroup; the selection kernel makes each head's log-sum-exp of these.
#include "kernels.hpp"

namespace skv {

// exp(x) for x <= 0 through the fp32 exp2 unit.  It only feeds the softmax normaliser (a sum of
// such terms kept in fp64): its ~1e-7 relative error moves a head's log-sum-exp by ~1e-7, an
// order below the 1e-6 at which two scores count as tied; the logits themselves stay fp64.
__device__ __forceinline__ double exp_neg(double x) {
  return (double)__builtin_amdgcn_exp2f((float)(x * 1.4426950408889634074));
}

// (m, s) <- (m, s) (+) (m2, s2) for s = sum exp(p - m)
__device__ __forceinline__ void lse_merge(double& m, double& s, double m2, double s2) {
  if (m2 == -INFINITY) return;
  if (m == -INFINITY) { m = m2; s = s2; return; }
  const double e = exp_neg(-fabs(m - m2));
  if (m2 > m) { s = s * e + s2; m = m2; } else { s += s2 * e; }
}

// (max, sum exp(p - max)) over NT values per lane and the 16 lanes of a row, in every lane of the row.  One maximum first,
// then every value against it: no branches and one exponential per value (merging (m, s) pairs value by value took a
// branch each, a third of the kernel's vector instructions with FP8 landmarks: 83 us against 77 at 16 x 128K, and 41 against
// 32 for one sequence of 1M tokens with 16 heads per group).  A value equal to the maximum counts 1; rows that do not exist
// carry -inf and count 0.  (Infinite logits end as NaN: where two waves meet the same one, lse_merge subtracts it from itself.)
template <int NT>
__device__ __forceinline__ void row16_lse(const double (&p)[NT], double& M, double& S) {
  M = p[0];
  if constexpr (NT >= 2) M = fmax(M, p[1]);
  if constexpr (NT == 4) M = fmax(M, fmax(p[2], p[3]));
  M = fmax(M, dpp_f64<0x128>(M, M));   // row_ror 8, 4, 2, 1
  M = fmax(M, dpp_f64<0x124>(M, M));
  M = fmax(M, dpp_f64<0x122>(M, M));
  M = fmax(M, dpp_f64<0x121>(M, M));
  S = 0.0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const double e = exp_neg(p[t] - M);
    S += p[t] == M ? (M == -INFINITY ? 0.0 : 1.0) : e;
  }
  S += dpp_f64<0x128>(S, S);
  S += dpp_f64<0x124>(S, S);
  S += dpp_f64<0x122>(S, S);
  S += dpp_f64<0x121>(S, S);
}

// EB = bytes per landmark element: 2 (bf16) or 1 (FP8 E5M2 storage; a row is then d bytes and a lane's
// piece holds twice as many elements, or the same number in 8 bytes when d is not a multiple of 64).
// HG = groups of four heads per landmark element: 1, or 2 for 5 to 8 query heads per KV head.  With HG = 2 every
// widened landmark element feeds two instructions (heads 0-3, heads 4-7; two accumulators per tile), so the
// landmarks are read and converted once for all eight heads.  The queries live in LDS as fp64.
template <int D, int EB, int HG, int NT>
__global__ __launch_bounds__(256) void score_kernel(const bf16_t* __restrict__ q, const uint8_t* __restrict__ L,
                                                    float* __restrict__ logits, double2* __restrict__ partials,
                                                    int hq, int hkv, int G, int n_c, int ld, int nc_stride, int n_tiles,
                                                    double scale) {
  constexpr int PB = (EB == 2 || D % 64 == 0) ? 16 : 8;  // bytes per piece
  constexpr int PE = PB / EB;                             // elements per piece
  constexpr int NI = D / (4 * PE);                        // pieces per lane per row
  constexpr int PW = PB / 4;                              // 32-bit words per piece
  __shared__ double2 wred[4][4 * HG];
  // q of the workgroup's heads as fp64; rows padded so that the four heads a block column reads at once fall
  // into different banks
  __shared__ double qs[4 * HG][D + 2];
  const int unit = blockIdx.y, tile = blockIdx.x, g0 = blockIdx.z * 4 * HG;
  const int b = unit / hkv, h = unit % hkv;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int kq = lane >> 4, blk = (lane >> 2) & 3, ij = lane & 3;
  const size_t head0 = (size_t)b * hq + (size_t)h * G + g0;

  const uint8_t* Lu = L + (size_t)unit * nc_stride * D * EB;  // the landmark array may have room to grow
  const int row0 = (tile * 4 + wave) * (16 * NT);
  // requested before q: the landmark rows are the long-latency loads.  FP8 rows past the end repeat the last one and count
  // as -inf below: a clamped index costs less than a lane mask around every load (step of 16 x 128K 129.5 -> 126.1 us; in
  // the 16-head kernel, 1M tokens, 104.8 -> 103 us); bf16 rows are bound by the memory system and lose by it (168.4 ->
  // 169.5 us).
  uint32_t w[NT][NI][PW];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int r = row0 + t * 16 + blk * 4 + ij;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int x = 0; x < PW; ++x) w[t][i][x] = 0u;
      if (EB == 1 || r < n_c) {
        const uint8_t* src = Lu + (size_t)(EB == 1 ? min(r, n_c - 1) : r) * D * EB + (size_t)(4 * PE * i + PE * kq) * EB;
        if constexpr (PW == 4) {
          const uint4 v = *reinterpret_cast<const uint4*>(src);
          w[t][i][0] = v.x; w[t][i][1] = v.y; w[t][i][2] = v.z; w[t][i][3] = v.w;
        } else {
          const uint2 v = *reinterpret_cast<const uint2*>(src);
          w[t][i][0] = v.x; w[t][i][1] = v.y;
        }
      }
    }
  }

  // A operand: q of the workgroup's heads as fp64, in LDS (registers are better spent on landmark rows in
  // flight); a lane reads head 4 hg + ij, the elements its k-slot meets
  for (int idx = threadIdx.x; idx < 4 * HG * D; idx += 256) {
    const int hh = idx / D, e = idx - hh * D;
    qs[hh][e] = g0 + hh < G ? (double)bf16_to_f32(q[(head0 + hh) * D + e]) : 0.0;
  }
  __syncthreads();

  double p[HG][NT];   // logits of heads g0 + 4 hg + lane / 16
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    double acc[HG];
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) acc[hg] = 0.0;
    // one widened landmark element against the matching q element of each head group
    auto step = [&](int i, int el, double lv) {
      const int col = 4 * PE * i + PE * kq + el;
#pragma unroll
      for (int hg = 0; hg < HG; ++hg)
        acc[hg] = __builtin_amdgcn_mfma_f64_4x4x4f64(qs[4 * hg + ij][col], lv, acc[hg], 0, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int x = 0; x < PW; ++x) {
        if constexpr (EB == 2) {
          step(i, 2 * x, (double)bf16_lo(w[t][i][x]));
          step(i, 2 * x + 1, (double)bf16_hi(w[t][i][x]));
        } else {
          float f[4];
          e5m2x4_to_f32(w[t][i][x], f);
#pragma unroll
          for (int e = 0; e < 4; ++e) step(i, 4 * x + e, (double)f[e]);
        }
      }
    }
    const int r = row0 + t * 16 + (lane & 15);
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) {
      const int hl = 4 * hg + (lane >> 4);   // head of this lane's result, inside the workgroup's heads
      p[hg][t] = r < n_c ? acc[hg] * scale : -INFINITY;   // the logit: exact products, fp64 sum
      if (r < n_c && g0 + hl < G) logits[(head0 + hl) * ld + r] = (float)p[hg][t];
    }
  }

  // (max, sum) of each head over the workgroup's rows
#pragma unroll
  for (int hg = 0; hg < HG; ++hg) {
    double m, s;
    row16_lse(p[hg], m, s);
    if ((lane & 15) == 0) wred[wave][4 * hg + (lane >> 4)] = make_double2(m, s);
  }
  __syncthreads();
  if (threadIdx.x < 4 * HG && g0 + (int)threadIdx.x < G) {
    const int g = threadIdx.x;
    double M = -INFINITY, S = 0.0;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) lse_merge(M, S, wred[wv][g].x, wred[wv][g].y);
    partials[(head0 + g) * n_tiles + tile] = make_double2(M, S);
  }
}

// Groups of more than 4 query heads per KV head: the 16x16x4 form of the fp64 matrix instruction takes up to
// 16 heads at once (A lane l = (head l % 16, k-slot l / 16), B lane l = (row l % 16, k-slot l / 16), result register j
// of lane l = (head 4 j + l / 16, row l % 16); measured on gfx950), so every landmark element is loaded and widened
// once instead of once per four heads.  Same tiles, same logits (exact products, fp64 sum) and partials as above.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
template <int D, int EB, int NT>
__global__ __launch_bounds__(256) void score_kernel_g16(const bf16_t* __restrict__ q, const uint8_t* __restrict__ L,
                                                        float* __restrict__ logits, double2* __restrict__ partials,
                                                        int hq, int hkv, int G, int n_c, int ld, int nc_stride,
                                                        int n_tiles, double scale) {
  constexpr int PB = (EB == 2 || D % 64 == 0) ? 16 : 8;
  constexpr int PE = PB / EB, NI = D / (4 * PE), PW = PB / 4;
  __shared__ double2 wred[4][16];
  const int unit = blockIdx.y, tile = blockIdx.x, g0 = blockIdx.z * 16;
  const int b = unit / hkv, h = unit % hkv;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int kq = lane >> 4, rl = lane & 15;
  const size_t head0 = (size_t)b * hq + (size_t)h * G + g0;
  const uint8_t* Lu = L + (size_t)unit * nc_stride * D * EB;
  const int row0 = (tile * 4 + wave) * (16 * NT);
  uint32_t w[NT][NI][PW];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const uint8_t* row = Lu + (size_t)min(row0 + t * 16 + rl, n_c - 1) * D * EB + PE * kq * EB;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint8_t* src = row + 4 * PE * i * EB;
      if constexpr (PW == 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(src);
        w[t][i][0] = v.x; w[t][i][1] = v.y; w[t][i][2] = v.z; w[t][i][3] = v.w;
      } else {
        const uint2 v = *reinterpret_cast<const uint2*>(src);
        w[t][i][0] = v.x; w[t][i][1] = v.y;
      }
    }
  }
  double qa[NI][PE];  // head g0 + rl, the elements this lane's k-slot meets (zero for heads past the group)
  const bool hv = g0 + rl < G;
  {
    const bf16_t* qp = q + (head0 + (hv ? rl : 0)) * D + PE * kq;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e8 = 0; e8 < PE / 8; ++e8) {
        float x[8];
        load_bf16_row<8>(qp + 4 * PE * i + 8 * e8, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) qa[i][8 * e8 + e] = hv ? (double)x[e] : 0.0;
      }
  }
  // the 16-row tiles of the wave take turns on the matrix pipe: consecutive instructions are independent where there are
  // several
  f64x4_t acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int x = 0; x < PW; ++x) {
      if constexpr (EB == 2) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[i][2 * x], (double)bf16_lo(w[t][i][x]), acc[t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[i][2 * x + 1], (double)bf16_hi(w[t][i][x]), acc[t], 0, 0, 0);
      } else {
        float f[NT][4];
#pragma unroll
        for (int t = 0; t < NT; ++t) e5m2x4_to_f32(w[t][i][x], f[t]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[i][4 * x + e], (double)f[t][e], acc[t], 0, 0, 0);
      }
    }
#pragma unroll
  for (int j = 0; j < 4; ++j) {   // heads g0 + 4 j + kq
    double p[NT], m, s;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int r = row0 + t * 16 + rl;
      p[t] = r < n_c ? acc[t][j] * scale : -INFINITY;   // the logit: exact products, fp64 sum
      if (r < n_c && g0 + 4 * j + kq < G) logits[(head0 + 4 * j + kq) * ld + r] = (float)p[t];
    }
    row16_lse(p, m, s);
    if (rl == 0) wred[wave][4 * j + kq] = make_double2(m, s);
  }
  __syncthreads();
  if (threadIdx.x < 16 && g0 + (int)threadIdx.x < G) {
    const int g = threadIdx.x;
    double M = -INFINITY, S = 0.0;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) lse_merge(M, S, wred[wv][g].x, wred[wv][g].y);
    partials[(head0 + g) * n_tiles + tile] = make_double2(M, S);
  }
}

// 16-row tiles per wave.  Many waves of few rows start and end evenly and fill a chip that few workgroups would leave idle;
// where there is enough of both, fewer workgroups stage the queries less often and leave fewer pairs to merge.  Short rows are
// there sooner, so that this line lies lower for them.  In workgroups of 256 rows, us with four / two / one tiles per wave:
//   up to four heads, rows of 256 bytes: 16 (1 x 4K) 9.4 / 7.3 / 6.7; 512 (4 x 32K) 15.6 / 13.3 / 12.6; 1024 23.4 / 20.6 / 20.5;
//     4096 (16 x 64K) 57.2 / 56.6 / 65.0; 8192 107.7 / 107.6 / 123.5; of 192: 512 11.7 / 11.3 / 11.7; 4096 45.4 / 44.4 / 50.7;
//     of 128: 256 9.1 / 8.5 / 8.6; 1024 16.7 / 16.1 / 17.7 (FP8), 13.1 / 12.1 / 13.5 (heads of 64); 2048 24.2 / 26.4 / 29.3, 18.9 /
//     19.3 / 21.8; of 96: 512 10.0 / 10.0 / 10.5
//   five to eight, rows of 256 bytes: 256 13.3 / 12.0 / 11.6; 1024 30.2 / 26.8 / 29.1; 4096 86.2 / 83.3 / 97.1; of 128: 128 10.1 /
//     8.2 / 7.9; 256 9.4 / 8.9 / 9.1; 1024 23.2 / 23.2 / 24.6, 17.4 / 17.2 / 18.5; 2048 36.4 / 39.6 / 43.5, 26.4 / 28.4 / 31.6
//   sixteen: 32 (1 x 32K) 12.1 / 8.8 / 7.4; 128 12.5 / 9.5 / 9.5; 512 18.7 / 18.8 / 20.2
int score_tiles(int units, int G, int d, int n_c, int kv_bytes) {
  const long z = G > 8 ? (G + 15) / 16 : 1, wgs = units * z * score_tile_count(n_c, 4);
  const bool short_rows = d * kv_bytes <= 128;
  const long one = G > 8 ? 64 : (G > 4 ? 256 : 512) / (short_rows ? 2 : 1), two = G > 8 ? 256 : short_rows ? 1024 : 4096;
  return wgs <= one ? 1 : wgs <= two ? 2 : 4;
}

hipError_t launch_score(const bf16_t* q, const void* landmarks, int kv_bytes, float* logits, int ld, double2* partials,
                        int batch, int hq, int hkv, int d, int n_c, int nc_stride, double scale, int tiles, hipStream_t st) {
  const int G = hq / hkv;
  const int n_tiles = score_tile_count(n_c, tiles);
  // up to four heads per KV head: score_kernel<.., 1>; five to eight: score_kernel<.., 2>; more: one pass per 16
  // heads on the 16x16x4 instruction (heads past the group are zero rows of its operand)
  const bool g16 = G > 8;
  dim3 grid(n_tiles, batch * hkv, g16 ? (G + 15) / 16 : 1), block(256);
  const uint8_t* L = static_cast<const uint8_t*>(landmarks);
#define SKV_LAUNCH(KERNEL_) hipLaunchKernelGGL(KERNEL_, grid, block, 0, st, q, L, logits, partials, hq, hkv, G, n_c, ld, nc_stride, n_tiles, scale)
#define SKV_SCORE_NT(D_, EB_, NT_)                                                                                    \
  do {                                                                                                                \
    if (g16) SKV_LAUNCH((score_kernel_g16<D_, EB_, NT_>));                                                            \
    else if (G > 4) SKV_LAUNCH((score_kernel<D_, EB_, 2, NT_>));                                                      \
    else SKV_LAUNCH((score_kernel<D_, EB_, 1, NT_>));                                                                 \
  } while (0)
#define SKV_SCORE(D_, EB_)                                                                                            \
  do {                                                                                                                \
    if (tiles == 1) SKV_SCORE_NT(D_, EB_, 1);                                                                         \
    else if (tiles == 2) SKV_SCORE_NT(D_, EB_, 2);                                                                    \
    else if (tiles == 4) SKV_SCORE_NT(D_, EB_, 4);                                                                    \
    else return hipErrorInvalidValue;                                                                                 \
  } while (0)
  switch (d * 4 + kv_bytes) {
    case 64 * 4 + 2: SKV_SCORE(64, 2); break;
    case 96 * 4 + 2: SKV_SCORE(96, 2); break;
    case 128 * 4 + 2: SKV_SCORE(128, 2); break;
    case 64 * 4 + 1: SKV_SCORE(64, 1); break;
    case 96 * 4 + 1: SKV_SCORE(96, 1); break;
    case 128 * 4 + 1: SKV_SCORE(128, 1); break;
    default: return hipErrorInvalidValue;
  }
#undef SKV_SCORE
#undef SKV_SCORE_NT
#undef SKV_LAUNCH
  return hipGetLastError();
}

}  // namespace skv
