// One more chunk of context from generated tokens (last paragraph of section "High-throughput
// Decoding" and its footnote): new pre-RoPE keys K' are kept as the low-rank states K' Psi, where
// Psi is the right singular matrix of the context keys -- here Psi^T = B over the full key width,
// Psi[(h, x), rho] = B[b, h, rho, x].  The c tokens become chunk n_ch = s / c of the context exactly
// as if the pre-filling algorithm had seen them: c rows of A, one landmark (mean of the chunk's
// post-RoPE keys, fp64, rounded once), its chunk id, and the chunk's values in the store (a plain
// copy; the store may be pinned host memory written over PCIe).  Small: what it takes is latency, so
// everything is one launch.
#include "kernels.hpp"

namespace skv {

typedef double f64x4_app __attribute__((ext_vector_type(4)));

// The first n_proj workgroups project: one per (16 rank indices, 16 tokens, sequence), on the fp64 matrix instruction
// v_mfma_f64_16x16x4f64 (A lane l = (token l % 16, k-slot l / 16), B lane l = (rank l % 16, k-slot l / 16), result
// register j of lane l = (token 4 j + l / 16, rank l % 16)).  The key width is cut into 32-column steps that the
// workgroup's eight waves take in turn, four steps (eight 16-byte pieces per lane) requested together; the partial sums
// meet in LDS.  B is read once for 16 tokens, and 10 x batch workgroups of eight waves share it: at 16 sequences, 8
// tokens, key width 1024 and rank 160 the launch takes 6.3 us, where one workgroup per token with a scalar loop over the
// ranks (each of them reading all of B) took 108 us, bound by its chain of 2-byte loads, and the landmark kernel 5 us
// behind it.
// The other workgroups (one per unit): landmark row, its chunk id, and the copy of the chunk's values.
// EB: bytes per stored element (2 = bf16, 1 = FP8 E5M2), inputs and outputs alike.
constexpr int kAppendNT = 512;
template <int EB>
__global__ __launch_bounds__(kAppendNT) void append_kernel(const uint8_t* __restrict__ k_pre,
                                                           const void* __restrict__ k_rope,
                                                           const uint4* __restrict__ v, const uint8_t* __restrict__ B,
                                                           void* __restrict__ A, void* __restrict__ landmarks,
                                                           int32_t* __restrict__ landmark_chunk_ids,
                                                           uint4* __restrict__ value_store, int hkv, int d, int s,
                                                           int s_cap, int c, int r, int o, int r_tiles, int t_tiles,
                                                           int n_proj) {
  if ((int)blockIdx.x < n_proj) {
    constexpr int NW = kAppendNT / kWave, U = 4, RW = RawWords<8, EB>::n;
    __shared__ double red[NW][16][17];
    const int rt = blockIdx.x % r_tiles, tt = blockIdx.x / r_tiles % t_tiles, b = blockIdx.x / (r_tiles * t_tiles);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int sub = lane & 15, kq = lane >> 4;
    const int D = hkv * d, n_steps = D / 32, steps_per_head = d / 32;
    // tokens and ranks past the end repeat the last real one; their results are not written
    const uint8_t* krow = k_pre + ((size_t)b * c + min(tt * 16 + sub, c - 1)) * D * EB;
    const uint8_t* brow = B + ((size_t)b * hkv * r + min(rt * 16 + sub, r - 1)) * d * EB;
    f64x4_app acc = {0.0, 0.0, 0.0, 0.0};
    for (int s0 = wave; s0 < n_steps; s0 += NW * U) {
      uint32_t kw[U][RW], bw[U][RW];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int step = min(s0 + u * NW, n_steps - 1);
        const int h = step / steps_per_head, x = (step - h * steps_per_head) * 32 + 8 * kq;
        load_raw<8, EB>(krow + (size_t)(h * d + x) * EB, kw[u]);
        load_raw<8, EB>(brow + ((size_t)h * r * d + x) * EB, bw[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u * NW < n_steps) {   // (uniform over the wave)
          float kx[8], bx[8];
          unpack_kv<8, EB>(kw[u], kx);
          unpack_kv<8, EB>(bw[u], bx);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)kx[e], (double)bx[e], acc, 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) red[wave][4 * j + kq][sub] = acc[j];
    __syncthreads();
    if (threadIdx.x < 256) {
      const int t = threadIdx.x >> 4, n = threadIdx.x & 15;
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) sum += red[w][t][n];
      const int tok = tt * 16 + t, rho = rt * 16 + n;
      if (tok < c && rho < r) kv_store_elem<EB>(A, ((size_t)b * s_cap + s + tok) * r + rho, sum);
    }
    return;
  }
  const int unit = blockIdx.x - n_proj;
  const int n_ch = s / c, n_c = n_ch - o, nc_stride = s_cap / c - o;
  for (int x = threadIdx.x; x < d; x += kAppendNT) {
    double acc = 0.0;
#pragma unroll 8
    for (int t = 0; t < c; ++t) acc += (double)kv_elem<EB>(k_rope, ((size_t)unit * c + t) * d + x);
    kv_store_elem<EB>(landmarks, ((size_t)unit * nc_stride + n_c) * d + x, acc / (double)c);
  }
  if (threadIdx.x == 0) landmark_chunk_ids[(size_t)unit * nc_stride + n_c] = n_ch;
  const int vec = c * d * EB / 16;
  uint4* dst = value_store + ((size_t)unit * s_cap + s) * d * EB / 16;
  for (int i = threadIdx.x; i < vec; i += kAppendNT) dst[i] = v[(size_t)unit * vec + i];
}

template <int EB>
static hipError_t launch_append_eb(const void* k_pre, const void* k_rope, const void* v, const void* B, void* A,
                                   void* landmarks, int32_t* landmark_chunk_ids, void* value_store, int batch, int hkv,
                                   int d, int s, int s_cap, int c, int r, int o, hipStream_t st) {
  const int r_tiles = (r + 15) / 16, t_tiles = (c + 15) / 16, n_proj = r_tiles * t_tiles * batch;
  hipLaunchKernelGGL(append_kernel<EB>, dim3(n_proj + batch * hkv), dim3(kAppendNT), 0, st,
                     static_cast<const uint8_t*>(k_pre), k_rope, reinterpret_cast<const uint4*>(v),
                     static_cast<const uint8_t*>(B), A, landmarks, landmark_chunk_ids,
                     reinterpret_cast<uint4*>(value_store), hkv, d, s, s_cap, c, r, o, r_tiles, t_tiles, n_proj);
  return hipGetLastError();
}

hipError_t launch_append_chunk(const void* k_pre, const void* k_rope, const void* v, const void* B, void* A,
                               void* landmarks, int32_t* landmark_chunk_ids, void* value_store, int kv_bytes, int batch,
                               int hkv, int d, int s, int s_cap, int c, int r, int o, hipStream_t st) {
  return kv_bytes == 1 ? launch_append_eb<1>(k_pre, k_rope, v, B, A, landmarks, landmark_chunk_ids, value_store, batch,
                                             hkv, d, s, s_cap, c, r, o, st)
                       : launch_append_eb<2>(k_pre, k_rope, v, B, A, landmarks, landmark_chunk_ids, value_store, batch,
                                             hkv, d, s, s_cap, c, r, o, st);
}

}  // namespace skv
