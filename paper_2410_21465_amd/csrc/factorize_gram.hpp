// Gram matrix G = K^T K of the stored keys on the 8-bit integer matrix instruction, exact but for the last additions: the keys of a column are taken
// as multiples of one power of two, cut into three signed 8-bit digits, and the digits' products are summed in 32-bit
// integers, which lose nothing.  (v_mfma_i32_32x32x32_i8: A lane l holds row l % 32, contraction elements 16 (l / 32) .. + 15,
// B the same of its columns, result register j of lane l is (row = 8 (j / 4) + 4 (l / 32) + j % 4, column = l % 32); measured
// on gfx950.)
//
// Column j of a sequence gets the exponent sh_j with |x| 2^sh_j < 2^22 for its largest element; v = x 2^sh_j rounded to an
// integer is d0 2^16 + d1 2^8 + d2 with digits in [-128, 127].  An element whose exponent lies at most 14 below the largest
// one's is such an integer itself; of normally distributed keys one in ten thousand is not.  What rounding leaves of those,
// r = x - v 2^-sh, goes on a list, and gram_finish_kernel adds what the digits miss: with Y = K - R,
//   K^T K = Y^T Y + H + H^T,  H = R^T (K - R / 2),
// in fp64.  The list of a part of the tokens and columns has room for three elements in 2048; keys that need more (a few rows
// far above the rest, columns next to the least bf16 numbers) and keys that are infinite, NaN or beyond 2^22 (2^-133, the
// least bf16 number, times their column's power of two would leave bf16) raise the sequence's flag, and gram_kernel forms
// that sequence's sums in fp64 instead.
#pragma once
#include "common.hpp"

namespace skv {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kDigitSegment = 32768;       // tokens whose digit sums fit 32 bits: 3 * 2^14 * 32768 < 2^31
constexpr int kDigitStage = 64;            // tokens in LDS at a time
// 2^23 + 0x408080: added to a number of magnitude up to 0x3f7f7f, it leaves the nearest integer v in the low bits of the fp32
// pattern, 0x408080 + v; the bytes of that are d0 + 64, d1 + 128 and d2 + 128
constexpr float kDigitMagic = 12615808.0f;

// Lists of the elements that their digits do not hold: where (token << 7 | column in the block of 128) and what the digits miss,
// as bf16 in units of 2^-sh of the column (it has at most 8 significant bits).  Six bytes an entry, and four for its place in
// the order by column: a workspace has room for few.
constexpr int kRestTokens = 1 << 25;       // tokens that an entry can name; longer sequences are summed in fp64
struct RestLists {
  uint32_t* where;
  uint16_t* rest;
};
// eight stored columns of a token as they lie in memory, and one of them as fp32
template <int EB>
struct Piece {
  uint32_t w[2 * EB];
  __device__ __forceinline__ void load(const uint8_t* p) {
    if constexpr (EB == 2) {
      const uint4 v = *reinterpret_cast<const uint4*>(p);
      w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else {
      const uint2 v = *reinterpret_cast<const uint2*>(p);
      w[0] = v.x; w[1] = v.y;
    }
  }
  template <int X>
  __device__ __forceinline__ float elem() const {
    if constexpr (EB == 2) return X & 1 ? bf16_hi(w[X / 2]) : bf16_lo(w[X / 2]);
    else return __builtin_amdgcn_cvt_f32_bf8((int)w[X / 4], X & 3);
  }
  // magnitudes (storage bits) of the i-th pair of columns: neighbours (bf16), two apart (E5M2: even and odd bytes of a word)
  static constexpr int first(int i) { return EB == 2 ? 2 * i : 4 * (i / 2) + i % 2; }
  static constexpr int second(int i) { return first(i) + EB % 2 + 1; }
  template <int I>
  __device__ __forceinline__ u16x2 magnitudes() const {
    const uint32_t a = EB == 2 ? w[I % (2 * EB)] & 0x7fff7fffu : (w[I / 2] >> (8 * (I % 2))) & 0x007f007fu;
    return *reinterpret_cast<const u16x2*>(&a);
  }
  // an element is an integer times 2^-sh if its last place is worth at least that: exponent - 134 + sh >= 0 (bf16; E5M2: - 17)
  static __device__ __forceinline__ uint16_t threshold(float scale) {
    const int sh = (int)(__float_as_uint(scale) >> 23) - 127;
    return (uint16_t)(EB == 2 ? max(134 - sh, 0) << 7 : max(17 - sh, 0) << 2);
  }
  // 2^sh as the products below take it: bf16 in the half of a word that meets the x-th element, or fp32 (E5M2)
  static __device__ __forceinline__ uint32_t scale_word(int x, float scale) {
    return EB == 2 && !(x & 1) ? __float_as_uint(scale) >> 16 : __float_as_uint(scale);
  }
};
// x 2^sh + kDigitMagic, rounded to an integer (nearest, ties to even), of four elements; the widening is left to the
// instruction.  w: the words that hold them, s: their scale words (Piece::scale_word).  bf16: the two-term product of the pair
// with (2^sh, 0) or (0, 2^sh) (v_dot2_f32_bf16 rounds once and keeps the least numbers: compared with the definition for every
// bf16 number and scale).  The compiler has only the form that adds to its result's register, a move more per element; the
// three idle cycles at the end are what another instruction has to wait for the result.
__device__ __forceinline__ void scaled4_bf16(const uint32_t (&w)[4], const uint32_t (&s)[4], uint32_t (&out)[4]) {
  asm("v_dot2_f32_bf16 %0, %4, %8, %12\n\t"
      "v_dot2_f32_bf16 %1, %5, %9, %12\n\t"
      "v_dot2_f32_bf16 %2, %6, %10, %12\n\t"
      "v_dot2_f32_bf16 %3, %7, %11, %12\n\t"
      "s_nop 2"
      : "=&v"(out[0]), "=&v"(out[1]), "=&v"(out[2]), "=&v"(out[3])
      : "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]), "s"(kDigitMagic));
}
// E5M2 (the upper byte of fp16): element X of the word
template <int X>
__device__ __forceinline__ uint32_t scaled_e5m2(uint32_t w, uint32_t s) {
  const uint32_t p = __builtin_amdgcn_perm(0u, w, X & 2 ? 0x030c020cu : 0x010c000cu);
  return __float_as_uint(fmaf((float)(*reinterpret_cast<const f16x2*>(&p))[X & 1], __uint_as_float(s), kDigitMagic));
}
// the digits of four such numbers, four bytes a digit, the most significant one first
__device__ __forceinline__ void split_digits(const uint32_t (&w)[4], uint32_t (&d)[3]) {
  const uint32_t lo01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), lo23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
  const uint32_t hi01 = __builtin_amdgcn_perm(w[1], w[0], 0x0c0c0602u), hi23 = __builtin_amdgcn_perm(w[3], w[2], 0x0c0c0602u);
  d[0] = (__builtin_amdgcn_perm(hi23, hi01, 0x05040100u) + 0x40404040u) ^ 0x80808080u;
  d[1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u;
  d[2] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u) ^ 0x80808080u;
}
// what the digits of element x leave out, in units of 2^-sh: x 2^sh - v
__device__ __forceinline__ float digit_rest(float x, float scale) {
  return fmaf(x, scale, -(fmaf(x, scale, kDigitMagic) - kDigitMagic));
}
// ---- largest magnitude of every column ------------------------------------------------------------------
// Storage bits without the sign order like the magnitudes.  chunk_max [b][n_chunks][D]; a thread takes one 16-byte piece of
// the rows of its chunk, 256 / LV rows of LV pieces at a time.  The first chunk's workgroup clears the sequence's flag.
// Bound by the read of the keys.
template <int EB>
__global__ __launch_bounds__(256) void column_max_kernel(const void* __restrict__ K, uint16_t* __restrict__ chunk_max,
                                                         int32_t* __restrict__ flags, int s, int D, int lv, int chunk,
                                                         int n_chunks) {
  constexpr int NE = 16 / EB;              // elements per piece
  __shared__ uint32_t red[256][NE / 2 + 1];
  const int b = blockIdx.y, ck = blockIdx.x, pieces = D / NE;
  if (threadIdx.x == 0 && ck == 0 && blockIdx.z == 0) flags[b] = 0;
  const int lane_v = threadIdx.x & (lv - 1), row = threadIdx.x / lv, rows = 256 / lv;
  const int piece = blockIdx.z * lv + lane_v, pc = min(piece, pieces - 1);
  const int t_end = min(s, (ck + 1) * chunk);
  const uint4* src = static_cast<const uint4*>(K) + (size_t)b * s * pieces + pc;
  u16x2 m[NE / 2];
#pragma unroll
  for (int i = 0; i < NE / 2; ++i) m[i] = u16x2{0, 0};
  auto take = [&](uint4 v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (EB == 2) {
        const uint32_t a = w[i] & 0x7fff7fffu;
        m[i] = __builtin_elementwise_max(m[i], *reinterpret_cast<const u16x2*>(&a));
      } else {
        const uint32_t a = w[i] & 0x007f007fu, c = (w[i] >> 8) & 0x007f007fu;
        m[2 * i] = __builtin_elementwise_max(m[2 * i], *reinterpret_cast<const u16x2*>(&a));
        m[2 * i + 1] = __builtin_elementwise_max(m[2 * i + 1], *reinterpret_cast<const u16x2*>(&c));
      }
    }
  };
  // (rows past the end repeat the last one: the maximum is the same)
  for (int t = ck * chunk + row; t < t_end; t += 8 * rows) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = src[(size_t)min(t + u * rows, t_end - 1) * pieces];
#pragma unroll
    for (int u = 0; u < 8; ++u) take(v[u]);
  }
#pragma unroll
  for (int i = 0; i < NE / 2; ++i) red[threadIdx.x][i] = *reinterpret_cast<const uint32_t*>(&m[i]);
  __syncthreads();
  if (row == 0 && piece < pieces) {
    for (int r = 1; r < rows; ++r)
#pragma unroll
      for (int i = 0; i < NE / 2; ++i) {
        const uint32_t o = red[r * lv + lane_v][i];
        m[i] = __builtin_elementwise_max(m[i], *reinterpret_cast<const u16x2*>(&o));
      }
    uint16_t* out = chunk_max + ((size_t)b * n_chunks + ck) * D + piece * NE;
#pragma unroll
    for (int i = 0; i < NE / 2; ++i) {
      // the two halves of m[i] are neighbours (bf16) or two apart (E5M2: even bytes in m[2 i], odd ones in m[2 i + 1])
      if constexpr (EB == 2) { out[2 * i] = m[i].x; out[2 * i + 1] = m[i].y; }
      else { out[4 * (i / 2) + (i & 1)] = m[i].x; out[4 * (i / 2) + 2 + (i & 1)] = m[i].y; }
    }
  }
}

// scale[b][j] = 2^sh_j, 1 <= scale <= 2^126; 64 columns per workgroup, sixteen threads each.  The flag of the sequence is raised
// by a column with an element beyond 2^22 (or not finite), and where a sample of kSample tokens (spaced evenly over the
// sequence, step 2^-32 tokens apart; all of a shorter one) says that the lists will not do: more than `share` of the workgroup's
// elements are not held by their digits, or several times that in one token part.  `share` is what the lists have room for,
// less four standard deviations of such a list's length, and the sample is large enough to tell that from three quarters of it:
// with 256 tokens and twice the lists' room, keys with 1 % of their chunks 10 to 16 times the others' size went through the
// digits' products, filled their lists and were summed in fp64 after all, 64.2 ms at 16 x 128K x 1024 where the fp64 sums alone
// take 53.9; now 32.5 to 54.0.  The sample takes 2 us of 11 for one sequence, 12 of 19 for 16.
constexpr int kSample = 2048;
template <int EB>
__global__ __launch_bounds__(1024) void column_scale_kernel(const void* __restrict__ K, const uint16_t* __restrict__ chunk_max,
                                                            float* __restrict__ scale, int32_t* __restrict__ flags, int s, int D,
                                                            int n_chunks, int tokens_per_split, uint64_t step, float share) {
  constexpr int kRows = 1024 / 64, kPass = 1024 / 8, kParts = 512;
  __shared__ uint32_t red[kRows][64];
  __shared__ float sc[64];
  __shared__ int32_t missed[kParts];   // elements of the sample that are not held, per token part
  __shared__ int32_t all_missed;
  const int b = blockIdx.y, x = threadIdx.x & 63, y = threadIdx.x >> 6, col0 = blockIdx.x * 64, col = min(col0 + x, D - 1);
  uint32_t m = 0;
#pragma unroll 8
  for (int c = y; c < n_chunks; c += kRows) m = max(m, (uint32_t)chunk_max[((size_t)b * n_chunks + c) * D + col]);
  red[y][x] = m;
  if (threadIdx.x < kParts) missed[threadIdx.x] = 0;
  if (threadIdx.x == 0) all_missed = 0;
  __syncthreads();
  if (y == 0) {
#pragma unroll
    for (int i = 1; i < kRows; ++i) m = max(m, red[i][x]);
    // exponent of the largest element, biased as in fp32; one more where the leading bits are all ones (two more units of
    // the last place of bf16 carry into it), since 2^22 itself is out of kDigitMagic's reach
    const uint32_t f = EB == 2 ? m << 16 : __float_as_uint(e5m2_to_f32((uint8_t)m));
    const int e = (int)((f + 0x20000u) >> 23);
    if (e > 148 || s > kRestTokens) flags[b] = 1;
    // |x| <= (1 - 3 / 256) 2^(e - 126): 2^(148 - e) |x| <= 0x3f4000
    sc[x] = __uint_as_float((uint32_t)(127 + 148 - min(max(e, 22), 148)) << 23);
    if (col0 + x < D) scale[(size_t)b * D + col] = sc[x];
  }
  __syncthreads();
  // eight columns of a token per thread, kPass tokens at a time
  const int c8 = 8 * (threadIdx.x & 7), n = min(kSample, s);
  auto token = [&](int i) { return (int)((uint64_t)i * step >> 32); };
#pragma unroll 1
  for (int i0 = threadIdx.x >> 3; i0 < n; i0 += 8 * kPass) {
    Piece<EB> v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int t = token(min(i0 + kPass * i, n - 1));
      v[i].load(static_cast<const uint8_t*>(K) + (((size_t)b * s + t) * D + min(col0 + c8, D - 8)) * EB);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i0 + kPass * i >= n) continue;
      int mine = 0;
      each_of(std::make_integer_sequence<int, 8>{}, [&](auto e) { mine += digit_rest(v[i].template elem<e>(), sc[c8 + e]) != 0.0f ? 1 : 0; });
      if (col0 + c8 < D && mine) {
        atomicAdd(&missed[min(token(i0 + kPass * i) / tokens_per_split, kParts - 1)], mine);
        atomicAdd(&all_missed, mine);
      }
    }
  }
  __syncthreads();
  // (eight elements fill no list)
  const float room = share * (float)min(64, D - col0), taken = (float)n * (float)min(s, tokens_per_split) / (float)s;   // of a part
  if (threadIdx.x < kParts && (float)missed[threadIdx.x] > 2.0f * room * taken + 8.0f) flags[b] = 1;
  if (threadIdx.x == 0 && (float)all_missed > fmaxf(room * (float)n, 8.0f)) flags[b] = 1;
}

// ---- the digits' products ---------------------------------------------------------------------------------
// A workgroup of eight waves owns one 128 x 128 tile (bi <= bj) of one sequence and one part of its tokens.  Per stage of 64
// tokens each wave cuts 16 tokens x 128 columns (waves 0-3 the row block's, 4-7 the column block's; on the diagonal only the
// former exist) into digits and leaves them in LDS, token-contiguous as the matrix instruction wants them, requests its keys
// of the stage after, and then takes its 64 x 32 part of the products of the stage before: nine 32 x 32 x 32 products per 32
// tokens, summed by weight, d_p d_q -> 2^(32 - 8 (p + q)), in five sets of accumulators (160 registers).
// LDS: digit planes of 128 columns x 64 tokens; two columns share 128 bytes, whose eight 16-byte pieces are turned by the
// column so that neither the writes (a lane: one word of eight columns) nor the operand reads (a lane: one piece of one
// column) meet in a bank.
// The tiles of one sequence and token part run on one XCD (workgroups go round the eight XCDs), whose L2 then serves most
// reads of a key (three in four; every key is read by nb2 + 1 tiles).
// 16 x 128K x 1024: 9.7 ms where the fp64 sums took 35.1; 1 x 32K: 0.175 and 0.61 ms.  The products alone (4.7 ms at the
// instruction's rate) take 6.0, cutting alone 3.5; they share the vector issue, and the wait for keys is another 0.8.  Tried:
// waves 4-7 multiplying while waves 0-3 cut 10.4 ms against 9.2 (all else as then), cutting spread between the products of
// the same wave 11.7, two stages of keys in flight no gain, raised wave priority for the products no gain.
// index of the pair (bi, bj), bi <= bj < nb, in the order of the partial sums
__device__ __forceinline__ int upper_block(int nb, int bi, int bj) { return bi * nb - bi * (bi - 1) / 2 + (bj - bi); }

struct GramTile {
  const uint8_t* K;          // the sequence's keys
  const float* scale;        // [D]
  double* out;               // partial sums of this sequence and token part
  RestLists rest;            // diagonal: four lists of this column block and token part
  int32_t* rest_count;
  int32_t* marks;            // [4][n_marks]: entries of each list before every 256th token
  int32_t* flag;
  int s, D, nb, bi, bj, t_begin, t_end, rest_cap, n_marks;
};
// byte offset in a plane of column c (of 128), tokens 16 t16 .. + 15 (of 64)
__device__ __forceinline__ int operand_at(int c, int t16) {
  const int m = c >> 1;
  return m * 128 + 16 * ((4 * (c & 1) + t16) ^ ((m ^ (m >> 2)) & 7));
}
template <int EB, bool DIAG>
__device__ __forceinline__ void gram_digits_tile(const GramTile& g, uint8_t* lds) {
  constexpr int kPlane = 128 * 64, kBlock = 3 * kPlane;      // bytes: one digit of a column block; all three
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int blk = wave >> 2, tq = wave & 3;
  const bool cuts = !DIAG || blk == 0;
  // this lane's eight columns (past the end they repeat the last eight: their results are not written) and the first of its
  // four tokens; half a wave has 64 columns of 16 tokens
  const int l8 = (lane & 7) + 8 * (lane >> 5), t4 = (lane >> 3) & 3;
  const int cl = 8 * l8, col = (blk ? g.bj : g.bi) * 128 + cl, cc = min(col, g.D - 8);
  const int tok = 16 * tq + 4 * t4;
  // operand_at(cl + x, tq) + 4 t4 is this with bits 4 to 6 turned by 4 (x % 2) + x / 2, plus 128 (x / 2)
  const int put = operand_at(cl, tq) + 4 * t4 + blk * kBlock;
  float sc[8];
  {
    const float4 lo = *reinterpret_cast<const float4*>(g.scale + cc), hi = *reinterpret_cast<const float4*>(g.scale + cc + 4);
    sc[0] = lo.x; sc[1] = lo.y; sc[2] = lo.z; sc[3] = lo.w; sc[4] = hi.x; sc[5] = hi.y; sc[6] = hi.z; sc[7] = hi.w;
  }
  u16x2 below[4];            // per pair of columns: magnitudes (storage bits) below which an element may not be an integer
  each_of(std::make_integer_sequence<int, 4>{}, [&](auto i) {
    below[i] = u16x2{Piece<EB>::threshold(sc[Piece<EB>::first(i)]), Piece<EB>::threshold(sc[Piece<EB>::second(i)])};
  });
  int n_rest = 0;
  constexpr auto kColumns = std::make_integer_sequence<int, 8>{};

  Piece<EB> raw[4];   // this wave's part of the next stage
  auto request = [&](int t0) {
    const int tb = min(t0 + 16 * tq, g.s - 1), last = g.s - 1 - tb;   // (tokens past the end repeat the last one)
    const uint8_t* base = g.K + (size_t)tb * g.D * EB;
#pragma unroll
    for (int u = 0; u < 4; ++u) raw[u].load(base + (uint32_t)((min(4 * t4 + u, last) * g.D + cc) * EB));
  };
  auto cut = [&](int t0, int buf) {
    if (t0 + 16 * tq + 16 > g.t_end) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 2 * EB; ++i) raw[u].w[i] = t0 + tok + u < g.t_end ? raw[u].w[i] : 0u;
    }
    if constexpr (DIAG) {
      if (((t0 - g.t_begin) & 255) == 0 && lane == 0) {
        g.marks[tq * g.n_marks + (t0 - g.t_begin) / 256] = n_rest;
        if (n_rest > g.rest_cap) __hip_atomic_store(g.flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      // Which elements may the digits not hold: those below their column's threshold, compared two at a time.  A pair of
      // columns where there are any (three stages of a wave in four have none where the keys are normally distributed) is
      // looked at element by element; the entries' order is that of column pair, column, token, lane.
      each_of(std::make_integer_sequence<int, 4>{}, [&](auto i) {
        u16x2 least = raw[0].template magnitudes<i>();
#pragma unroll
        for (int u = 1; u < 4; ++u) least = __builtin_elementwise_min(least, raw[u].template magnitudes<i>());
        if (__any((least.x < below[i].x || least.y < below[i].y) && col < g.D)) {
          each_of(std::integer_sequence<int, Piece<EB>::first(i), Piece<EB>::second(i)>{}, [&](auto x) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const float r = digit_rest(raw[u].template elem<x>(), sc[x]);
              const bool have = r != 0.0f && col < g.D;
              const uint64_t mask = __ballot(have);
              if (mask) {
                const int at = n_rest + __popcll(mask & ((1ull << lane) - 1ull));
                if (have && at < g.rest_cap) {
                  g.rest.where[tq * g.rest_cap + at] = (uint32_t)(t0 + tok + u) << 7 | (uint32_t)(cl + x);
                  g.rest.rest[tq * g.rest_cap + at] = (uint16_t)(__float_as_uint(r) >> 16);
                }
                n_rest += __popcll(mask);
              }
            }
          });
        }
      });
    }
    int dst = put + buf * 2 * kBlock;
    asm volatile("" : "+v"(dst));   // (the eight places are formed here and not kept through the products)
    each_of(kColumns, [&](auto x) {
      uint32_t w[4], d[3];
      const uint32_t sw = Piece<EB>::scale_word(x, sc[x]);
      if constexpr (EB == 2) {
        scaled4_bf16({raw[0].w[x / 2], raw[1].w[x / 2], raw[2].w[x / 2], raw[3].w[x / 2]}, {sw, sw, sw, sw}, w);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = scaled_e5m2<x % 4>(raw[u].w[x / 4], sw);
      }
      split_digits(w, d);
      uint8_t* at = lds + (dst ^ (16 * (4 * (x & 1) + x / 2))) + 128 * (x / 2);
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<uint32_t*>(at + p * kPlane) = d[p];
    });
  };

  const int wr = wave & 1, wc = wave >> 1;   // this wave's 64 rows and 32 columns of the tile
  const int sub = lane & 31, half = lane >> 5;

#pragma unroll 1
  for (int seg = g.t_begin; seg < g.t_end; seg += kDigitSegment) {
    const int seg_end = min(g.t_end, seg + kDigitSegment), stages = (seg_end - seg + kDigitStage - 1) / kDigitStage;
    i32x16 acc[5][2];
#pragma unroll
    for (int w = 0; w < 5; ++w)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[w][t][j] = 0;
    if (cuts) {
      request(seg);
      cut(seg, 0);
      request(seg + kDigitStage);
    }
    __syncthreads();
    // (what is requested past the segment's end is clamped to the sequence and not cut)
#pragma unroll 1
    for (int st = 0; st < stages; ++st) {
      const int buf = st & 1, next = seg + (st + 1) * kDigitStage;
      const bool more = cuts && st + 1 < stages;
      if (more) { cut(next, buf ^ 1); request(next + kDigitStage); }
      const uint8_t* pa = lds + buf * 2 * kBlock;
      const uint8_t* pb = pa + (DIAG ? 0 : kBlock);
      // four steps of nine products (32 tokens, one of the two row groups); each step's operands are read from LDS during the
      // step before
      i32x4 a[2][3], bb[2][3];
      auto read_a = [&](int n) {
#pragma unroll
        for (int p = 0; p < 3; ++p)
          a[n & 1][p] = *reinterpret_cast<const i32x4*>(pa + p * kPlane + operand_at(64 * wr + 32 * (n & 1) + sub, (n & 2) + half));
      };
      auto read_b = [&](int kk) {
#pragma unroll
        for (int q = 0; q < 3; ++q) bb[kk][q] = *reinterpret_cast<const i32x4*>(pb + q * kPlane + operand_at(32 * wc + sub, 2 * kk + half));
      };
      read_b(0);
      read_a(0);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        if (n < 3) read_a(n + 1);
        if (n == 1) read_b(1);
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
          for (int q = 0; q < 3; ++q)
            acc[p + q][n & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[n & 1][p], bb[n >> 1][q], acc[p + q][n & 1], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
    }
    // five sums -> one integer -> fp64, times the columns' scales
    int row0 = g.bi * 128 + 64 * wr + 4 * half, col0 = g.bj * 128 + 32 * wc + sub;
    asm volatile("" : "+v"(row0), "+v"(col0));   // (addresses are formed here and not kept through the loop above)
    const int cb = col0 >> 6;
    const double inv_c = 1.0 / (double)g.scale[min(col0, g.D - 1)];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int i = row0 + 32 * t + 8 * (j >> 2) + (j & 3), ib = i >> 6;
        if (i < g.D && col0 < g.D && ib <= cb) {
          int64_t v = acc[0][t][j];
#pragma unroll
          for (int w = 1; w < 5; ++w) v = v * 256 + acc[w][t][j];
          // (powers of two, 1 to 2^126: their reciprocals are exact)
          const double x = (double)v * (1.0 / (double)g.scale[i]) * inv_c;
          double* o = g.out + (size_t)upper_block(g.nb, ib, cb) * 4096 + (i & 63) * 64 + (col0 & 63);
          if (seg == g.t_begin) *o = x; else *o += x;
        }
      }
  }
  if (DIAG && blk == 0 && lane == 0) {
    g.rest_count[tq] = n_rest;
    g.marks[tq * g.n_marks + (g.t_end - g.t_begin + 255) / 256] = n_rest;
    if (n_rest > g.rest_cap) __hip_atomic_store(g.flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <int EB>
__global__ __launch_bounds__(512, 2) void gram_digits_kernel(const void* __restrict__ K, const float* __restrict__ scale,
                                                             double* __restrict__ part, RestLists rest,
                                                             int32_t* __restrict__ rest_count, int32_t* __restrict__ marks,
                                                             int32_t* __restrict__ flags, int s, int D, int nb, int nb2,
                                                             int tokens_per_split, int n_splits, int batch, int rest_cap,
                                                             int n_marks) {
  extern __shared__ __align__(16) uint8_t lds[];             // [2 stages][2 column blocks][3 digits][64 pairs][128]
  __shared__ int32_t raised;
  const int tiles = nb2 * (nb2 + 1) / 2, groups = batch * n_splits;
  int group, tile;
  if (groups % 8 == 0) {
    const int j = blockIdx.x >> 3;
    group = (blockIdx.x & 7) + 8 * (j / tiles); tile = j % tiles;
  } else {
    group = blockIdx.x / tiles; tile = blockIdx.x % tiles;
  }
  const int b = group / n_splits, split = group % n_splits;
  if (threadIdx.x == 0) raised = __hip_atomic_load(&flags[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (raised) return;   // (gram_kernel forms this sequence's sums)
  GramTile g;
  // diagonal tiles first (they may raise the flag), then row by row
  if (tile < nb2) { g.bi = g.bj = tile; }
  else {
    int p = tile - nb2;
    g.bi = 0;
    while (p >= nb2 - 1 - g.bi) { p -= nb2 - 1 - g.bi; ++g.bi; }
    g.bj = g.bi + 1 + p;
  }
  g.K = static_cast<const uint8_t*>(K) + (size_t)b * s * D * EB;
  g.scale = scale + (size_t)b * D;
  g.out = part + ((size_t)split * batch + b) * (nb * (nb + 1) / 2) * 4096;
  const size_t lists = ((size_t)group * nb2 + g.bi) * 4 * rest_cap;
  g.rest = RestLists{rest.where + lists, rest.rest + lists};
  g.rest_count = rest_count + ((size_t)group * nb2 + g.bi) * 4;
  g.marks = marks + ((size_t)group * nb2 + g.bi) * 4 * n_marks;
  g.n_marks = n_marks;
  g.flag = flags + b;
  g.s = s; g.D = D; g.nb = nb; g.rest_cap = rest_cap;
  g.t_begin = split * tokens_per_split; g.t_end = min(s, g.t_begin + tokens_per_split);
  if (g.bi == g.bj) gram_digits_tile<EB, true>(g, lds);
  else gram_digits_tile<EB, false>(g, lds);
}

// ---- what the digits miss, by column ---------------------------------------------------------------------
// The lists of one block of 128 columns (four of each token part) as one, sorted by column; within a column the order is
// that of the walk below, the same on every run, and so is that of the sums.  by_col [b][nb2][n_lists * rest_cap]: places in the
// sequence's lists; col_begin [b][nb2][129].  32 lists at a time, 64 entries of each, go through LDS; eight threads per column,
// each with four of the 32 lists, count their entries and then place them.  (A thread per column for all lists: 250 us at
// 16 x 128K x 1024, 80 at 1 x 32K.)
__global__ __launch_bounds__(1024) void rest_by_column_kernel(const uint32_t* __restrict__ where, const int32_t* __restrict__ rest_count,
                                                              const int32_t* __restrict__ flags, uint32_t* __restrict__ by_col,
                                                              int32_t* __restrict__ col_begin, int nb2, int n_splits, int rest_cap) {
  constexpr int kLists = 32, kTake = 64, kShare = kLists / 8;
  __shared__ uint8_t buf[kLists][kTake];
  __shared__ int32_t have[kLists];
  __shared__ int32_t counts[8][128];
  const int bi = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, c = tid & 127, share = tid >> 7;
  const int n_lists = 4 * n_splits;
  if (flags[b]) return;
  const size_t first_list = (size_t)b * n_splits * nb2 * 4;   // of the sequence
  auto list_of = [&](int l) { return (((size_t)(l >> 2)) * nb2 + bi) * 4 + (l & 3); };
  auto walk = [&](auto&& each) {
    for (int l0 = 0; l0 < n_lists; l0 += kLists) {
      __syncthreads();
      if (tid < kLists) have[tid] = l0 + tid < n_lists ? min(rest_count[first_list + list_of(l0 + tid)], rest_cap) : 0;
      __syncthreads();
      int most = 0;
      for (int l = 0; l < kLists; ++l) most = max(most, have[l]);
      for (int p0 = 0; p0 < most; p0 += kTake) {
        if (p0) __syncthreads();
        const int l = tid >> 5, n = min(have[l] - p0, kTake);   // 32 threads copy a list
        if (n > 0) {
          const uint32_t* src = where + (first_list + list_of(l0 + l)) * rest_cap + p0;
          for (int i = tid & 31; i < n; i += 32) buf[l][i] = (uint8_t)(src[i] & 127u);
        }
        __syncthreads();
        for (int m = kShare * share; m < kShare * share + kShare; ++m)
          for (int i = 0; i < min(have[m] - p0, kTake); ++i)
            if (buf[m][i] == c) each(l0 + m, p0 + i);
      }
    }
  };
  int n = 0;
  walk([&](int, int) { ++n; });
  counts[share][c] = n;
  __syncthreads();
  int at = 0;   // entries of the columns before this one, then of this column's shares before this one
  for (int i = 0; i < c; ++i)
#pragma unroll
    for (int x = 0; x < 8; ++x) at += counts[x][i];
  int32_t* begin = col_begin + ((size_t)b * nb2 + bi) * 129;
  if (share == 0) begin[c] = at;
  for (int x = 0; x < share; ++x) at += counts[x][c];
  if (tid == 1023) begin[128] = at + n;
  uint32_t* dst = by_col + ((size_t)b * nb2 + bi) * n_lists * rest_cap;
  walk([&](int l, int i) { dst[at++] = (uint32_t)(list_of(l) * rest_cap + i); });
}

// G[b][i][j] = sum over the splits of the block that holds (i, j), plus what the digits miss, written to (j, i) as well.  One
// 32 x 32 tile on or above the diagonal per workgroup; the mirrored copy goes through LDS so that both are written in rows.
// (Reading the mirrored element per thread instead took 165 us for 32 splits of 1024 columns.)
template <int EB>
__global__ __launch_bounds__(256) void gram_finish_kernel(const double* __restrict__ part, double* __restrict__ G,
                                                          const void* __restrict__ K, const float* __restrict__ scale,
                                                          RestLists rest, const uint32_t* __restrict__ by_col,
                                                          const int32_t* __restrict__ col_begin,
                                                          const int32_t* __restrict__ flags, int s, int D, int nt, int nb, int nb2,
                                                          int n_splits, int batch, int rest_cap) {
  constexpr int kDeep = 16;
  __shared__ double tile[32][33];
  __shared__ int32_t strip_begin[33];
  __shared__ uint32_t strip_token[32 * kDeep];
  __shared__ float strip_rest[32 * kDeep];
  int p = blockIdx.x, ti = 0;   // tile index -> (ti, tj), ti <= tj, row by row of the upper triangle
  while (p >= nt - ti) { p -= nt - ti; ++ti; }
  const int tj = ti + p, b = blockIdx.y;
  const int x = threadIdx.x & 31, y0 = threadIdx.x >> 5;
  const size_t off = (size_t)b * D * D, pairs = (size_t)nb * (nb + 1) / 2;
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
  // the tile's quarter of the 64 x 64 block that holds it
  const double* src = part + (b * pairs + upper_block(nb, ti >> 1, tj >> 1)) * 4096 + ((ti & 1) * 32 + y0) * 64 + (tj & 1) * 32 + x;
#pragma unroll 4
  for (int sp = 0; sp < n_splits; ++sp)
#pragma unroll
    for (int u = 0; u < 4; ++u) sum[u] += src[(size_t)sp * batch * pairs * 4096 + 8 * u * 64];
  if (!flags[b]) {
    // h[u] = H(row, col) = sum over the listed elements (t, row) of r_t,row (K - R / 2)(t, col): rows y0 + 8 u of strip sr,
    // column x of strip sc.  The strip's entries go through LDS, kDeep of each row at a time, so that only the keys are waited
    // for: 311 us at 16 x 128K x 1024, 519 with each thread following its column's places in the lists by itself; 437 at
    // 3 x 1M x 1024, 710 with the strip's entries in order, where a column's many leave the other rows idle.
    auto missed = [&](int sr, int sc, double (&h)[4]) {
      const float sx = scale[(size_t)b * D + sc * 32 + x];
      const double inv = 0.5 / (double)sx;
      const uint32_t* list = by_col + ((size_t)b * nb2 + (sr >> 2)) * 4 * n_splits * rest_cap;
      const size_t first = (size_t)b * n_splits * nb2 * 4 * rest_cap;   // entry of the sequence's lists
      const int32_t* begin = col_begin + ((size_t)b * nb2 + (sr >> 2)) * 129 + (sr & 3) * 32;
      __syncthreads();
      if (threadIdx.x < 33) strip_begin[threadIdx.x] = begin[threadIdx.x];
      __syncthreads();
      int most = strip_begin[(threadIdx.x & 31) + 1] - strip_begin[threadIdx.x & 31];
#pragma unroll
      for (int m = 16; m >= 1; m >>= 1) most = max(most, __shfl_xor(most, m, kWave));
      float inv_row[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        inv_row[u] = 1.0f / scale[(size_t)b * D + sr * 32 + y0 + 8 * u];
        h[u] = 0.0;
      }
      for (int k0 = 0; k0 < most; k0 += kDeep) {
        if (k0) __syncthreads();
        for (int i = threadIdx.x; i < 32 * kDeep; i += 256) {
          const int at = strip_begin[i / kDeep] + k0 + i % kDeep;
          if (at < strip_begin[i / kDeep + 1]) {
            const size_t place = first + list[at];
            strip_token[i] = rest.where[place] >> 7;
            strip_rest[i] = bf16_to_f32(rest.rest[place]);
          }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int row = y0 + 8 * u, n = min(kDeep, strip_begin[row + 1] - strip_begin[row] - k0);
#pragma unroll 4
          for (int i = 0; i < n; ++i) {
            const float k = kv_elem<EB>(K, ((size_t)b * s + strip_token[row * kDeep + i]) * D + sc * 32 + x);
            h[u] = fma((double)(strip_rest[row * kDeep + i] * inv_row[u]), (double)k - inv * (double)digit_rest(k, sx), h[u]);
          }
        }
      }
    };
    double h[4];
    missed(ti, tj, h);
#pragma unroll
    for (int u = 0; u < 4; ++u) sum[u] += h[u];
    if (ti != tj) missed(tj, ti, h);
#pragma unroll
    for (int u = 0; u < 4; ++u) tile[y0 + 8 * u][x] = h[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) sum[u] += tile[x][y0 + 8 * u];
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    G[off + (size_t)(ti * 32 + y0 + 8 * u) * D + tj * 32 + x] = sum[u];
    tile[y0 + 8 * u][x] = sum[u];
  }
  if (ti == tj) return;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) G[off + (size_t)(tj * 32 + y0 + 8 * u) * D + ti * 32 + x] = tile[x][y0 + 8 * u];
}

}  // namespace skv
