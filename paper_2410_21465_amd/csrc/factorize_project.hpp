// A = K Psi on the 8-bit integer matrix instruction: the keys as in factorize_gram.hpp (three digits, columns scaled by powers
// of two, lists of what the digits leave out), each right singular vector as seven 8-bit digits of Psi / (its column's power
// of two), 54 bits below the vector's largest such number.  (Cutting the operands of a product into integers whose products
// and sums are exact is the splitting of Ozaki, Ogita, Oishi and Rump, 2012.)  Every sum of digit products is exact; what is
// lost is the rounding of Psi to those digits, and that of adding the sums and what the lists hold in fp64.  Measured against
// the result's root mean square that is less than fp64 sums lose: against 64-bit-mantissa sums 1.3e-16 to 6e-16 for key widths
// 128 to 3072, columns of like and of graded scale, where sums in fp64 are off by 4e-16 to 1.7e-15.
// Entry by entry it can be more: where one column is far above the others, its component of the vector takes the leading
// bits, the other components have few or none left, and a token that is zero in that column has only those.  So every entry is
// held against a bound of its own: an error of half a unit per component makes at most N / 2 units, N the sum of the token's
// digit numbers.  An entry smaller than 2^kSureBits times that is summed again from the keys and the vector in fp64; a wave
// with more than kAgain such entries raises the sequence's flag, and project_kernel forms the whole sequence's A.
// 16 x 128K x 1024, the call: normal keys 25.08 -> 25.24 ms; one token with a key of 2^26 times the others in a column that
// is zero elsewhere, where the entries of its vector came out wrong, 26.6 -> 31.8.
#pragma once
#include "factorize_gram.hpp"

namespace skv {

// Digits of the vectors, 32 vectors x 64 columns at a time, as they lie in LDS: seven planes (the most significant digit first)
// of 32 vectors x 64 columns in operand_at's order, then the columns' scale words.  psi_digits [b][nt][stages][kPsiStage].
constexpr int kPsiDigits = 7, kPsiPlane = 32 * 64, kPsiScale = kPsiDigits * kPsiPlane, kPsiStage = kPsiScale + 64 * 4;
constexpr int kPsiDeep = 4;   // stages between barriers
constexpr int kSureBits = 24; // an entry from digits is off by less than 2^-24 of its value
constexpr int kAgain = 16;    // entries that a wave sums again, of 1024 (not searched: keys either need hardly any or whole vectors)
// flags[b]: the digits do not hold the sequence's keys; its entries of A need more bits of the vectors than these have
constexpr int kFlagKeys = 1, kFlagVectors = 2;
// One workgroup per vector (those past r are zero).  exps [b][32 nt]: the digits stand for Psi 2^(exps - sh).
template <int EB>
__global__ __launch_bounds__(256) void psi_digits_kernel(const double* __restrict__ Psi_t, const float* __restrict__ scale,
                                                         uint8_t* __restrict__ psi_digits, int32_t* __restrict__ exps, int D, int r,
                                                         int nt) {
  __shared__ double most[4];
  const int rho = blockIdx.x, b = blockIdx.y, stages = (D + 63) / 64;
  const double* v = Psi_t + ((size_t)b * r + min(rho, r - 1)) * D;
  const float* sc = scale + (size_t)b * D;
  double m = 0.0;
  for (int x = threadIdx.x; x < D; x += 256) m = fmax(m, fabs(v[x]) / (double)sc[x]);
  m = wave_max_f64(m);
  if ((threadIdx.x & 63) == 0) most[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmax(fmax(most[0], most[1]), fmax(most[2], most[3]));
  // every digit number is below 2^54 (a vector of zeros is exact: no bound on its entries)
  const int e = rho < r && m > 0.0 ? 54 - __builtin_amdgcn_frexp_exp(m) : 4096;
  if (threadIdx.x == 0) exps[(size_t)b * nt * 32 + rho] = e;
  uint8_t* out = psi_digits + ((size_t)b * nt + rho / 32) * stages * kPsiStage;
  for (int c0 = 4 * threadIdx.x; c0 < 64 * stages; c0 += 1024) {
    uint64_t w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double x = rho < r && c0 + u < D ? ldexp(v[min(c0 + u, D - 1)] / (double)sc[min(c0 + u, D - 1)], e) : 0.0;
      w[u] = (uint64_t)(int64_t)rint(x) + 0x0080808080808080ull;   // bytes: the digits + 128
    }
    uint8_t* st = out + (size_t)(c0 / 64) * kPsiStage;
#pragma unroll
    for (int q = 0; q < kPsiDigits; ++q) {
      uint32_t d = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) d |= (uint32_t)((w[u] >> (8 * (kPsiDigits - 1 - q))) & 0xff) << (8 * u);
      *reinterpret_cast<uint32_t*>(st + q * kPsiPlane + operand_at(rho & 31, (c0 & 63) >> 4) + (c0 & 15)) = d ^ 0x80808080u;
    }
    if ((rho & 31) == 0)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        reinterpret_cast<uint32_t*>(st + kPsiScale)[(c0 & 63) + u] = c0 + u < D ? Piece<EB>::scale_word(u, sc[c0 + u]) : 0u;   // (digits of zeros)
  }
}

// A workgroup of eight waves owns 256 tokens (of one token part of the Gram matrix, so that the lists' marks fit) and 32
// vectors; a wave 32 tokens, whose keys it takes from memory straight into operand order (a lane: 16 neighbouring columns of
// one token), cuts into digits and multiplies with the vectors' digits in LDS: 21 products of 32 x 32 x 32 per 32 columns,
// nine sums by weight (144 registers).  The keys are cut once per 32 vectors, which costs less than a trip through LDS.  The
// workgroups of the same tokens run side by side on one XCD.
// 16 x 128K x 1024, rank 160: 7.7 ms where the fp64 sums took 11.5; 1 x 32K: 0.142 and 0.196 ms.  The products alone take 4.5 to
// 5.2 ms (at the clock the chip holds with its matrix cores this busy, about 2 GHz); the rest is waiting for keys (1.4 ms) and
// for the vectors' digits (0.4), and what the lists add (0.3).  Barriers every stage instead of every fourth: 1.5 % more.
template <int EB>
__global__ __launch_bounds__(512, 2) void project_digits_kernel(const void* __restrict__ K, const uint8_t* __restrict__ psi_digits,
                                                                const int32_t* __restrict__ exps, const double* __restrict__ Psi_t,
                                                                RestLists rest, const int32_t* __restrict__ marks,
                                                                int32_t* __restrict__ flags, const float* __restrict__ scale,
                                                                void* __restrict__ Aout, int s, int s_cap, int D, int r, int nt,
                                                                int nb2, int tokens_per_split, int n_splits, int batch,
                                                                int rest_cap, int n_marks) {
  constexpr int kPieces = kPsiStage / 16, kEntries = 64;
  extern __shared__ __align__(16) uint8_t lds[];   // [2][kPsiDeep][kPsiStage]
  struct Entry { uint32_t where, rest; };   // as in the lists
  __shared__ Entry entries[kEntries];
  __shared__ int32_t columns[kEntries];
  __shared__ double products[kEntries][32];
  __shared__ int32_t list_n[512];
  __shared__ int32_t raised;
  const int per_split = n_marks - 1, j = blockIdx.x >> 3, n = j % nt, block = (j / nt) * 8 + (blockIdx.x & 7);
  if (block >= batch * n_splits * per_split) return;
  const int group = block / per_split, in_split = block % per_split, b = group / n_splits, split = group % n_splits;
  // (another workgroup may raise kFlagVectors at any time, kFlagKeys is settled)
  if (flags[b] == kFlagKeys) return;
  const int flag = threadIdx.x == 0 ? __hip_atomic_load(&flags[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  const int t_begin = split * tokens_per_split + in_split * 256;
  const int t_end = min(min(s, (split + 1) * tokens_per_split), t_begin + 256);
  if (t_begin >= t_end) return;
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int sub = lane & 31, half = lane >> 5, stages = (D + 63) / 64;
  const uint8_t* src = psi_digits + ((size_t)b * nt + n) * stages * kPsiStage;
  // (tokens past the end repeat the last one: their results are not written)
  const uint8_t* row = static_cast<const uint8_t*>(K) + ((size_t)b * s + min(t_begin + 32 * wave + sub, s - 1)) * D * EB;

  uint4 next_b0, next_b1;   // (an array of the two was kept in scratch memory)
  auto request_b = [&](int st) {
    const uint4* p = reinterpret_cast<const uint4*>(src + (size_t)min(st, stages - 1) * kPsiStage);
    next_b0 = p[threadIdx.x];
    next_b1 = p[min((int)threadIdx.x + 512, kPieces - 1)];
  };
  auto put_b = [&](int st) {
    uint4* p = reinterpret_cast<uint4*>(lds + st % (2 * kPsiDeep) * kPsiStage);
    p[threadIdx.x] = next_b0;
    p[min((int)threadIdx.x + 512, kPieces - 1)] = next_b1;   // (several threads the last piece: the same bytes)
  };
  using Raw = Piece<EB>[2][2];
  Raw raw0, raw1;   // this lane's keys of the stage at hand and the next
  auto request_k = [&](Raw& raw, int st) {   // (columns past the end repeat the last ones: scaled by zero, and their digits of Psi are zero)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int x = 0; x < 2; ++x) raw[kk][x].load(row + (size_t)(min(64 * st + 32 * kk, D - 32) + 16 * half + 8 * x) * EB);
  };
  i32x16 acc[9];
#pragma unroll
  for (int g = 0; g < 9; ++g)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[g][i] = 0;
  // this thread's list of what the digits left out: its part for these tokens, and the first entry of that
  const int n_lists = 4 * nb2;
  int from = 0, to = 0;
  Entry first{};
  auto find = [&](int l0) {
    const size_t list = (size_t)group * n_lists + min(l0 + (int)threadIdx.x, n_lists - 1);
    from = marks[list * n_marks + in_split];
    to = l0 + (int)threadIdx.x < n_lists ? marks[list * n_marks + in_split + 1] : from;
    if (from < to) first = Entry{rest.where[list * rest_cap + from], rest.rest[list * rest_cap + from]};
  };
  request_k(raw0, 0);
  find(0);
#pragma unroll 1
  for (int st = 0; st < kPsiDeep; ++st) { request_b(st); put_b(st); }
  if (threadIdx.x == 0) raised = flag;
  __syncthreads();
  if (raised) return;
  auto stage = [&](const Raw& raw, Raw& next, int st) {
    const uint8_t* plane = lds + st % (2 * kPsiDeep) * kPsiStage;
    request_b(st + kPsiDeep);
    request_k(next, st + 1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      i32x4 a[3];
      const uint4* words = reinterpret_cast<const uint4*>(plane + kPsiScale) + 8 * kk + 4 * half;
      each_of(std::make_integer_sequence<int, 4>{}, [&](auto y_tag) {   // four columns at a time
        constexpr int y = y_tag, c = 4 * (y & 1);
        const uint4 sw = words[y];
        const Piece<EB>& p = raw[kk][y / 2];
        uint32_t w[4];
        if constexpr (EB == 2) {
          scaled4_bf16({p.w[c / 2], p.w[c / 2], p.w[c / 2 + 1], p.w[c / 2 + 1]}, {sw.x, sw.y, sw.z, sw.w}, w);
        } else {
          w[0] = scaled_e5m2<0>(p.w[c / 4], sw.x); w[1] = scaled_e5m2<1>(p.w[c / 4], sw.y);
          w[2] = scaled_e5m2<2>(p.w[c / 4], sw.z); w[3] = scaled_e5m2<3>(p.w[c / 4], sw.w);
        }
        uint32_t d[3];
        split_digits(w, d);
#pragma unroll
        for (int x = 0; x < 3; ++x) a[x][y] = (int)d[x];
      });
      i32x4 bq[kPsiDigits];
#pragma unroll
      for (int q = 0; q < kPsiDigits; ++q) bq[q] = *reinterpret_cast<const i32x4*>(plane + q * kPsiPlane + operand_at(sub, 2 * kk + half));
      // (in this order no product waits for the sum of one of the six before it)
#pragma unroll
      for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int q = 0; q < kPsiDigits; ++q) acc[x + q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[x], bq[q], acc[x + q], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    put_b(st + kPsiDeep);
    if (st % kPsiDeep == kPsiDeep - 1) __syncthreads();   // (the stages just read are written over from here on)
  };
#pragma unroll 1
  for (int st = 0; st < stages; st += 2) {
    stage(raw0, raw1, st);
    if (st + 1 < stages) stage(raw1, raw0, st + 1);
  }
  __syncthreads();
  const int rho = 32 * n + sub;
  const int e = exps[(size_t)b * nt * 32 + rho];
  // the nine sums from the most significant one down: the first three steps are exact (below 2^53 for every width), the others
  // round once each
  double v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    v[i] = (double)acc[0][i];
#pragma unroll
    for (int g = 1; g < 9; ++g) v[i] = fma(v[i], 256.0, (double)acc[g][i]);
    v[i] = ldexp(v[i], -e);
  }
  // what the digits of these tokens' keys left out, in the order of the lists: the entries and their products with the
  // vectors go through LDS, kEntries at a time, and each wave adds those of its tokens
  for (int l0 = 0; l0 < n_lists; l0 += 512) {
    if (l0) find(l0);
    __syncthreads();
    list_n[threadIdx.x] = to - from;
    __syncthreads();
    int at = 0, total = 0;
    for (int i = 0; i < min(512, n_lists - l0); ++i) { at += i < (int)threadIdx.x ? list_n[i] : 0; total += list_n[i]; }
    for (int c0 = 0; c0 < total; c0 += kEntries) {
      if (c0) __syncthreads();
      for (int i = max(from, from + c0 - at); i < min(to, from + c0 + kEntries - at); ++i) {
        const int l = l0 + threadIdx.x;
        const size_t place = ((size_t)group * n_lists + l) * rest_cap + i;
        entries[at + (i - from) - c0] = i == from ? first : Entry{rest.where[place], rest.rest[place]};
        columns[at + (i - from) - c0] = (l >> 2) * 128;
      }
      __syncthreads();
      const int here = min(kEntries, total - c0);
      for (int i = threadIdx.x; i < 32 * here; i += 512) {
        const Entry x = entries[i >> 5];
        const int col = columns[i >> 5] + (int)(x.where & 127u);
        const double psi = Psi_t[((size_t)b * r + min(32 * n + (i & 31), r - 1)) * D + col], sc = (double)scale[(size_t)b * D + col];
        products[i >> 5][i & 31] = (double)__uint_as_float(x.rest << 16) / sc * psi;
      }
      __syncthreads();
      for (int i = 0; i < here; ++i) {
        const int token = __builtin_amdgcn_readfirstlane((int)(entries[i].where >> 7)) - t_begin;
        if (token >> 5 != wave) continue;
        const double x = products[i][sub];
#pragma unroll
        for (int y = 0; y < 16; ++y) v[y] += (token & 31) == 8 * (y >> 2) + 4 * half + (y & 3) ? x : 0.0;
      }
    }
  }
  // Entries that their bound does not vouch for: held against the most that a token can have first, and where that leaves many
  // (a token of zeros is exact, and a faint one has less), against what each token has.  (Summing the magnitudes along with
  // the products took 3 % of the kernel.)
  const double unit = ldexp(1.0, kSureBits - 1 - e);
  uint32_t unsure = 0;
  int n_unsure = 0;
  auto look = [&](auto&& bound) {   // bound(x): N of the wave's token x
    unsure = 0; n_unsure = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int x = 8 * (i >> 2) + 4 * half + (i & 3);
      const bool low = fabs(v[i]) < unit * (double)bound(x) && rho < r && t_begin + 32 * wave + x < t_end;
      unsure |= low ? 1u << i : 0u;
      n_unsure += __popcll(__ballot(low));
    }
  };
  double least = fabs(v[0]);
#pragma unroll
  for (int i = 1; i < 16; ++i) least = fmin(least, fabs(v[i]));
  if (__any(least < unit * (double)(4194304.0f * (float)D))) look([&](int) { return 4194304.0f * (float)D; });
  if (n_unsure > kAgain) {
    const uint8_t* first_row = static_cast<const uint8_t*>(K) + (size_t)b * s * D * EB;
    uint32_t present = 0;   // tokens that are not all zeros
    for (int x0 = 0; x0 < 32; x0 += 8)
      for (int c0 = 0; c0 < D; c0 += 8 * kWave) {
        Piece<EB> p[8];
#pragma unroll
        for (int x = 0; x < 8; ++x)
          p[x].load(first_row + ((size_t)min(t_begin + 32 * wave + x0 + x, s - 1) * D + min(c0 + 8 * lane, D - 8)) * EB);
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          uint32_t any = 0;
#pragma unroll
          for (int i = 0; i < 2 * EB; ++i) any |= p[x].w[i] & (EB == 2 ? 0x7fff7fffu : 0x7f7f7f7fu);
          present |= __any(any != 0) ? 1u << (x0 + x) : 0u;
        }
      }
    look([&](int x) { return present >> x & 1 ? 4194304.0f * (float)D : 0.0f; });
    if (n_unsure > kAgain) {
      float sum = 0.0f;   // of half of token `sub`
#pragma unroll 4
      for (int c = half * (D / 2); c < (half + 1) * (D / 2); c += 8) {
        Piece<EB> p;
        p.load(row + (size_t)c * EB);
        const float* sc = scale + (size_t)b * D + c;
        each_of(std::make_integer_sequence<int, 8>{}, [&](auto x) { sum += fabsf(fmaf(p.template elem<x>(), sc[x], kDigitMagic) - kDigitMagic); });
      }
      sum += __shfl_xor(sum, 32, kWave);
      look([&](int x) { return __shfl(sum, x, kWave); });
    }
  }
  if (n_unsure > kAgain) {
    if (lane == 0) __hip_atomic_store(&flags[b], kFlagVectors, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (n_unsure) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      uint64_t which = __ballot(unsure >> i & 1);
      while (which) {
        const int l = __ffsll((unsigned long long)which) - 1;
        which &= which - 1;
        const size_t t = (size_t)b * s + t_begin + 32 * wave + 8 * (i >> 2) + 4 * (l >> 5) + (i & 3);
        const double* psi = Psi_t + ((size_t)b * r + 32 * n + (l & 31)) * D;
        double sum = 0.0;
#pragma unroll 4
        for (int x = lane; x < D; x += kWave) sum = fma((double)kv_elem<EB>(K, t * D + x), psi[x], sum);
        sum = wave_sum_f64(sum);
        v[i] = lane == l ? sum : v[i];
      }
    }
  }
  if (rho >= r) return;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int t = t_begin + 32 * wave + 8 * (i >> 2) + 4 * half + (i & 3);
    if (t < t_end) kv_store_elem<EB>(Aout, ((size_t)b * s_cap + t) * r + rho, v[i]);
  }
}

}  // namespace skv
