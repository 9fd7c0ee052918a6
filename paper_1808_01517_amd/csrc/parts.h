// FP32 arithmetic on the bfloat16 matrix cores.
//
// x = x0 + x1 + x2 with each part the bfloat16 rounding (RNE) of what the
// parts before it leave, so |x1| <= 2^-9 |x|, |x2| <= 2^-18 |x| and the three
// hold all 24 bits, down to |x| = 2^-109 (below, x2's lie under bfloat16's
// smallest number, 2^-133).  A product takes the six part products above 2^-26 of it
// (kPartA, kPartB); the three left out are below float32's own rounding of
// the product.  x0 y0 goes to one accumulator and the other five, at most
// 2^-8 of it, to a second, added at the end: the long sum then has one
// float32 rounding per 32 k, where the float32 instructions have 32.  (All
// six in one accumulator, which the matrix core truncates as it adds, was
// further from float64 than the float32 instructions on long sums: 1.0e-6
// against 7.3e-7 on a weight gradient over 8192 voxels.)
//
// Six 16x16x32 bfloat16 instructions take 96 matrix-core cycles per 32 k
// where eight 16x16x4 float32 ones take 256.
//
// Infinities, NaN and values that round to an infinite x0 end as NaN here, and
// an operand below 2^-109 is off by up to 2^-134.  Kernels look for results
// that are not finite, or not zero and below 2^-80 (any_odd), and compute those
// again with the float32 instructions from the values themselves
// (activations, and the table's beside its parts), so that float32's rules
// hold.  (A result above 2^-80 is off by less than float32's rounding unless
// the sum of the factors beside such operands exceeds 2^30.)
#pragma once

#include "gemm_common.h"

namespace dlm {

constexpr int kProducts = 6;
constexpr int kPartA[kProducts] = {2, 0, 1, 1, 0, 0};
constexpr int kPartB[kProducts] = {0, 2, 1, 0, 1, 0};

// Two floats rounded to bfloat16 (RNE) in one instruction, lo in the low half;
// with REST they become what the rounding leaves (exact).
template <bool REST>
__device__ __forceinline__ uint32_t part2(float &lo, float &hi) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 h2 __attribute__((ext_vector_type(2)));
  const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, h2));
  if constexpr (REST) {
    lo -= __builtin_bit_cast(float, w << 16);
    hi -= __builtin_bit_cast(float, w & 0xffff0000u);
  }
  return w;
}

__device__ __forceinline__ void split3(floatx4 lo, floatx4 hi, bf16x8 (&p)[3]) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  u4 w[3];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x = e < 2 ? lo[2 * e] : hi[2 * e - 4], y = e < 2 ? lo[2 * e + 1] : hi[2 * e - 3];
    w[0][e] = part2<true>(x, y);
    w[1][e] = part2<true>(x, y);
    w[2][e] = part2<false>(x, y);
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) p[i] = __builtin_bit_cast(bf16x8, w[i]);
}

// The 16 x 16 x 32 step of NI x NJ tiles (columns j0 .. of the wave's) in its
// six part products: hi += a0 b0, lo += the rest.
template <int NI, int NJ, int TN>
__device__ __forceinline__ void mma_parts(const bf16x8 (&a)[NI][3], const bf16x8 (&b)[NJ][3], floatx4 (&hi)[NI][TN],
                                          floatx4 (&lo)[NI][TN], int j0) {
#pragma unroll
  for (int u = 0; u < kProducts; ++u)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (j0 + j >= TN) continue;
        floatx4 &c = u == kProducts - 1 ? hi[i][j0 + j] : lo[i][j0 + j];
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][kPartB[u]], a[i][kPartA[u]], c, 0, 0, 0);
      }
}

// The same with one accumulator: the step's six products are summed from
// zero, small ones first, and added to it in float32 (RNE).  It takes half the
// accumulator registers and one vector add per value and step.  SWAP: the A
// operand first (a lane holds four rows of one column, not four columns of a
// row).  The matrix unit cuts what lies below its sum off towards minus
// infinity, which adds up over the steps where the sum itself hardly grows:
// the caller negates A in every other step (flip_sign) and gives sign = -1 for
// it, and the cuts cancel.  Weight gradient of 43 521 voxels, 1 -> 8 channels,
// against 64 bits: 6e-7 without, 1.3e-7 with it (float32 instruction 3e-7); of
// 1M voxels, 3 -> 32 channels, 3e-7 (1.1e-6).
template <bool SWAP, int NI, int NJ, int TN>
__device__ __forceinline__ void mma_parts_sum(const bf16x8 (&a)[NI][3], const bf16x8 (&b)[NJ][3],
                                              floatx4 (&acc)[NI][TN], int j0, float sign) {
  floatx4 c[NI][NJ];
#pragma unroll
  for (int u = 0; u < kProducts; ++u)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (j0 + j >= TN) continue;
        const bf16x8 x = SWAP ? a[i][kPartA[u]] : b[j][kPartB[u]], y = SWAP ? b[j][kPartB[u]] : a[i][kPartA[u]];
        c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, u == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : c[i][j], 0, 0, 0);
      }
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (j0 + j < TN)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j0 + j][e] = fmaf(sign, c[i][j][e], acc[i][j0 + j][e]);
}

__device__ __forceinline__ bf16x8 flip_sign(bf16x8 v, unsigned mask) {  // mask 0 or 0x80008000
  typedef unsigned words __attribute__((ext_vector_type(4)));
  words w = __builtin_bit_cast(words, v);
  w ^= mask;
  return __builtin_bit_cast(bf16x8, w);
}

template <int TM, int TN>
__device__ __forceinline__ void add_parts(floatx4 (&hi)[TM][TN], const floatx4 (&lo)[TM][TN]) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) hi[i][j] += lo[i][j];
}

// Whether a wave's tiles hold a value that is not finite, or not zero and
// below 2^-80.  Doubled, a value's bits are its magnitude's, and one less than
// them leaves zero above all others.
constexpr unsigned kTiny = (127u - 80u) << 24;
template <int TM, int TN>
__device__ __forceinline__ bool any_odd(const floatx4 (&acc)[TM][TN]) {
  float z = 0.0f;
  unsigned least = ~0u;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        z = fmaf(acc[i][j][e], 0.0f, z);
        least = min(least, (__builtin_bit_cast(unsigned, acc[i][j][e]) << 1) - 1u);
      }
  return __any(z != z || least < kTiny - 1u);
}
__device__ __forceinline__ bool not_finite(float v) { return (__builtin_bit_cast(unsigned, v) & 0x7f800000u) == 0x7f800000u; }
__device__ __forceinline__ bool is_odd(float v) {
  return not_finite(v) || (__builtin_bit_cast(unsigned, v) << 1) - 1u < kTiny - 1u;
}

// The slow path reads its operands from global memory, 16 rows of four k at a
// time: op.at(k, l) is the value of lane (q16, g4) of rows r .. r + 15 at
// k + g4, k a multiple of 4 and the same in all lanes, with l = op.lane(r, q16,
// g4) its place among them.  About kLoads of them are in flight: twice as many
// cost the cores' own loops registers and gained nothing.
constexpr int kLoads = 20;

// Which of 16 rows have a NaN among their k, one bit each; stops once all of
// `want` have.
template <class OP>
__device__ __forceinline__ unsigned nan_rows(const OP &op, int64_t r, int kbeg, int kend, unsigned want) {
  constexpr int kSteps = 16;
  const int lane = threadIdx.x & 63, q16 = lane & 15, g4 = lane >> 4;
  unsigned found = 0;
  auto add = [&](bool nan) {
    const uint64_t m = __ballot(nan);
    found |= (unsigned)(m | m >> 16 | m >> 32 | m >> 48) & 0xffffu;
  };
  const auto l = op.lane(r, q16, g4);
  int k = kbeg;
#pragma unroll 1
  for (; k + 4 * kSteps <= kend && (found & want) != want; k += 4 * kSteps) {
    bool nan = false;
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const float v = op.at(k + 4 * u, l);
      nan |= v != v;
    }
    add(nan);
  }
#pragma unroll 1
  for (; k < kend && (found & want) != want; k += 4) {
    const float v = op.at(k, op.lane(r, q16, min(g4, kend - 1 - k)));
    add(v != v);
  }
  return found;
}

// The same of 64 rows per word, a row per lane, in the first 16 k only (weights
// that have gone NaN are so all over).
template <int NM, class OP>
__device__ __forceinline__ void nan_heads(const OP &op, int64_t r, int kbeg, int kend, uint64_t (&m)[NM]) {
  const int lane = threadIdx.x & 63, q16 = lane & 15, g4 = lane >> 4;
#pragma unroll
  for (int p = 0; p < NM; ++p) {
    bool nan = false;
#pragma unroll 2
    for (int k = kbeg; k < min(kend, kbeg + 16); k += 4)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float v = op.at(k, op.lane(r + 64 * p + 16 * g4, q16, min(g, kend - 1 - k)));
        nan |= v != v;
      }
    m[p] = __ballot(nan);
  }
}

// TN 16 x 16 tiles beside each other in float32 (16x16x4).
template <bool SWAP, int TN, class AO, class BO>
__device__ __forceinline__ void redo_row(const AO &ao, const BO &bo, int64_t ra, int64_t rb, int kbeg, int kend,
                                         floatx4 (&c)[TN]) {
  constexpr int kSteps = kLoads / (1 + TN);
  const int lane = threadIdx.x & 63, q16 = lane & 15, g4 = lane >> 4;
#pragma unroll
  for (int j = 0; j < TN; ++j) c[j] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto mma = [&](int j, float a, float b) {
    c[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(SWAP ? a : b, SWAP ? b : a, c[j], 0, 0, 0);
  };
  const auto la = ao.lane(ra, q16, g4);
  int k = kbeg;
#pragma unroll 1
  for (; k + 4 * kSteps <= kend; k += 4 * kSteps) {
    float a[kSteps], b[TN][kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) a[u] = ao.at(k + 4 * u, la);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const auto lb = bo.lane(rb + 16 * j, q16, g4);
#pragma unroll
      for (int u = 0; u < kSteps; ++u) b[j][u] = bo.at(k + 4 * u, lb);
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u)
#pragma unroll
      for (int j = 0; j < TN; ++j) mma(j, a[u], b[j][u]);
  }
#pragma unroll 1
  for (; k < kend; k += 4) {
    const int g = min(g4, kend - 1 - k);
    const float a = ao.at(k, ao.lane(ra, q16, g));
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const float b = bo.at(k, bo.lane(rb + 16 * j, q16, g));
      mma(j, g == g4 ? a : 0.0f, g == g4 ? b : 0.0f);
    }
  }
}

__device__ __forceinline__ unsigned wave_or(unsigned x) {
  for (int off = 32; off > 0; off >>= 1) x |= __shfl_xor(x, off, 64);
  return x;
}

// Values of a wave's tiles that the parts may have got wrong, again in float32:
// every one below 2^-80, and every one that is not finite, unless a NaN in its row or column (rows below
// M, N) makes it NaN anyway.  Data with a background of NaN rows are ordinary
// (a division by a b = 0 signal of zero), so those cost a look at the rows;
// infinities cost a second, slower product of their 16 rows.  a_nan(i, r, want):
// those of the 16 rows from r, the wave's i-th group, that have a NaN.
// 65 536 voxels, 3 -> 32 channels, forward / input / weight gradient: finite
// 176 / 158 / 238 us, every other voxel NaN 234 / 160 / 260 (each tile computed
// again, four k at a time, whatever the reason: 4418 / 5507 / 2830), an infinity
// in every 1024th 545 / 352 / 761 (912 / 972 / 1159).
template <bool SWAP, int TM, int TN, class AO, class BO, class ANAN>
__device__ __forceinline__ void mend_odd(const AO &ao, const BO &bo, int64_t ra, int64_t rb, int64_t M, int64_t N, int kbeg,
                                         int kend, floatx4 (&acc)[TM][TN], ANAN a_nan) {
  const int lane = threadIdx.x & 63, q16 = lane & 15, g4 = lane >> 4;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t r = ra + 16 * i;
    unsigned odd[TN], rows = 0, any = 0;  // odd: the lane's values, four bits a tile; rows: the 16 with one not finite
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      odd[j] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int x = SWAP ? 4 * g4 + e : q16, y = 16 * j + (SWAP ? q16 : 4 * g4 + e);
        const bool o = is_odd(acc[i][j][e]) && r + x < M && rb + y < N;
        odd[j] |= (o ? 1u : 0u) << e;
        any |= o ? 1u : 0u;
        rows |= (o && not_finite(acc[i][j][e]) ? 1u : 0u) << x;
      }
    }
    if (!__any(any)) continue;
    rows = wave_or(rows);
    const unsigned na = rows ? a_nan(i, r, rows) : 0u;
    any = 0;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      odd[j] &= SWAP ? ~(na >> (4 * g4)) : (na >> q16 & 1 ? 0u : ~0u);
      any |= odd[j];
    }
    if (!__any(any)) continue;
    uint64_t heads[(TN + 3) / 4];
    nan_heads(bo, rb, kbeg, kend, heads);
    any = 0;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const unsigned nb = (unsigned)(heads[j / 4] >> (16 * (j % 4))) & 0xffffu;
      odd[j] &= SWAP ? (nb >> q16 & 1 ? 0u : ~0u) : ~(nb >> (4 * g4));
      any |= odd[j];
    }
    if (!__any(any)) continue;
    floatx4 c[TN];
    redo_row<SWAP>(ao, bo, r, rb, kbeg, kend, c);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = odd[j] >> e & 1 ? c[j][e] : acc[i][j][e];
  }
}

}  // namespace dlm
