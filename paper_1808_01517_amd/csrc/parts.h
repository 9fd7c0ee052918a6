// FP32 arithmetic on the bfloat16 matrix cores.
//
// x = x0 + x1 + x2 with each part the bfloat16 rounding (RNE) of what the
// parts before it leave, so |x1| <= 2^-9 |x|, |x2| <= 2^-18 |x| and the three
// hold all 24 bits.  A product takes the six part products above 2^-26 of it
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
// Infinities, NaN and values that round to an infinite x0 end as NaN here;
// kernels look for results that are not finite (bad_tiles) and compute those
// tiles again with the float32 instructions from the values themselves
// (activations, and the table's beside its parts), so that float32's rules
// hold.
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

// Which of a wave's tiles hold a value that is not finite, one bit each.
template <int TM, int TN>
__device__ __forceinline__ uint64_t bad_tiles(const floatx4 (&acc)[TM][TN]) {
  static_assert(TM * TN <= 64, "one bit per tile");
  float z = 0.0f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) z = fmaf(acc[i][j][e], 0.0f, z);
  if (!__any(z != z)) return 0;
  uint64_t bad = 0;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const floatx4 v = acc[i][j];
      const float y = ((v[0] * 0.0f + v[1] * 0.0f) + v[2] * 0.0f) + v[3] * 0.0f;
      if (__any(y != y)) bad |= uint64_t(1) << (i * TN + j);
    }
  return bad;
}

// Tiles `bad` of a wave again, in float32 from global memory (16x16x4, k in
// order).  Never taken for finite results, so its speed does not matter.
template <bool SWAP, class AO, class BO>
__device__ __attribute__((noinline)) floatx4 redo_tile(const AO ao, const BO bo, int64_t ra, int64_t rb, int kbeg,
                                                       int kend) {
  const int lane = threadIdx.x & 63, q16 = lane & 15, g4 = lane >> 4;
  floatx4 c{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int k0 = kbeg; k0 < kend; k0 += 4) {
    const int k = k0 + g4;
    const float a = k < kend ? ao.at(ra + q16, k) : 0.0f;
    const float b = k < kend ? bo.at(rb + q16, k) : 0.0f;
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(SWAP ? a : b, SWAP ? b : a, c, 0, 0, 0);
  }
  return c;
}

template <bool SWAP, int TM, int TN, class AO, class BO>
__device__ __forceinline__ void redo_tiles(const AO &ao, const BO &bo, int64_t ra, int64_t rb, int kbeg, int kend,
                                           uint64_t bad, floatx4 (&acc)[TM][TN]) {
#pragma unroll 1
  for (int t = 0; t < TM * TN; ++t) {
    if (!((bad >> t) & 1)) continue;
    const floatx4 c = redo_tile<SWAP>(ao, bo, ra + 16 * (t / TN), rb + 16 * (t % TN), kbeg, kend);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        if (i * TN + j == t) acc[i][j] = c;
  }
}

}  // namespace dlm
