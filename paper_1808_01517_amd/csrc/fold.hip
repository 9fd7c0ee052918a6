// Kernel-tensor side of the folded LSC layer (Sec. 2.3: resampling, cyclic
// kernel dot and refit composed into one matrix per layer).
//
//   fold:    T[(o,k)][(c,j)] = sum_t W[o][c][t] Q[t][k][j]      (or T^T)
//   unfold:  dW[o][c][t]     = sum_{k,j} dT[(o,k)][(c,j)] Q[t][k][j]
//            db[o]           = sum_k dT[(o,k)][C K_in] (P_m 1)[k]
//
// Both are thin (17 taps) contractions against the small table Q (138 KB at
// order 8, L2-resident); what they cannot do without is one pass over the
// O K_out x C K_in matrix, so they are laid out for that pass.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "gemm_common.h"
#include "internal.h"

namespace dlm {
namespace fold {

constexpr int kPairs = 8;  // (o, c) pairs per block of the fold
constexpr int kTaps = 32;  // taps held in registers at a time

// Store entry (row, col) of the folded matrix; of three parts also the value
// itself, in rows of ldc: parts hold neither infinities, nor what rounds to
// one, nor all bits of what is below 2^-109, and results that such entries
// may have reached are computed again from it.
template <int KIND>
__device__ __forceinline__ void put(void *out, int64_t ld, int64_t row, int64_t col, float v, float *copy = nullptr,
                                    int64_t ldc = 0) {
  if constexpr (KIND == kFoldParts) {
    if (copy) copy[row * ldc + col] = v;
    uint16_t *o = static_cast<uint16_t *>(out) + row * 3 * ld + col;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const __bf16 h = (__bf16)v;  // the part: what is left so far, rounded (RNE)
      o[i * ld] = __builtin_bit_cast(uint16_t, h);
      v -= (float)h;
    }
  } else if constexpr (KIND == kFoldBf16) {
    static_cast<uint16_t *>(out)[row * ld + col] = to_bf16_bits(v);
  } else {
    static_cast<float *>(out)[row * ld + col] = v;
  }
}

// A thread owns one (k, j) entry of Q for all taps, in registers, and runs
// through kPairs (o, c) pairs, whose taps the block keeps in LDS (one address
// per wave: broadcasts); consecutive threads write consecutive columns.  TR
// writes T^T from the transposed table (Q is then [t][j][k]), so its columns
// are consecutive too.  Row padding (columns ncol .. ld - 1, zeros) and the folded
// bias are written by the blocks of the last grid column of the same launch.
// Inside a group of 16 the taps are added in the order 0 4 8 12, 1 5 9 13, ..
// (that of four 16x16x4 matrix instructions whose lane group g holds taps 4 g
// .. 4 g + 3), so the rounding of the table is the same whichever kernel
// makes it.  It is bound by the stores' address and issue work.  64 -> 64
// channels in BF16 45.8 -> 19.5 us, 32 -> 64 in FP32 25.9 -> 12.7 us, 3 -> 32
// 9.6 -> 5 us (the values beside the parts add 2.5 us to the second and 0.4 to
// the third) against a matrix-core GEMM with a 17-deep reduction and
// element-wise scattered stores, which also needed a launch each for the
// padding and the bias (2-5 us).
template <bool TR, int KIND>
__global__ __launch_bounds__(256) void fold_kernel(const float *W, const float *Q, int C, int O, int T, int Ki, int Ko,
                                                   void *out, int64_t ld, float *copy, const float *bias,
                                                   const float *pm1, float *bvec, int nbE) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x == nbE) {
    const int64_t id = (int64_t)blockIdx.y * 256 + tid, nth = (int64_t)gridDim.y * 256;
    const int64_t rows = TR ? (int64_t)C * Ki : (int64_t)O * Ko, ncol = TR ? (int64_t)O * Ko : (int64_t)C * Ki;
    const int64_t pad = ld - ncol;
    for (int64_t i = id; i < rows * pad; i += nth) {
      const int64_t r = i / pad;
      put<KIND>(out, ld, r, ncol + (i - r * pad), 0.0f);
    }
    if (bvec)
      for (int64_t i = id; i < (int64_t)O * Ko; i += nth) {
        const int o = (int)(i / Ko), k = (int)i - o * Ko;
        bvec[i] = bias ? bias[o] * pm1[k] : 0.0f;
      }
    return;
  }
  __shared__ __attribute__((aligned(16))) float taps[kPairs][kTaps];
  static_assert(kPairs * kTaps == 256, "one tap per thread");
  const int KK = Ko * Ki, e = blockIdx.x * 256 + tid;
  const int nq = TR ? Ko : Ki, np = TR ? Ki : Ko;  // columns, rows of one pair's block
  const int p = e / nq, q = e - p * nq;
  const int Y = TR ? O : C, pairs = C * O;
  const int p0 = blockIdx.y * kPairs;
  float acc[kPairs];
#pragma unroll
  for (int i = 0; i < kPairs; ++i) acc[i] = 0.0f;
  for (int t0 = 0; t0 < T; t0 += kTaps) {
    // the pairs' taps t0 .. t0 + kTaps - 1 in the order of the sum (four to a
    // 16-byte read), zeros beyond T
    __syncthreads();
    {
      const int i = tid / kTaps, t = tid - i * kTaps;
      const int x = (p0 + i) / Y, y = (p0 + i) - x * Y;
      const int u = (t & 16) + 4 * (t & 3) + ((t >> 2) & 3);
      taps[i][u] = p0 + i < pairs && t0 + t < T ? W[((int64_t)(TR ? y : x) * C + (TR ? x : y)) * T + t0 + t] : 0.0f;
    }
    float qv[kTaps];
#pragma unroll
    for (int t = 0; t < kTaps; ++t) qv[t] = e < KK && t0 + t < T ? Q[(int64_t)(t0 + t) * KK + e] : 0.0f;
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kTaps; h += 16)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (t0 + h + j >= T) break;
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
          const floatx4 w = *reinterpret_cast<const floatx4 *>(&taps[i][h + 4 * j]);
#pragma unroll
          for (int g = 0; g < 4; ++g) acc[i] = fmaf(w[g], qv[h + 4 * g + j], acc[i]);
        }
      }
  }
  if (e >= KK) return;
  int x = p0 / Y, y = p0 - x * Y;
#pragma unroll
  for (int i = 0; i < kPairs; ++i) {
    if (p0 + i >= pairs) break;
    put<KIND>(out, ld, (int64_t)x * np + p, (int64_t)y * nq + q, acc[i], copy, (int64_t)Y * nq);
    if (++y == Y) {
      y = 0;
      ++x;
    }
  }
}

// Sum over the wave, in every lane, without LDS: within rows of 16 lanes by
// data-parallel primitives, between rows by the lane swaps.
__device__ __forceinline__ float wave_sum(float x) {
  auto dpp = [](float v, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf,
                                                                 0xf, false));
  };
  x += dpp(x, std::integral_constant<int, 0xb1>{});   // quad_perm 1 0 3 2
  x += dpp(x, std::integral_constant<int, 0x4e>{});   // quad_perm 2 3 0 1
  x += dpp(x, std::integral_constant<int, 0x141>{});  // row_half_mirror
  x += dpp(x, std::integral_constant<int, 0x140>{});  // row_mirror
  const Both s16 = swap16(__builtin_bit_cast(unsigned, x));
  x = __builtin_bit_cast(float, s16.a) + __builtin_bit_cast(float, s16.b);
  const Both s32 = swap32(__builtin_bit_cast(unsigned, x));
  return __builtin_bit_cast(float, s32.a) + __builtin_bit_cast(float, s32.b);
}

// dW of PC channels c of one output channel per block: the block reads their
// K_out x K_in gradients once (adding up the SP partial matrices as it reads),
// keeps them in registers and runs through its taps of Q, TB at a time, which
// the PC pairs share.  Few pairs (PC = 1) also split the taps over blocks.
// It is bound by the latency of its loads and of the wave sums.  64 -> 64
// channels 135 + 15 + 7 us (a wave per (o, c, t), the partial sums and the
// bias gradient in kernels of their own) -> 33 us in one launch, 32 -> 64
// with two partials 72.6 + 11 + 15 -> 26 us, 3 -> 32 15.5 + 15.2 -> 5.4 us.
constexpr int kChunk = 2048;  // gradient entries held by a block at a time
constexpr int kTapBlock = 4;  // taps per step

template <int PC, int SP>
__global__ __launch_bounds__(256) void unfold_kernel(const float *part, int64_t mstride, const float *Q,
                                                     const float *pm1, int C, int O, int T, int Ki, int Ko, int N1,
                                                     float *dW, float *db, int nb) {
  constexpr int PER = kChunk / 256, TB = kTapBlock;
  __shared__ float red[4][PC * TB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x >= nb) {  // the bias gradient, one wave per output channel
    const int o = ((int)blockIdx.x - nb) * 4 + wave;
    if (o >= O || blockIdx.y != 0) return;
    float s = 0.0f;
    for (int k = lane; k < Ko; k += 64) {
      const float *g = part + ((int64_t)o * Ko + k) * N1 + (N1 - 1);
      float v = 0.0f;
#pragma unroll
      for (int p = 0; p < SP; ++p) v += g[p * mstride];
      s += v * pm1[k];
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) db[o] = s;
    return;
  }
  const int cb = (C + PC - 1) / PC, KK = Ko * Ki;
  const int o = blockIdx.x / cb, c0 = (blockIdx.x - o * cb) * PC;
  float g[PC][PER];
  auto load = [&](int base) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = base + i * 256 + tid;
      const int kk = e / Ki, j = e - kk * Ki;
      const float *src = part + ((int64_t)o * Ko + kk) * N1 + (int64_t)c0 * Ki + j;
#pragma unroll
      for (int c = 0; c < PC; ++c) {
        g[c][i] = 0.0f;
        if (e < KK && c0 + c < C) {
#pragma unroll
          for (int p = 0; p < SP; ++p) g[c][i] += src[p * mstride + c * Ki];
        }
      }
    }
  };
  const bool one = KK <= kChunk;
  if (one) load(0);
  for (int t0 = blockIdx.y * TB; t0 < T; t0 += gridDim.y * TB) {
    float s[PC][TB];
#pragma unroll
    for (int c = 0; c < PC; ++c)
#pragma unroll
      for (int u = 0; u < TB; ++u) s[c][u] = 0.0f;
    for (int base = 0; base < KK; base += kChunk) {
      if (!one) load(base);
      float q[TB][PER];
#pragma unroll
      for (int u = 0; u < TB; ++u)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          const int e = base + i * 256 + tid;
          q[u][i] = e < KK && t0 + u < T ? Q[(int64_t)(t0 + u) * KK + e] : 0.0f;
        }
#pragma unroll
      for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int c = 0; c < PC; ++c)
#pragma unroll
          for (int u = 0; u < TB; ++u) s[c][u] = fmaf(g[c][i], q[u][i], s[c][u]);
    }
#pragma unroll
    for (int c = 0; c < PC; ++c)
#pragma unroll
      for (int u = 0; u < TB; ++u) s[c][u] = wave_sum(s[c][u]);
    if (lane == 0)
#pragma unroll
      for (int c = 0; c < PC; ++c)
#pragma unroll
        for (int u = 0; u < TB; ++u) red[wave][c * TB + u] = s[c][u];
    __syncthreads();
    if (tid < PC * TB) {
      const int c = tid / TB, u = tid - c * TB;
      if (c0 + c < C && t0 + u < T)
        dW[((int64_t)o * C + c0 + c) * T + t0 + u] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
    }
    __syncthreads();
  }
}

// out[i] = sum_p part[p * n + i], in the order of p; eight loads in flight
// per thread (one at a time took 55 us for 128 partials of 135 x 1441).  The sum
// is in 64 bits, which the loads hide: in 32 bits its roundings were a tenth of
// a small layer's gradient error.
__global__ __launch_bounds__(256) void sum_partials_kernel(const float *part, int splits, int64_t n, float *out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  int p = 0;
  for (; p + 8 <= splits; p += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(p + u) * n + i];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; p < splits; ++p) s += part[(int64_t)p * n + i];
  out[i] = (float)s;
}

// Tables are transposed once, when a plan is made: one entry per thread.
template <class T>
__global__ __launch_bounds__(256) void transpose_kernel(const T *src, T *dst, int64_t n, int rows, int cols) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t slice = (int64_t)rows * cols, b = i / slice, e = i - b * slice, c = e / rows, r = e - c * rows;
  dst[i] = src[b * slice + r * cols + c];
}

}  // namespace fold

int launch_transpose(const void *src, void *dst, int batch, int rows, int cols, int size, void *stream) {
  const int64_t n = (int64_t)batch * rows * cols, blocks = (n + 255) / 256;
  if (n <= 0 || blocks > 0x7fffffff) return -4;
  hipStream_t st = (hipStream_t)stream;
  if (size == 4)
    hipLaunchKernelGGL(fold::transpose_kernel<uint32_t>, dim3((unsigned)blocks), dim3(256), 0, st,
                       static_cast<const uint32_t *>(src), static_cast<uint32_t *>(dst), n, rows, cols);
  else
    hipLaunchKernelGGL(fold::transpose_kernel<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, st,
                       static_cast<const uint16_t *>(src), static_cast<uint16_t *>(dst), n, rows, cols);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_lsc_fold(const FoldOut &f, void *stream) {
  const int KK = f.Ko * f.Ki, pairs = f.C * f.O;
  const int nbE = (KK + 255) / 256;
  const dim3 grid(nbE + 1, (pairs + fold::kPairs - 1) / fold::kPairs);
  hipStream_t st = (hipStream_t)stream;
#define DLM_FOLD(TR, BF)                                                                                          \
  hipLaunchKernelGGL((fold::fold_kernel<TR, BF>), grid, dim3(256), 0, st, f.W, f.Q, f.C, f.O, f.T, f.Ki, f.Ko, f.out, \
                     f.ld, f.copy, f.bias, f.pm1, f.bvec, nbE)
  if (f.transposed) {
    if (f.kind == kFoldBf16) DLM_FOLD(true, kFoldBf16);
    else if (f.kind == kFoldParts) DLM_FOLD(true, kFoldParts);
    else DLM_FOLD(true, kFoldF32);
  } else {
    if (f.kind == kFoldBf16) DLM_FOLD(false, kFoldBf16);
    else if (f.kind == kFoldParts) DLM_FOLD(false, kFoldParts);
    else DLM_FOLD(false, kFoldF32);
  }
#undef DLM_FOLD
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_sum_partials(const float *part, int splits, int64_t n, float *out, void *stream) {
  hipLaunchKernelGGL(fold::sum_partials_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                     part, splits, n, out);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int SP>
static void unfold(const float *part, const float *Q, const float *pm1, int C, int O, int T, int Ki, int Ko, float *dW,
                   float *db, hipStream_t st) {
  const int N1 = C * Ki + 1;
  const int64_t ms = (int64_t)O * Ko * N1;
  const int extra = db ? (O + 3) / 4 : 0, nb4 = O * ((C + 3) / 4);
  // four channels per block once that still gives every compute unit a block
  if (nb4 >= 256)
    hipLaunchKernelGGL((fold::unfold_kernel<4, SP>), dim3(nb4 + extra), dim3(256), 0, st, part, ms, Q, pm1, C, O, T, Ki,
                       Ko, N1, dW, db, nb4);
  else
    hipLaunchKernelGGL((fold::unfold_kernel<1, SP>),
                       dim3(O * C + extra, (T + fold::kTapBlock - 1) / fold::kTapBlock), dim3(256), 0, st, part, ms, Q,
                       pm1, C, O, T, Ki, Ko, N1, dW, db, O * C);
}

int launch_lsc_unfold(const float *part, int splits, const float *Q, const float *pm1, int C, int O, int T, int Ki,
                      int Ko, float *dW, float *db, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  if (splits == 1) unfold<1>(part, Q, pm1, C, O, T, Ki, Ko, dW, db, st);
  else if (splits == 2) unfold<2>(part, Q, pm1, C, O, T, Ki, Ko, dW, db, st);
  else return -3;
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace dlm
