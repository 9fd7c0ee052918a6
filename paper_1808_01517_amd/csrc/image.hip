// Signal2SH, SH2Signal (Sec. 2.2) and their adjoints on images
// [subjects][channels][voxels], read and written as they are:
//
//   out[b][g c_gs + n][v] = sum_k Bt_g[n][k] in[b][g a_gs + k][v]
//
// The transforms are streams (15 flop per byte), so what counts is that every
// access is wide and that nothing stands between the loads and the matrix
// cores.  A wave takes 64 voxels of one shell: for a channel, 16 lanes load
// four consecutive voxels each (256 contiguous bytes), and the four lane
// groups load four different channels, which is the operand order of the
// matrix instructions if lane q's four values go to four of them: instruction
// t works on voxels 4 q + t.  All loads are issued before the first
// instruction; no LDS, no transposes, no barriers.  The outputs come out with
// the four voxels of a lane side by side again (one 16-byte store per
// channel).  The tables are those of the per-shell kernel (fragment order).
// Sums run in the same order as there, so BF16 results are the same bits.
#include <hip/hip_runtime.h>

#include "gemm_common.h"
#include "internal.h"

namespace dlm {
namespace image {

// HM: groups of 16 input channels held (the reduction's length / 16, rounded
// up; an even number in BF16).
template <bool F32, int HM>
__global__ __launch_bounds__(256) void sh_image_kernel(ShellImage x, int chunks, int64_t nwaves) {
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= nwaves) return;  // whole waves only; no barriers in this kernel
  const int lane = threadIdx.x & 63, q16 = lane & 15, g4 = lane >> 4;
  const int64_t zb = w / chunks;  // (image, shell); neighbouring waves take neighbouring voxels
  const int64_t v = (w - zb * chunks) * 64 + 4 * q16;
  const int b = (int)(zb / x.groups), g = (int)(zb - (int64_t)b * x.groups);
  const float *in = x.in + ((int64_t)b * x.in_ch + (int64_t)g * x.a_gs) * x.P;
  float *out = x.out + ((int64_t)b * x.out_ch + (int64_t)g * x.c_gs) * x.P;
  const int H = F32 ? (x.nred + 15) / 16 : (x.nred + 31) / 32 * 2;
  const int cnt = v + 4 <= x.P ? 4 : v < x.P ? (int)(x.P - v) : 0;
  // a[h][e]: FP32 channel 16 h + 4 g4 + e; BF16 channel 32 (h / 2) + 8 g4 + 4 (h % 2) + e
  floatx4 a[HM][4];
#pragma unroll
  for (int h = 0; h < HM; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = F32 ? 16 * h + 4 * g4 + e : 32 * (h / 2) + 8 * g4 + 4 * (h % 2) + e;
      a[h][e] = floatx4{0.f, 0.f, 0.f, 0.f};
      if (h < H && k < x.nred) {
        const float *src = in + (int64_t)k * x.P + v;
        if (cnt == 4) {
          a[h][e] = ld4(src);
        } else {
#pragma unroll
          for (int t = 0; t < 3; ++t)
            if (t < cnt) a[h][e][t] = src[t];
        }
      }
    }
  const int NT = (x.ncol + 15) / 16;
  auto store = [&](int j, const floatx4 (&c)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = 16 * j + 4 * g4 + e;
      if (n >= x.ncol) continue;
      const floatx4 r{c[0][e], c[1][e], c[2][e], c[3][e]};
      float *o = out + (int64_t)n * x.P + v;
      if (cnt == 4) {
        __builtin_memcpy(o, &r, 16);
      } else {
#pragma unroll
        for (int t = 0; t < 3; ++t)
          if (t < cnt) o[t] = r[t];
      }
    }
  };
  if constexpr (F32) {
    const floatx4 *fr = reinterpret_cast<const floatx4 *>(x.frag_f) + (int64_t)g * x.frag_gs_f / 16;
    for (int j = 0; j < NT; ++j) {
      floatx4 acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < HM; ++h) {
        if (h >= H) break;
        const floatx4 bt = fr[((int64_t)j * H + h) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(bt[e], a[h][e][t], acc[t], 0, 0, 0);
      }
      store(j, acc);
    }
  } else {
    constexpr int SM = HM / 2;
    const int S = H / 2;
    const bf16x8 *fr = reinterpret_cast<const bf16x8 *>(x.frag_h) + (int64_t)g * x.frag_gs_h / 16;
    bf16x8 ah[SM][4];
#pragma unroll
    for (int s = 0; s < SM; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ah[s][t][e] = (__bf16)a[2 * s][e][t];
          ah[s][t][4 + e] = (__bf16)a[2 * s + 1][e][t];
        }
    for (int j = 0; j < NT; ++j) {
      floatx4 acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < SM; ++s) {
        if (s >= S) break;
        const bf16x8 bt = fr[((int64_t)j * S + s) * 64 + lane];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bt, ah[s][t], acc[t], 0, 0, 0);
      }
      store(j, acc);
    }
  }
}

template <bool F32, int HM>
int run(const ShellImage &x, hipStream_t st) {
  const int64_t chunks = (x.P + 63) / 64, nwaves = chunks * x.groups * x.B, blocks = (nwaves + 3) / 4;
  if (chunks > 0x7fffffff || blocks > 0x7fffffff) return -4;
  hipLaunchKernelGGL((sh_image_kernel<F32, HM>), dim3((unsigned)blocks), dim3(256), 0, st, x, (int)chunks, nwaves);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace image

int launch_shell_image(const ShellImage &x, dlm_precision prec, void *stream) {
  if (x.nred <= 0 || x.nred > 128 || x.ncol <= 0 || x.P <= 0 || x.B <= 0) return -3;
  hipStream_t st = (hipStream_t)stream;
  // registers for the input are sized by the reduction
  if (prec == DLM_BF16) {
    if (x.nred <= 32) return image::run<false, 2>(x, st);
    if (x.nred <= 64) return image::run<false, 4>(x, st);
    return x.nred <= 96 ? image::run<false, 6>(x, st) : image::run<false, 8>(x, st);
  }
  if (x.nred <= 32) return image::run<true, 2>(x, st);
  if (x.nred <= 48) return image::run<true, 3>(x, st);
  return x.nred <= 96 ? image::run<true, 6>(x, st) : image::run<true, 8>(x, st);
}

}  // namespace dlm
