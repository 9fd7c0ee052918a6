// Signal2SH, SH2Signal (Sec. 2.2) and their adjoints on voxel rows, every
// shell of the table in one pass; Signal2SH also from raw acquisitions.
//
//   out[v][out_off_s + n] = sum_k Bt_s[n][k] in[v][in_off_s + k],  s = 0 .. S-1
//
// The transforms are streams (15 flop per byte): what bounds them is how
// evenly whole cache lines move.  A row is n_in floats of all shells, so 32
// rows are one contiguous run of memory on either side.  A block copies that
// run into LDS as it is (DMA, 16 bytes a lane), its eight waves take the
// (shell, 16 columns) units of the tile in turn with both groups of 16 rows,
// keep the results in registers, write them to the same LDS once the inputs
// have been read, and the block stores them as one contiguous run.  35 KB for
// three shells of 90 directions leaves four blocks on a compute unit to cover
// each other's latency (four waves a block measured 5-15% slower: two or three
// units one after another are then the longest part of a block's life); a
// unit's table fragments come from L2.
// Short rows are taken in several groups of 32, so that a block moves about as
// much (30 volumes, order 2, 200 000 voxels, one group 15.3 us, six 10.5);
// rows of a multiple of eight floats are padded by four in LDS (three shells
// of 96, order 12, BF16, 200 000 voxels: Signal2SH 304 us with 16 rows of a
// column in one bank, 95 padded).
// 450 000 voxels, three shells of 90: BF16 order 12 267 -> 200 us (4.9 TB/s)
// either way, FP32 SH2Signal 256 -> 220 us, FP32 Signal2SH from raw volumes
// 377 + 130 (the means in a pass of their own) -> 280 us; 100 003 voxels of 30
// + 60 directions, FP32 order 6, 28 -> 18.5 us, against one wave per 16 voxels
// and shell that reads its rows and writes its results straight from
// registers, partial lines at every shell's edge, a launch per unequal shell.
//
// Fragments and the order of the sums are those of the other SH kernels: BF16
// v_mfma_f32_16x16x32_bf16, lane (q16, g4) with k = 32 s + 8 g4 .. + 7; FP32
// v_mfma_f32_16x16x4_f32, k = 16 h + 4 g4 + e for instruction e.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gemm_common.h"
#include "internal.h"

namespace dlm {
namespace rows {

constexpr int kRows = 32;   // voxels per block
constexpr int kWaves = 8;   // waves per block
constexpr int kThreads = 64 * kWaves;
constexpr int kUnits = 3;   // units per wave, at most
constexpr int kMaxLds = 64 * 1024;
constexpr int kGroupLds = 36 * 1024;
constexpr int kSlots = 1024;  // blocks on the chip at a time, four per compute unit
constexpr int kMaxRow = 512;  // entries of a row, at most (64 KB a tile)

// Copies between nv rows of n floats in global memory, one contiguous run, and
// LDS rows of `stride` floats.  stride == n moves the run as it is; else n is a
// multiple of 8 and the LDS rows have four floats more.  ALIGNED: the global
// side is 16-byte aligned.
template <bool ALIGNED>
__device__ __forceinline__ void copy_in(float *lds, const float *src, int nv, int n, int stride, unsigned magic) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n4 = nv * stride >> 2, cs = stride >> 2, last = (n >> 2) - 1;
  const bool pad = stride != n;
  for (int i0 = wave * 64; i0 < n4; i0 += kThreads) {
    const int i = i0 + lane;
    int64_t from = 4 * (int64_t)i;
    if (pad) {  // the LDS slot's row and 16-byte piece; the filler takes the last piece again
      const int r = (int)__umulhi((unsigned)i, magic), c = i - r * cs;
      from = (int64_t)r * n + 4 * (c < last ? c : last);
    }
    if (i < n4) {
      if constexpr (ALIGNED)
        dma_to_lds<16>(src + from, lds + 4 * i0);
      else
        *reinterpret_cast<floatx4 *>(lds + 4 * i) = ld4(src + from);
    }
  }
  const int rest = nv * stride & 3;
  if ((int)threadIdx.x < rest) lds[4 * n4 + threadIdx.x] = src[4 * n4 + threadIdx.x];
}

__device__ __forceinline__ void copy_out(float *dst, const float *lds, int nv, int n, int stride, unsigned magic) {
  const int n4 = nv * n >> 2, cs = n >> 2;
  const bool pad = stride != n;
  for (int i = threadIdx.x; i < n4; i += kThreads) {
    int at = 4 * i;
    if (pad) {
      const int r = (int)__umulhi((unsigned)i, magic);
      at = r * stride + 4 * (i - r * cs);
    }
    const floatx4 v = *reinterpret_cast<const floatx4 *>(lds + at);
    __builtin_memcpy(dst + 4 * (int64_t)i, &v, 16);
  }
  const int rest = nv * n & 3;
  if ((int)threadIdx.x < rest) dst[4 * n4 + threadIdx.x] = lds[4 * n4 + threadIdx.x];
}

// Four entries of an LDS row from k (a multiple of 4 beyond the row's shell
// start, so at any dword), zeros at and beyond nred.
__device__ __forceinline__ floatx4 run4(const float *row, int k, int nred) {
  floatx4 v;
  __builtin_memcpy(&v, row + k, 16);
  if (k + 3 >= nred)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = k + e < nred ? v[e] : 0.0f;
  return v;
}

// HM: 16-k groups of the longest shell (an even number in BF16).  RAW: rows of
// x.raw_n volumes in acquisition order, divided by the mean of their b = 0
// volumes on the way (in LDS, as one pass from the raw tile to the row tile).
template <bool F32, bool RAW, bool ALIGNED, int HM>
__global__ __launch_bounds__(kThreads) void sh_rows_kernel(ShellRows x) {
  extern __shared__ __attribute__((aligned(16))) float tile[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q16 = lane & 15, g4 = lane >> 4;
  const int rows = RAW ? kRows : kRows * x.groups;
  const int64_t v0 = (int64_t)blockIdx.x * rows;
  const int nv = x.V - v0 < rows ? (int)(x.V - v0) : rows;
  const int units = RAW ? x.units : x.units * x.groups;
  // BF16: the wave's first fragments are loaded along with the rows (FP32 has
  // no registers for them: 66 and one block fewer per compute unit)
  constexpr bool kAhead = !F32 && !RAW;
  bf16x8 ahead[kAhead ? HM / 2 : 1];
  float *in = tile;
  if constexpr (RAW) {
    float *raw = tile, *inv = tile + x.lds_rows;
    copy_in<ALIGNED>(raw, x.in + v0 * x.raw_n, nv, x.raw_n, x.raw_n, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid < nv) {
      float s = 0.0f;
#pragma unroll 6
      for (int i = 0; i < x.n_b0; ++i) s += raw[tid * x.raw_n + x.b0[i]];
      inv[tid] = (float)x.n_b0 / s;
    }
    __syncthreads();
    // half the block takes the even rows, half the odd ones; a thread entries
    // k, k + kThreads / 2, .. of each, through registers: the row tile takes
    // the raw tile's place
    constexpr int kHalf = kThreads / 2, kCols = kMaxRow / kHalf;
    const int k0 = tid & (kHalf - 1), odd = tid / kHalf;
    float val[kCols][kRows / 2];
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
      const int k = k0 + c * kHalf;
      if (k >= x.n_in) break;
      const int d = x.dw[k];
#pragma unroll
      for (int r = 0; r < kRows / 2; ++r) val[c][r] = raw[(2 * r + odd) * x.raw_n + d] * inv[2 * r + odd];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
      const int k = k0 + c * kHalf;
      if (k >= x.n_in) break;
#pragma unroll
      for (int r = 0; r < kRows / 2; ++r) in[(2 * r + odd) * x.in_stride + k] = val[c][r];
    }
  } else {
    copy_in<ALIGNED>(in, x.in + v0 * x.n_in, nv, x.n_in, x.in_stride, x.in_magic);
    if constexpr (kAhead)
      if (wave < units) {
        int unit = wave, shell = 0;
        while (unit >= x.units) unit -= x.units;
        while (shell + 1 < x.S && unit >= x.sh[shell + 1].unit0) ++shell;
        const ShellRows::Shell s = x.sh[shell];
        const int S = (s.nred + 31) / 32;
        const bf16x8 *fr = reinterpret_cast<const bf16x8 *>(x.frag_h + s.frag_h) + (int64_t)(unit - s.unit0) * S * 64 + lane;
#pragma unroll
        for (int t = 0; t < HM / 2; ++t)
          if (t < S) ahead[t] = fr[t * 64];
      }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __syncthreads();

  floatx4 acc[kUnits][2];
#pragma unroll
  for (int u = 0; u < kUnits; ++u) {
    int unit = wave + kWaves * u, row = q16;
    if (unit < units) {
      for (; unit >= x.units; unit -= x.units) row += kRows;
      int shell = 0;
      while (shell + 1 < x.S && unit >= x.sh[shell + 1].unit0) ++shell;
      const ShellRows::Shell s = x.sh[shell];
      const int j = unit - s.unit0;
      const float *r0 = in + row * x.in_stride, *r1 = r0 + 16 * x.in_stride;
      acc[u][0] = acc[u][1] = floatx4{0.f, 0.f, 0.f, 0.f};
      if constexpr (F32) {
        const int H = (s.nred + 15) / 16;
        const floatx4 *fr = reinterpret_cast<const floatx4 *>(x.frag_f + s.frag_f) + (int64_t)j * H * 64 + lane;
        floatx4 b[HM];
#pragma unroll
        for (int h = 0; h < HM; ++h)
          if (h < H) b[h] = fr[h * 64];
#pragma unroll
        for (int h = 0; h < HM; ++h) {
          if (h >= H) break;
          const int k = 16 * h + 4 * g4;
          const floatx4 a0 = run4(r0 + s.in_off, k, s.nred), a1 = run4(r1 + s.in_off, k, s.nred);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[h][e], a0[e], acc[u][0], 0, 0, 0);
            acc[u][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[h][e], a1[e], acc[u][1], 0, 0, 0);
          }
        }
      } else {
        constexpr int SM = HM / 2;
        const int S = (s.nred + 31) / 32;
        const bf16x8 *fr = reinterpret_cast<const bf16x8 *>(x.frag_h + s.frag_h) + (int64_t)j * S * 64 + lane;
        bf16x8 b[SM];
#pragma unroll
        for (int t = 0; t < SM; ++t) {
          if constexpr (kAhead)
            if (u == 0) {
              b[t] = ahead[t];
              continue;
            }
          if (t < S) b[t] = fr[t * 64];
        }
#pragma unroll
        for (int t = 0; t < SM; ++t) {
          if (t >= S) break;
          const int k = 32 * t + 8 * g4;
          bf16x8 a[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const float *r = (i ? r1 : r0) + s.in_off;
            const floatx4 lo = run4(r, k, s.nred), hi = run4(r, k + 4, s.nred);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              a[i][e] = (__bf16)lo[e];
              a[i][4 + e] = (__bf16)hi[e];
            }
          }
#pragma unroll
          for (int i = 0; i < 2; ++i) acc[u][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[t], a[i], acc[u][i], 0, 0, 0);
        }
      }
    }
  }
  __syncthreads();  // the inputs have been read: the tile takes the results
#pragma unroll
  for (int u = 0; u < kUnits; ++u) {
    int unit = wave + kWaves * u, row = q16;
    if (unit < units) {
      for (; unit >= x.units; unit -= x.units) row += kRows;
      int shell = 0;
      while (shell + 1 < x.S && unit >= x.sh[shell + 1].unit0) ++shell;
      const ShellRows::Shell s = x.sh[shell];
      const int n = 16 * (unit - s.unit0) + 4 * g4;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float *o = tile + (row + 16 * i) * x.out_stride + s.out_off + n;
        if (n + 3 < s.ncol) {
          __builtin_memcpy(o, &acc[u][i], 16);
        } else {
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (n + e < s.ncol) o[e] = acc[u][i][e];
        }
      }
    }
  }
  __syncthreads();
  copy_out(x.out + v0 * x.n_out, tile, nv, x.n_out, x.out_stride, x.out_magic);
}

template <bool F32, bool RAW, bool ALIGNED, int HM>
int run(const ShellRows &x, size_t lds, hipStream_t st) {
  const int rows = kRows * x.groups;
  const int64_t blocks = (x.V + rows - 1) / rows;
  if (blocks > 0x7fffffff) return -4;
  hipLaunchKernelGGL((sh_rows_kernel<F32, RAW, ALIGNED, HM>), dim3((unsigned)blocks), dim3(kThreads), lds, st, x);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <bool F32, bool RAW, bool ALIGNED>
int run_h(const ShellRows &x, size_t lds, hipStream_t st) {
  if (x.max_red <= 32) return run<F32, RAW, ALIGNED, 2>(x, lds, st);
  if (x.max_red <= 64) return run<F32, RAW, ALIGNED, 4>(x, lds, st);
  if (x.max_red <= 96) return run<F32, RAW, ALIGNED, 6>(x, lds, st);
  return run<F32, RAW, ALIGNED, 8>(x, lds, st);
}

// LDS rows whose length is a multiple of eight floats are four floats longer:
// sixteen rows read at one column then lie in all banks and not in two to
// eight of them.
int stride(int n) { return n % 8 == 0 ? n + 4 : n; }
// i / d as the high word of i * magic, for i < 2^16 and 2 <= d < 2^8 (a tile
// is at most 4096 pieces of 16 bytes)
unsigned magic(int d) { return d < 2 ? 0u : unsigned(((uint64_t(1) << 32) + d - 1) / d); }

// Floats of LDS: the tile (raw rows, inputs, then results; its last run may be
// read up to 31 entries beyond the last row) and behind it, for RAW, the
// voxels' inverse means.
size_t row_floats(const ShellRows &x) {
  return (size_t(kRows) * x.groups * std::max(std::max(stride(x.n_in), stride(x.n_out)), x.raw_n) + 128 + 3) / 4 * 4;
}
size_t lds_floats(const ShellRows &x) { return row_floats(x) + (x.raw_n ? kRows : 0); }

// Groups of 32 rows per block, up to what the waves take units of and a quarter
// of a compute unit's LDS holds: the number whose rounds of blocks over the
// chip move the least, counting a block's fixed part as 10 KB (30 volumes,
// order 2, 200 000 voxels: 7 rounds of 3.8 KB 15.3 us, 2 rounds of 23 KB 10.5;
// 30 + 60 volumes, order 6, 100 003 voxels, both transforms and adjoints: 2
// rounds of 34 KB 92 us, 2 of 23 KB 81).
int groups(const ShellRows &x) {
  if (x.raw_n) return 1;
  const int64_t bytes = int64_t(4) * kRows * std::max(stride(x.n_in), stride(x.n_out));
  const int most = int(std::min<int64_t>(kWaves * kUnits / std::max(x.units, 1), kGroupLds / bytes));
  int best = 1;
  int64_t least = 0;
  for (int g = 1; g <= std::max(most, 1); ++g) {
    const int64_t rounds = ((x.V + kRows * g - 1) / (kRows * g) + kSlots - 1) / kSlots, cost = rounds * (g * bytes + 10240);
    if (g == 1 || cost < least) {
      best = g;
      least = cost;
    }
  }
  return best;
}

}  // namespace rows

// Tables with more units than the waves hold, and tiles that leave a compute
// unit fewer than two blocks, stay on the per-shell kernels.
bool shell_rows_ok(const ShellRows &x) {
  return x.S >= 1 && x.S <= kMaxRowShells && x.units <= rows::kWaves * rows::kUnits && x.max_red <= 128 && x.n_in <= rows::kMaxRow &&
         rows::lds_floats(x) * 4 <= size_t(rows::kMaxLds);
}

// Where whole rows are the faster way.  Unequal shells: always (1.1 to 2.5
// times; the per-shell kernels take a launch per shell).  Equal shells are one
// launch there as well, of waves that need no barrier, and what decides is
// whether their slices are whole 16-byte pieces on either side.  With neither,
// rows win (three shells of 90, 200 000 voxels, order 8: BF16 Signal2SH 86 ->
// 61 us, FP32 SH2Signal 115 -> 93; one shell only in BF16, 1.05 to 1.3 times
// against 0.85 to 1.1 in FP32); with one or both only over many shells and
// voxels (three shells of 96, order 12, BF16: 200 000 voxels 118 -> 95 us, 30 000
// voxels 20.3 against 21.9; not for FP32 products that read such slices, order
// 10 121 against 133; two shells of 45, order 6, 200 000 voxels, FP32
// SH2Signal 28 against 33).  FP32 products of long reductions in more than two
// units a wave outlast the copies and need later blocks to hide behind them
// (three shells of 90, order 12, 30 000 voxels: 29.0 against 30.6 us; 200 000
// voxels 191 -> 153).
// Rows save reading lines twice that two shells share, which costs little
// while a call's data stays in the last-level cache (half of its 256 MB: a step
// has another call's data beside it; at 130 MB rows still take 1.03 to 1.1 times
// as long in the cases below, at 144 MB 0.82 to 1.01).  There the per-shell waves win wherever every wave of a row
// block has products to do and either the rows start on 16 bytes, so that
// shells' slices are read in whole pieces all the same (two shells of 90, order
// 10, 80 000 voxels, 100 MB, BF16 SH2Signal 25 against 31 us, 300 000 voxels 97
// -> 95; four of 45, order 8, 20 000 voxels 9.7 against 11.8), or the FP32
// reduction is long (three shells of 90, order 8, 40 000 voxels Signal2SH 22.4
// against 25.2 us; two of 90, order 12, 25.2 against 28.4), or FP32 reads short
// slices and writes whole pieces (three shells of 60, order 2, 70 000 voxels
// 17.2 against 18.5).
bool shell_rows_pay(const ShellRows &x, dlm_precision prec) {
  constexpr int64_t kMany = 65536, kCached = 128 << 20;
  const bool f32 = prec != DLM_BF16;
  for (int s = 1; s < x.S; ++s)
    if (x.sh[s].nred != x.sh[0].nred || x.sh[s].ncol != x.sh[0].ncol) return true;
  const int nred = x.sh[0].nred, ncol = x.sh[0].ncol;
  const int64_t bytes = int64_t(4) * x.V * (x.n_in + x.n_out);
  const bool busy = x.units >= rows::kWaves && bytes < kCached;
  if (busy && x.n_in % 4 == 0 && x.n_out % 4 == 0 && bytes >= kCached / 16) return false;
  if (nred % 4 == 0 || ncol % 4 == 0)
    return x.S > 2 && x.V >= kMany && !(f32 && (nred % 4 == 0 || (nred <= 64 && bytes < kCached)));
  if (f32 && x.V < kMany && x.units > 2 * rows::kWaves && x.max_red > 64) return false;
  if (f32 && busy && nred > 64 && bytes >= kCached / 4) return false;
  return x.S > 1 || !f32;
}

int launch_shell_rows(ShellRows x, dlm_precision prec, void *stream) {
  if (!shell_rows_ok(x)) return -3;
  if (x.V <= 0) return 0;
  x.groups = rows::groups(x);
  x.in_stride = rows::stride(x.n_in);
  x.out_stride = rows::stride(x.n_out);
  x.in_magic = rows::magic(x.in_stride / 4);
  x.out_magic = rows::magic(x.n_out / 4);
  x.lds_rows = (int)rows::row_floats(x);
  const size_t lds = rows::lds_floats(x) * 4;
  hipStream_t st = (hipStream_t)stream;
  const bool al = (reinterpret_cast<uintptr_t>(x.in) & 15) == 0, f32 = prec != DLM_BF16;
  using namespace rows;
  if (x.raw_n) {
    if (f32) return al ? run_h<true, true, true>(x, lds, st) : run_h<true, true, false>(x, lds, st);
    return al ? run_h<false, true, true>(x, lds, st) : run_h<false, true, false>(x, lds, st);
  }
  if (f32) return al ? run_h<true, false, true>(x, lds, st) : run_h<true, false, false>(x, lds, st);
  return al ? run_h<false, false, true>(x, lds, st) : run_h<false, false, false>(x, lds, st);
}

}  // namespace dlm
