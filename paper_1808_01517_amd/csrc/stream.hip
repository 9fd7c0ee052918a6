// Streaming GEMM core for the large contractions of the folded LSC layer
// (Sec. 2.3: resampling, cyclic-kernel dot and refit composed into one
// matrix per layer) and its adjoints.
//
// These contractions do 15-60 flop per HBM byte, far below the bf16
// matrix-core ridge (~300 flop/B): BF16 is bandwidth-bound.  FP32 runs them in
// six bfloat16 part products (parts.h), which puts it near the ridge: 1.0M
// voxels of the K = 135 forward take 1.2 ms of matrix-core cycles and 1.3 ms
// of HBM.  Both want the operand traffic off the register file and out of the
// way of the matrix cores:
//
// * Operands travel from global memory straight into LDS with
//   global_load_lds_dword / _dwordx4 (no register staging), through a ring of
//   NS stages, so NS-1 slices of 32 k are in flight while one is multiplied.
// * Float32 operands stay float32 in LDS and are rounded to bfloat16 (RNE),
//   or split into parts, when a wave reads its MFMA fragment (each row is read
//   by one wave); bfloat16 tables, the FP32 tables' parts and activations
//   stored in bfloat16 are copied as is.
//   A stage wholly inside the reduction range copies from one wave-uniform
//   base address plus per-lane 32-bit offsets computed once per block, so
//   the loop spends a scalar add and one instruction per copy.  In the one
//   stage where the range ends, lanes at or beyond the end copy zeros from a
//   4 KB zero buffer (spread over lanes, so no single cache line is hot).
//   LDS thus holds the exact operands and fragment reads need no
//   conditionals.  Rows beyond the matrix are clamped to valid rows (their
//   outputs are never stored).
// * Every LDS layout is swizzled so that fragment reads avoid bank
//   conflicts while each DMA instruction still fills 64 consecutive slots
//   (the hardware writes lane i of an instruction to base + i * size).
// * Waits are explicit: s_waitcnt vmcnt(n) for the slice about to be used,
//   then a barrier.  A slot is refilled only after the barrier that follows
//   its last read by every wave.
// * The epilogue's side inputs (bias, ReLU mask) are loaded behind the last
//   DMA, after the second-to-last stage's wait, when they fit in registers;
//   only the last stage's wait then covers them.
//
// MFMA v_mfma_f32_16x16x32_bf16, B fragment first, so each accumulator is the
// transposed 16 x 16 tile (a lane holds four consecutive output columns of one
// row), the same epilogue as the register-staged cores; lane (q16, g4) holds
// k = 8 g4 .. 8 g4 + 7.  The ring's depth goes with the tile: two stages where a
// stage of part products outlasts a load, up to eight where few rows leave the
// chip idle.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "gemm_common.h"
#include "internal.h"
#include "parts.h"

namespace dlm {
namespace streaming {

constexpr int SBK = 32;  // reduction entries per stage (one MFMA deep)

#ifndef DLM_ASTAT
#define DLM_ASTAT 1  // the short-reduction kernel below (0: tiled core only)
#endif

// Source of the DMA lanes that fill padding (zero-initialised, never written).
__device__ __attribute__((aligned(16))) float kZeros[1024];
__device__ __forceinline__ const float *zeros_for(int s) { return kZeros + ((s & 255) << 2); }

// Wait until at most N vector-memory operations of this wave are pending and
// its LDS operations are complete, then join the workgroup barrier.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__device__ __forceinline__ bf16x8 to_bf16x8(floatx4 lo, floatx4 hi) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    r[e] = (__bf16)lo[e];
    r[4 + e] = (__bf16)hi[e];
  }
  return r;
}

// ------------------------------------------------------ streamed operands
// Each operand type gives, for a tile of BR rows and one stage of SBK
// reduction entries: bytes() of LDS, slots() DMA lanes of kUnit bytes,
// base(r0, k0) + lane_off(slot, r0) the global address slot `slot` copies,
// k_of(slot) its reduction index within the stage (for zero padding), and
// frag() the bfloat16 MFMA fragment of 16 rows (row group rg) x 8 k for lane
// (q16, g4): row rg*16 + q16, k = 8*g4 .. 8*g4 + 7.

// k-contiguous float32: element (r, k) at p[r * ld + k], valid for r < rows,
// k < K.  LDS: [BR][32] floats, 4-float chunk c of row r stored at chunk
// c ^ (r & 7).  VEC (16-byte lanes) needs 16-byte aligned rows and K % 4
// == 0, so a chunk lies wholly inside or wholly beyond the range.
template <bool VEC>
struct SKc {
  const float *p;
  int64_t ld, rows;
  static constexpr int kUnit = VEC ? 16 : 4;
  template <int BR>
  static constexpr int bytes() { return BR * SBK * 4; }
  template <int BR>
  static constexpr int slots() { return bytes<BR>() / kUnit; }
  // Stage with every k inside the range: lane s copies from
  // base(r0, k0) + lane_off(s, r0) bytes.
  __device__ const char *base(int64_t r0, int k0) const {
    return reinterpret_cast<const char *>(p + r0 * ld + k0);
  }
  template <int BR>
  __device__ uint32_t lane_off(int s, int64_t r0) const {
    int r, k;
    if constexpr (VEC) {
      r = s >> 3;
      k = ((s & 7) ^ (r & 7)) << 2;
    } else {
      r = s >> 5;
      k = ((((s >> 2) & 7) ^ (r & 7)) << 2) | (s & 3);
    }
    const int64_t gr = r0 + r < rows ? r0 + r : rows - 1;
    return (uint32_t)(((gr - r0) * ld + k) * 4);
  }
  // reduction index (within the stage) of slot s: its first, for 16-byte lanes
  template <int BR>
  __device__ static int k_of(int s) {
    if constexpr (VEC) return ((s & 7) ^ ((s >> 3) & 7)) << 2;
    else return ((((s >> 2) & 7) ^ ((s >> 5) & 7)) << 2) | (s & 3);
  }
  template <int BR>
  __device__ bf16x8 frag(const char *lds, int rg, int q16, int g4) const {
    const int r = rg * 16 + q16;
    const float *row = reinterpret_cast<const float *>(lds) + r * SBK;
    const floatx4 lo = *reinterpret_cast<const floatx4 *>(row + (((2 * g4) ^ (r & 7)) << 2));
    const floatx4 hi = *reinterpret_cast<const floatx4 *>(row + (((2 * g4 + 1) ^ (r & 7)) << 2));
    return to_bf16x8(lo, hi);
  }
  template <int BR>
  __device__ void frag3(const char *lds, int rg, int q16, int g4, bf16x8 (&v)[3]) const {
    const int r = rg * 16 + q16;
    const float *row = reinterpret_cast<const float *>(lds) + r * SBK;
    split3(*reinterpret_cast<const floatx4 *>(row + (((2 * g4) ^ (r & 7)) << 2)),
           *reinterpret_cast<const floatx4 *>(row + (((2 * g4 + 1) ^ (r & 7)) << 2)), v);
  }
  // the slow path's reads (parts.h)
  struct Lane {
    const float *first;  // of rows r .. r + 15, the same in all lanes
    uint32_t off;
  };
  __device__ Lane lane(int64_t r, int q16, int g) const {
    const int64_t r0 = r < rows ? r : rows - 1, n = rows - 1 - r0;
    return Lane{p + r0 * ld, (uint32_t)((n < q16 ? n : q16) * ld + g)};
  }
  __device__ float at(int k, const Lane &l) const { return (l.first + k)[l.off]; }
};

// bfloat16 table: element (r, k) at p[r * ldp + k], ldp a multiple of 32,
// entries k >= K stored as zeros.  LDS: [BR][32] bf16, 16-byte chunk c
// (8 k) of row r stored at chunk c ^ ((r >> 1) & 3).
struct SKh {
  const uint16_t *p;
  int64_t ldp, rows;
  static constexpr int kUnit = 16;
  template <int BR>
  static constexpr int bytes() { return BR * SBK * 2; }
  template <int BR>
  static constexpr int slots() { return bytes<BR>() / kUnit; }
  __device__ const char *base(int64_t r0, int k0) const {
    return reinterpret_cast<const char *>(p + r0 * ldp + k0);
  }
  template <int BR>
  __device__ uint32_t lane_off(int s, int64_t r0) const {
    const int r = s >> 2, c = (s & 3) ^ ((r >> 1) & 3);
    const int64_t gr = r0 + r < rows ? r0 + r : rows - 1;
    return (uint32_t)(((gr - r0) * ldp + 8 * c) * 2);
  }
  // the table is zero-padded to a whole stage: no copy lies beyond the range
  template <int BR>
  __device__ static int k_of(int) { return 0; }
  template <int BR>
  __device__ bf16x8 frag(const char *lds, int rg, int q16, int g4) const {
    const int r = rg * 16 + q16;
    return *reinterpret_cast<const bf16x8 *>(lds + r * 64 + ((g4 ^ ((r >> 1) & 3)) << 4));
  }
};

// The three-part float32 table: part i of element (r, k) at p[r * 3 ldp + i ldp
// + k], each part as an SKh table.  LDS: the parts' tiles one after another.
struct SK3 {
  const uint16_t *p;
  int64_t ldp, rows;
  const float *f;  // the values, rows of ldf
  int64_t ldf;
  static constexpr int kUnit = 16;
  template <int BR>
  static constexpr int bytes() { return 3 * BR * SBK * 2; }
  template <int BR>
  static constexpr int slots() { return bytes<BR>() / kUnit; }
  __device__ const char *base(int64_t r0, int k0) const {
    return reinterpret_cast<const char *>(p + r0 * 3 * ldp + k0);
  }
  template <int BR>
  __device__ uint32_t lane_off(int s, int64_t r0) const {
    const int part = s / (BR * 4), q = s - part * (BR * 4);
    const int r = q >> 2, c = (q & 3) ^ ((r >> 1) & 3);
    const int64_t gr = r0 + r < rows ? r0 + r : rows - 1;
    return (uint32_t)(((gr - r0) * 3 * ldp + part * ldp + 8 * c) * 2);
  }
  template <int BR>
  __device__ static int k_of(int) { return 0; }
  template <int BR>
  __device__ void frag3(const char *lds, int rg, int q16, int g4, bf16x8 (&v)[3]) const {
    const int r = rg * 16 + q16;
    const char *t = lds + r * 64 + ((g4 ^ ((r >> 1) & 3)) << 4);
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] = *reinterpret_cast<const bf16x8 *>(t + i * BR * SBK * 2);
  }
  using Lane = SKc<false>::Lane;
  __device__ Lane lane(int64_t r, int q16, int g) const { return SKc<false>{f, ldf, rows}.lane(r, q16, g); }
  __device__ float at(int k, const Lane &l) const { return (l.first + k)[l.off]; }
};

// bfloat16 k-contiguous rows (activations stored in bfloat16): element
// (r, k) at p[r * ldp + k], valid for r < rows, k < K; ldp a multiple of 8
// with 16-byte aligned rows and K a multiple of 8, so a 16-byte chunk
// (8 k) lies wholly inside or wholly beyond the range.  LDS as SKh.
struct SKb : SKh {
  template <int BR>
  __device__ static int k_of(int s) {
    const int r = s >> 2;
    return 8 * ((s & 3) ^ ((r >> 1) & 3));
  }
};

// ------------------------------------------------------------------ core
template <int BM_, int BN_, int WM_, int WN_, int NS_>
struct SCfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_;
  static constexpr int TM = BM / (WM * 16), TN = BN / (WN * 16);
  static constexpr int NW = WM * WN;  // waves per block
  static_assert(NW == 4 || NW == 8, "waves per block");
  static_assert(TM * WM * 16 == BM && TN * WN * 16 == BN, "tile shape");
  static_assert(NS >= 2 && NS <= 8, "ring depth");
};

// One stage (32 k) of MFMAs for a wave's TM x TN tiles.  FP32 works in part
// products (parts.h), the B tiles two at a time, so that consecutive
// instructions go to 2 TM accumulators and the B parts stay within 24
// registers.
template <class CF, bool F32, class AO, class BO>
__device__ __forceinline__ void mma_stage(const AO &ao, const BO &bo, const char *sa, const char *sb, int wm, int wn,
                                          int q16, int g4, floatx4 (&acc)[CF::TM][CF::TN],
                                          floatx4 (&low)[F32 ? CF::TM : 1][CF::TN]) {
  constexpr int BM = CF::BM, BN = CF::BN;
  if constexpr (F32) {
    bf16x8 a[CF::TM][3];
#pragma unroll
    for (int i = 0; i < CF::TM; ++i) ao.template frag3<BM>(sa, wm * CF::TM + i, q16, g4, a[i]);
#pragma unroll
    for (int j = 0; j < CF::TN; j += 2) {
      bf16x8 b[2][3];
      bo.template frag3<BN>(sb, wn * CF::TN + j, q16, g4, b[0]);
      if (j + 1 < CF::TN) bo.template frag3<BN>(sb, wn * CF::TN + j + 1, q16, g4, b[1]);
      mma_parts(a, b, acc, low, j);
    }
  } else {
    bf16x8 a[CF::TM], b[CF::TN];
#pragma unroll
    for (int i = 0; i < CF::TM; ++i) a[i] = ao.template frag<BM>(sa, wm * CF::TM + i, q16, g4);
#pragma unroll
    for (int j = 0; j < CF::TN; ++j) b[j] = bo.template frag<BN>(sb, wn * CF::TN + j, q16, g4);
#pragma unroll
    for (int i = 0; i < CF::TM; ++i)
#pragma unroll
      for (int j = 0; j < CF::TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
  }
}

// Side inputs (bias of the lane's columns, mask of its elements) of a
// wave's tiles, loaded ahead of the epilogue when they fit in registers
// (at most 12 tiles per wave).
template <class CF, class CS>
struct SidePre {
  static constexpr bool kOn = CS::kSide && CF::TM * CF::TN <= 12;
  floatx4 cb[CF::TN];
  floatx4 em[CF::TM][CF::TN];
};

template <class CF, class CS>
__device__ __forceinline__ void load_side(const CS &cs, SidePre<CF, CS> &sp, int64_t M, int N, int64_t m0, int n0,
                                          int wm, int wn, int q16, int g4) {
#pragma unroll
  for (int j = 0; j < CF::TN; ++j) {
    const int n = n0 + (wn * CF::TN + j) * 16 + 4 * g4;
    sp.cb[j] = n + 3 < N ? cs.colside(n) : floatx4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int i = 0; i < CF::TM; ++i) {
    const int64_t r = m0 + (wm * CF::TM + i) * 16 + q16;
#pragma unroll
    for (int j = 0; j < CF::TN; ++j) {
      const int n = n0 + (wn * CF::TN + j) * 16 + 4 * g4;
      sp.em[i][j] = r < M && n + 3 < N ? cs.elside(r, n, 0) : floatx4{0.f, 0.f, 0.f, 0.f};
    }
  }
}

// Store a consumer wave's tiles: lane (q16, g4) holds row m0 + (wm*TM+i)*16
// + q16 and columns n0 + (wn*TN+j)*16 + 4 g4 .. + 3 of tile (i, j).
template <class CF, class CS>
__device__ __forceinline__ void store_tiles(const CS &cs, const floatx4 (&acc)[CF::TM][CF::TN], int64_t M, int N,
                                            int64_t m0, int n0, int wm, int wn, int q16, int g4,
                                            const SidePre<CF, CS> &sp) {
  if constexpr (SidePre<CF, CS>::kOn) {
#pragma unroll
    for (int i = 0; i < CF::TM; ++i) {
      const int64_t r = m0 + (wm * CF::TM + i) * 16 + q16;
      if (r >= M) continue;
#pragma unroll
      for (int j = 0; j < CF::TN; ++j) {
        const int n = n0 + (wn * CF::TN + j) * 16 + 4 * g4;
        if (n + 3 < N) {
          cs.store4s(r, n, 0, acc[i][j], sp.cb[j], sp.em[i][j]);
        } else {
          for (int q = 0; q < 4; ++q)
            if (n + q < N) cs(r, n + q, 0, acc[i][j][q]);
        }
      }
    }
  } else if constexpr (CS::kSide) {
    // side inputs (bias, mask) of a chunk of tiles first, then its stores;
    // chunks of RG tile rows keep the prefetched values within ~12 tiles
    constexpr int RG = CF::TN >= 12 ? 1 : (12 / CF::TN < CF::TM ? 12 / CF::TN : CF::TM);
    floatx4 cb[CF::TN];
#pragma unroll
    for (int j = 0; j < CF::TN; ++j) {
      const int n = n0 + (wn * CF::TN + j) * 16 + 4 * g4;
      cb[j] = n + 3 < N ? cs.colside(n) : floatx4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i0 = 0; i0 < CF::TM; i0 += RG) {
      floatx4 em[RG][CF::TN];
#pragma unroll
      for (int ii = 0; ii < RG; ++ii) {
        const int64_t r = m0 + (wm * CF::TM + i0 + ii) * 16 + q16;
#pragma unroll
        for (int j = 0; j < CF::TN; ++j) {
          const int n = n0 + (wn * CF::TN + j) * 16 + 4 * g4;
          em[ii][j] = i0 + ii < CF::TM && r < M && n + 3 < N ? cs.elside(r, n, 0) : floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
      // Let the side loads land before the first store.  Without this the
      // compiler may find one of them still pending at the next stage (on a
      // path that stores nothing, e.g. rows beyond M) and wait there for every
      // outstanding store too.  (vmcnt(0), expcnt and lgkmcnt untouched.)
      __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
      for (int ii = 0; ii < RG; ++ii) {
        const int i = i0 + ii;
        if (i >= CF::TM) break;
        const int64_t r = m0 + (wm * CF::TM + i) * 16 + q16;
        if (r >= M) continue;
        auto one = [&](int j) {
          const int n = n0 + (wn * CF::TN + j) * 16 + 4 * g4;
          if (n + 3 < N) {
            cs.store4s(r, n, 0, acc[i][j], cb[j], em[ii][j]);
          } else {
            for (int q = 0; q < 4; ++q)
              if (n + q < N) cs(r, n + q, 0, acc[i][j][q]);
          }
        };
        if constexpr (CS::kPair) {
          // two adjacent tiles per 16-byte store when both lie inside N
          // (a condition uniform over the wave, so every lane swaps)
#pragma unroll
          for (int jp = 0; jp < CF::TN / 2; ++jp) {
            const int j = 2 * jp;
            const int nt = n0 + (wn * CF::TN + j) * 16;
            if (nt + 32 <= N) {
              cs.store_pair(r, nt, g4, acc[i][j], cb[j], em[ii][j], acc[i][j + 1], cb[j + 1], em[ii][j + 1]);
            } else {
              one(j);
              one(j + 1);
            }
          }
          if constexpr (CF::TN % 2 != 0) one(CF::TN - 1);
        } else {
#pragma unroll
          for (int j = 0; j < CF::TN; ++j) one(j);
        }
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < CF::TM; ++i) {
      const int64_t r = m0 + (wm * CF::TM + i) * 16 + q16;
      if (r >= M) continue;
#pragma unroll
      for (int j = 0; j < CF::TN; ++j) {
        const int n = n0 + (wn * CF::TN + j) * 16 + 4 * g4;
        if (n + 3 < N) {
          cs.store4(r, n, 0, acc[i][j]);
        } else {
          for (int q = 0; q < 4; ++q)
            if (n + q < N) cs(r, n + q, 0, acc[i][j][q]);
        }
      }
    }
  }
}

// The stage where the range ends (krem = K - k0 < SBK reduction entries
// left): lanes whose entries lie beyond it copy zeros instead.
template <int BR, class OPND, int STEP, int NW>
__device__ __forceinline__ void dma_stage_tail(const char *base, const uint32_t (&off)[NW], char *dst, int first,
                                               int lane, int krem) {
  constexpr int NSL = OPND::template slots<BR>();
  constexpr int NI = (NSL + 63) / 64;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int inst = first + STEP * i;
    const int s = inst * 64 + lane;
    if ((NI % STEP == 0 || inst < NI) && (NSL % 64 == 0 || s < NSL)) {
      const void *src = OPND::template k_of<BR>(s) < krem ? (const void *)(base + off[i]) : (const void *)zeros_for(s);
      dma_to_lds<OPND::kUnit>(src, dst + inst * 64 * OPND::kUnit);
    }
  }
}

// Number of DMA instructions of an operand that wave `first` (of `step`)
// issues per stage, at most.
template <int BR, class OPND>
constexpr int dma_per_wave(int step) {
  return ((OPND::template slots<BR>() + 63) / 64 + step - 1) / step;
}

// Byte offsets of the lane's DMA copies within a full stage (loop-invariant).
template <int BR, class OPND, int NW>
__device__ __forceinline__ void dma_offsets(const OPND &op, uint32_t (&off)[NW], int first, int step, int lane,
                                            int64_t r0) {
  constexpr int NSL = OPND::template slots<BR>();
  constexpr int NI = (NSL + 63) / 64;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int inst = first + step * i;
    const int s = inst * 64 + lane;
    off[i] = inst < NI && s < NSL ? op.template lane_off<BR>(s, r0) : 0u;
  }
}

// A full stage: every lane copies from the stage's wave-uniform base plus
// its precomputed offset.  The offset passes through an empty asm inside the
// loop so that its zero extension stays next to the add and the copy is
// selected in the scalar-base + 32-bit vector-offset form (a hoisted 64-bit
// offset would cost a 64-bit add and two registers per copy).
template <int BR, class OPND, int STEP, int NW>
__device__ __forceinline__ void dma_stage_full(const char *base, const uint32_t (&off)[NW], char *dst, int first,
                                               int lane) {
  constexpr int NSL = OPND::template slots<BR>();
  constexpr int NI = (NSL + 63) / 64;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int inst = first + STEP * i;
    if ((NI % STEP == 0 || inst < NI) && (NSL % 64 == 0 || inst * 64 + lane < NSL)) {
      uint32_t o = off[i];
      asm volatile("" : "+v"(o));
      dma_to_lds<OPND::kUnit>(base + o, dst + inst * 64 * OPND::kUnit);
    }
  }
}

// One output tile per block; all its waves issue
// their share of every stage's DMA and compute.  Several blocks per CU keep
// loads in flight while another block multiplies or stores.
template <int OP, class CF, bool F32, class AO, class BO, class CS>
__global__ __launch_bounds__(64 * CF::NW, F32 ? 2 : 1) void gemm_stream_kernel(AO ao, BO bo, CS cs, int64_t M,
                                                                              int N, int K, int nbM, int nbN) {
  constexpr int BM = CF::BM, BN = CF::BN, NW = CF::NW;
  constexpr int AB = AO::template bytes<BM>(), BB = BO::template bytes<BN>(), SB = AB + BB;
  constexpr int NIA = (AO::template slots<BM>() + 63) / 64, NIB = (BO::template slots<BN>() + 63) / 64;
  // DMA instructions every wave issues per stage, at least (wave w issues
  // instructions w, w + NW, ...); waits use this count, so a wave with more
  // waits for slightly more than it needs.
  constexpr int NIW = NIA / NW + NIB / NW;
  // ring depth as configured while the pending count fits vmcnt (6 bits)
  constexpr int NS = (CF::NS - 2) * NIW < 64 ? CF::NS : 2, D = NS - 1;
  __shared__ __attribute__((aligned(16))) char lds[NS * SB];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % CF::WM, wn = wave / CF::WM;
  const int q16 = lane & 15, g4 = lane >> 4;
  const TileMap tm(blockIdx.x, nbM, nbN, 1, false);
  const int64_t m0 = (int64_t)tm.mt * BM;
  const int n0 = tm.nt * BN;
  const int niter = (K + SBK - 1) / SBK;

  constexpr int NWA = dma_per_wave<BM, AO>(NW), NWB = dma_per_wave<BN, BO>(NW);
  uint32_t offa[NWA], offb[NWB];
  dma_offsets<BM>(ao, offa, wave, NW, lane, m0);
  dma_offsets<BN>(bo, offb, wave, NW, lane, n0);
  auto issue = [&](int it) {
    char *sa = lds + (it % NS) * SB;
    const int k0 = it * SBK;
    if (k0 + SBK <= K) {
      dma_stage_full<BM, AO, NW>(ao.base(m0, k0), offa, sa, wave, lane);
      dma_stage_full<BN, BO, NW>(bo.base(n0, k0), offb, sa + AB, wave, lane);
    } else {  // the range ends inside this stage: zeros beyond it
      dma_stage_tail<BM, AO, NW>(ao.base(m0, k0), offa, sa, wave, lane, K - k0);
      dma_stage_tail<BN, BO, NW>(bo.base(n0, k0), offb, sa + AB, wave, lane, K - k0);
    }
  };

  floatx4 acc[CF::TM][CF::TN], low[F32 ? CF::TM : 1][CF::TN];
#pragma unroll
  for (int i = 0; i < CF::TM; ++i)
#pragma unroll
    for (int j = 0; j < CF::TN; ++j) {
      acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      if constexpr (F32) low[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

#pragma unroll
  for (int s = 0; s < D; ++s)
    if (s < niter) issue(s);
  auto wait_issue = [&](int it) {
    // D - 1 stages were issued after this one; near the end fewer, and by then
    // they have had the time to arrive
    if (it + D <= niter) wait_barrier<(D - 1) * NIW>();
    else wait_barrier<0>();
    if (it + D < niter) issue(it + D);
  };
  // Side inputs of the epilogue go out after the wait of the second-to-last
  // stage (behind every DMA, so no stage wait has to cover them except the
  // last, which waits for everything): their latency overlaps the last two
  // stages instead of stalling the stores.
  SidePre<CF, CS> sp;
  const int side_it = niter >= 2 ? niter - 2 : 0;
  for (int it = 0; it < niter; ++it) {
    wait_issue(it);
    if constexpr (SidePre<CF, CS>::kOn)
      if (it == side_it) load_side<CF>(cs, sp, M, N, m0, n0, wm, wn, q16, g4);
    const char *sa = lds + (it % NS) * SB;
    mma_stage<CF, F32>(ao, bo, sa, sa + AB, wm, wn, q16, g4, acc, low);
  }
  if constexpr (F32) {
    add_parts(acc, low);
    if (any_odd(acc)) {
      mend_odd<false>(ao, bo, m0 + wm * CF::TM * 16, (int64_t)n0 + wn * CF::TN * 16, M, N, 0, K, acc,
                      [&](int, int64_t r, unsigned want) { return nan_rows(ao, r, 0, K, want); });
      // again, so that they take no registers there
      if constexpr (SidePre<CF, CS>::kOn) load_side<CF>(cs, sp, M, N, m0, n0, wm, wn, q16, g4);
    }
  }
  if constexpr (SidePre<CF, CS>::kOn)
    if (niter == 0) load_side<CF>(cs, sp, M, N, m0, n0, wm, wn, q16, g4);
  store_tiles<CF>(cs, acc, M, N, m0, n0, wm, wn, q16, g4, sp);
}

template <int OP, class CF, bool F32, class AO, class BO, class CS>
int run_stream(AO ao, BO bo, CS cs, int64_t M, int N, int K, hipStream_t st) {
  if (M <= 0 || N <= 0) return 0;
  const int64_t nbM = (M + CF::BM - 1) / CF::BM;
  const int nbN = (N + CF::BN - 1) / CF::BN;
  if (nbM * nbN > 0x7fffffff) return -4;
  hipLaunchKernelGGL((gemm_stream_kernel<OP, CF, F32, AO, BO, CS>), dim3((unsigned)(nbM * nbN)), dim3(64 * CF::NW), 0,
                     st, ao, bo, cs, M, N, K, (int)nbM, nbN);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Row-major output with compile-time side inputs: BIAS adds bias_n[n], MASK
// zeroes entries where omask (indexed as C) <= 0; optional ReLU in between.
// ReLU bit masks (BM): 1 = write bit (stored value > 0) of every output to
// obits, 2 = take the mask (MASK) from mbits instead of omask.  Bit c % 16 of
// word r * ldm + c / 16 belongs to element (r, c); N is a multiple of 16, so
// a 16-column tile is one word, held four bits per lane by the four lanes
// (q16, g4) of one row.
__device__ __forceinline__ floatx4 bits_mask(const uint16_t *mbits, int64_t ldm, int64_t r, int n) {
  const unsigned w = (unsigned)mbits[r * ldm + n / 16] >> (n & 15);
  return floatx4{(float)(w & 1u), (float)((w >> 1) & 1u), (float)((w >> 2) & 1u), (float)((w >> 3) & 1u)};
}
__device__ __forceinline__ void bits_store(uint16_t *obits, int64_t ldm, int64_t r, int n, unsigned nib) {
  // OR the nibbles of the four lanes of this row (lanes q16 + 16 g4): the
  // row swaps exchange lane l with l ^ 16, then with l ^ 32, in registers
  const unsigned w = bits_word(nib, (n & 15) >> 2);
  if ((n & 15) == 0) obits[r * ldm + n / 16] = (uint16_t)w;
}

// Row-major output with compile-time side inputs: BIAS adds bias_n[n], MASK
// zeroes entries where omask (indexed as C) <= 0, or where the ReLU bit is
// clear (BM = 2); optional ReLU in between; BM = 1 also writes the ReLU bits.
template <bool BIAS, bool MASK, int BM = 0>
struct CRowSide {
  static constexpr bool kSide = BIAS || MASK;
  static constexpr bool kPair = false;
  static constexpr bool kBias = BIAS, kMask = MASK, kHalf = false;
  static constexpr int kBits = BM;
  float *C;
  int64_t ldc;
  int relu;
  const float *bias_n, *omask;
  const uint16_t *mbits = nullptr;
  uint16_t *obits = nullptr;
  int64_t ldm = 0;
  __device__ void operator()(int64_t r, int n, int, float v) const {
    const int64_t o = r * ldc + n;
    if constexpr (BIAS) v += bias_n[n];
    if (relu) v = fmaxf(v, 0.0f);
    if constexpr (MASK) {
      if constexpr (BM == 2) v = (mbits[r * ldm + n / 16] >> (n & 15)) & 1u ? v : 0.0f;
      else v = omask[o] > 0.0f ? v : 0.0f;
    }
    C[o] = v;
  }
  __device__ void store4(int64_t r, int n, int g, floatx4 v) const {
    for (int q = 0; q < 4; ++q) (*this)(r, n + q, g, v[q]);
  }
  __device__ floatx4 colside(int n) const {
    if constexpr (BIAS) return ld4(bias_n + n);
    else return floatx4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ floatx4 elside(int64_t r, int n, int) const {
    if constexpr (MASK && BM == 2) return bits_mask(mbits, ldm, r, n);
    else if constexpr (MASK) return ld4(omask + r * ldc + n);
    else return floatx4{1.f, 1.f, 1.f, 1.f};
  }
  __device__ void store4s(int64_t r, int n, int, floatx4 v, floatx4 cb, floatx4 em) const {
    unsigned nib = 0;
    for (int q = 0; q < 4; ++q) {
      if constexpr (BIAS) v[q] += cb[q];
      if (relu) v[q] = fmaxf(v[q], 0.0f);
      if constexpr (MASK) v[q] = em[q] > 0.0f ? v[q] : 0.0f;
      nib |= (v[q] > 0.0f ? 1u : 0u) << q;
    }
    __builtin_memcpy(C + r * ldc + n, &v, 16);
    if constexpr (BM == 1) bits_store(obits, ldm, r, n, nib);
  }
};

// The same with a bfloat16 output (RNE) and a bfloat16 mask: activations and
// their gradients stored in bfloat16.  ldc a multiple of 4, 8-byte aligned rows.
// ReLU bits (BM = 1) describe the stored (rounded) values.
template <bool BIAS, bool MASK, int BM = 0>
struct CRowSideH {
  static constexpr bool kSide = BIAS || MASK;
  static constexpr bool kPair = true;
  static constexpr bool kBias = BIAS, kMask = MASK, kHalf = true;
  static constexpr int kBits = BM;
  uint16_t *C;
  int64_t ldc;
  int relu;
  const float *bias_n;
  const uint16_t *omask;
  const uint16_t *mbits = nullptr;
  uint16_t *obits = nullptr;
  int64_t ldm = 0;
  __device__ static float widen(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }
  __device__ void operator()(int64_t r, int n, int, float v) const {
    const int64_t o = r * ldc + n;
    if constexpr (BIAS) v += bias_n[n];
    if (relu) v = fmaxf(v, 0.0f);
    if constexpr (MASK) {
      if constexpr (BM == 2) v = (mbits[r * ldm + n / 16] >> (n & 15)) & 1u ? v : 0.0f;
      else v = widen(omask[o]) > 0.0f ? v : 0.0f;
    }
    C[o] = to_bf16_bits(v);
  }
  __device__ void store4(int64_t r, int n, int g, floatx4 v) const {
    for (int q = 0; q < 4; ++q) (*this)(r, n + q, g, v[q]);
  }
  __device__ floatx4 colside(int n) const {
    if constexpr (BIAS) return ld4(bias_n + n);
    else return floatx4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ floatx4 elside(int64_t r, int n, int) const {
    if constexpr (MASK && BM == 2) {
      return bits_mask(mbits, ldm, r, n);
    } else if constexpr (MASK) {
      uint16_t h[4];
      __builtin_memcpy(h, omask + r * ldc + n, 8);
      return floatx4{widen(h[0]), widen(h[1]), widen(h[2]), widen(h[3])};
    } else {
      return floatx4{1.f, 1.f, 1.f, 1.f};
    }
  }
  __device__ void store4s(int64_t r, int n, int, floatx4 v, floatx4 cb, floatx4 em) const {
    uint16_t h[4];
    unsigned nib = 0;
    for (int q = 0; q < 4; ++q) {
      if constexpr (BIAS) v[q] += cb[q];
      if (relu) v[q] = fmaxf(v[q], 0.0f);
      if constexpr (MASK) v[q] = em[q] > 0.0f ? v[q] : 0.0f;
      h[q] = to_bf16_bits(v[q]);
      nib |= (widen(h[q]) > 0.0f ? 1u : 0u) << q;
    }
    __builtin_memcpy(C + r * ldc + n, h, 8);
    if constexpr (BM == 1) bits_store(obits, ldm, r, n, nib);
  }
  // Tiles j (columns nt..nt+15) and j+1 (nt+16..nt+31) of one row: lane g4
  // holds columns 4 g4..4 g4+3 of both.  A row swap (lane l with l ^ 16,
  // i.e. g4 with g4 ^ 1) hands each even lane its neighbour's half of tile
  // j and each odd lane its neighbour's half of tile j+1, so every lane
  // stores 8 contiguous columns (16 bytes) with one instruction.
  __device__ void store_pair(int64_t r, int nt, int g4, floatx4 v0, floatx4 cb0, floatx4 em0, floatx4 v1,
                             floatx4 cb1, floatx4 em1) const {
    uint32_t w0[2], w1[2];
    unsigned nib0 = 0, nib1 = 0;
    for (int q = 0; q < 4; ++q) {
      if constexpr (BIAS) {
        v0[q] += cb0[q];
        v1[q] += cb1[q];
      }
      if (relu) {
        v0[q] = fmaxf(v0[q], 0.0f);
        v1[q] = fmaxf(v1[q], 0.0f);
      }
      if constexpr (MASK) {
        v0[q] = em0[q] > 0.0f ? v0[q] : 0.0f;
        v1[q] = em1[q] > 0.0f ? v1[q] : 0.0f;
      }
    }
    for (int q = 0; q < 2; ++q) {
      const uint16_t a = to_bf16_bits(v0[2 * q]), b = to_bf16_bits(v0[2 * q + 1]);
      const uint16_t c = to_bf16_bits(v1[2 * q]), d = to_bf16_bits(v1[2 * q + 1]);
      w0[q] = (uint32_t)a | ((uint32_t)b << 16);
      w1[q] = (uint32_t)c | ((uint32_t)d << 16);
      if constexpr (BM == 1) {
        nib0 |= ((widen(a) > 0.0f ? 1u : 0u) | (widen(b) > 0.0f ? 2u : 0u)) << (2 * q);
        nib1 |= ((widen(c) > 0.0f ? 1u : 0u) | (widen(d) > 0.0f ? 2u : 0u)) << (2 * q);
      }
    }
    if constexpr (BM == 1) {
      bits_store(obits, ldm, r, nt + 4 * g4, nib0);
      bits_store(obits, ldm, r, nt + 16 + 4 * g4, nib1);
    }
    const bool odd = g4 & 1;
    uint32_t out[4];
    for (int q = 0; q < 2; ++q) {
      const uint32_t mine = odd ? w0[q] : w1[q];  // the half the partner stores
      const Both x = swap16(mine);
      // one of the two results is this lane's own value, the other the partner's
      const uint32_t theirs = x.a ^ x.b ^ mine;
      if (odd) {
        out[q] = theirs;
        out[2 + q] = w1[q];
      } else {
        out[q] = w0[q];
        out[2 + q] = theirs;
      }
    }
    const int col = odd ? nt + 16 + 4 * (g4 - 1) : nt + 4 * g4;
    __builtin_memcpy(C + r * ldc + col, out, 16);
  }
};

// --------------------------------------------- short-reduction kernel
// C[M][N] = A[M][K] B[N][K]^T for 128 < K <= 160 and N <= 1440: the folded
// forward of a layer with three input channels and the input gradient of a
// layer with three output channels (K = 135, N = 1440 in the three-shell
// stack).  With five k-slices per tile, a block of the tiled core above
// spends most of its life waiting for the loads of its first slices.  Here
// a block keeps its rows of A in registers, loaded once, and sweeps every
// column tile of the table, which streams through an LDS ring by DMA (the
// table stays in L2).  The stores of one tile are in flight while the next
// tiles are loaded and multiplied.
//
// Waits count vector-memory operations in issue order: the DMA of tile t
// is waited for with s_waitcnt vmcnt(n), n = a lower bound of the
// operations the wave issued after it (the stores of the tiles in between,
// the DMA of later tiles).  The block holding the last rows skips the
// stores of rows beyond M, so there the store count is taken as zero.
//
// Side data stay in LDS for the block's whole life: the bias of every
// column (forward), the ReLU bit words of the block's rows (the input
// gradient's mask), or the bit words the forward produces for the block's
// rows, which go to memory once, as one contiguous run, when the block ends.
// Per element the epilogue is the tiled core's (bias, ReLU, mask, RNE
// rounding, bits of the stored value) with the ReLU chosen at compile time;
// the accumulation order is also the tiled core's (k-slices in order; FP32:
// within a slice the six part products of parts.h in their order), so the
// results are bitwise the same.
namespace astat {

#ifndef DLM_ASTAT_TM
#define DLM_ASTAT_TM 2
#endif
#ifndef DLM_ASTAT_BN_BF16
#define DLM_ASTAT_BN_BF16 32
#endif
#ifndef DLM_ASTAT_BN_F32
#define DLM_ASTAT_BN_F32 32
#endif
#ifndef DLM_ASTAT_D_BF16
#define DLM_ASTAT_D_BF16 3
#endif
#ifndef DLM_ASTAT_D_F32
#define DLM_ASTAT_D_F32 1
#endif

constexpr int TM = DLM_ASTAT_TM;  // 16-row groups per wave
// Waves per block: the FP32 form's three-part tiles leave LDS for one block
// per CU, so it has eight waves in it; BF16 has two or three blocks of four.
template <bool F32>
constexpr int NW = F32 ? 8 : 4;
template <bool F32>
constexpr int BM = 16 * TM * NW<F32>;  // rows per block
constexpr int KS = 5;             // 32-k slices (128 < K <= 160)
constexpr int kMaxN = 1440;       // columns whose side data fit in LDS

// Lane (q16, g4) holds A[row][32 s + 8 g4 .. + 7] (row = 16 i + q16 of the
// wave) rounded to bfloat16, in FP32 its three parts.
template <bool F32>
struct AFrag {
  bf16x8 v[KS][TM];
};
template <>
struct AFrag<true> {
  bf16x8 v[KS][TM][3];
};

// NV consecutive values of a row from k0 on, zeros at and beyond K.
template <int NV>
__device__ __forceinline__ void load_run(const float *row, int k0, int K, float (&out)[NV]) {
  if (k0 + NV <= K) {
#pragma unroll
    for (int q = 0; q < NV / 4; ++q) {
      const floatx4 t = ld4(row + k0 + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) out[4 * q + e] = t[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < NV; ++e) out[e] = k0 + e < K ? row[k0 + e] : 0.0f;
  }
}

template <bool F32>
__device__ __forceinline__ void load_a(const float *A, int64_t lda, int64_t M, int K, int64_t r0, int q16, int g4,
                                       AFrag<F32> &a) {
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    int64_t r = r0 + i * 16 + q16;
    if (r >= M) r = M - 1;  // rows beyond M read a valid row and are never stored
    const float *row = A + r * lda;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float t[8];
      load_run<8>(row, 32 * s + 8 * g4, K, t);
      if constexpr (F32) {
        split3(floatx4{t[0], t[1], t[2], t[3]}, floatx4{t[4], t[5], t[6], t[7]}, a.v[s][i]);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) a.v[s][i][e] = (__bf16)t[e];
      }
    }
  }
}

// Which of the 16 rows of group i have a NaN, one bit each (from their first
// parts, which are NaN where the value is).
__device__ __forceinline__ unsigned nan_group(const AFrag<true> &a, int i) {
  bool nan = false;
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float v = (float)a.v[s][t][0][e];
        nan |= t == i && v != v;
      }
  const uint64_t m = __ballot(nan);
  return (unsigned)(m | m >> 16 | m >> 32 | m >> 48) & 0xffffu;
}

template <class CS>
constexpr int bias_bytes() {
  return CS::kBias ? kMaxN * 4 : 0;
}
template <class CS, int ROWS>
constexpr int side_bytes() {
  constexpr int b = bias_bytes<CS>() + ((CS::kMask || CS::kBits == 1) ? ROWS * (kMaxN / 16) * 2 : 0);
  return b > 0 ? b : 16;
}

// Two floats rounded to bfloat16 (nearest even) and packed, lo in the low
// half: one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 h2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, h2));
}

// Two adjacent 16-column tiles of one row in bfloat16 (lane g4 holds
// columns 4 g4 .. 4 g4 + 3 of both, two packed words each): a row swap
// hands each lane 8 contiguous columns, stored with one 16-byte store.
__device__ __forceinline__ void store_pair_bf16(uint16_t *C, int64_t ldc, int64_t r, int nt, int g4,
                                                const uint32_t (&w0)[2], const uint32_t (&w1)[2]) {
  const bool odd = g4 & 1;
  uint32_t out[4];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint32_t mine = odd ? w0[q] : w1[q];  // the half the partner stores
    const Both x = swap16(mine);
    const uint32_t theirs = x.a ^ x.b ^ mine;  // one result is this lane's own value
    if (odd) {
      out[q] = theirs;
      out[2 + q] = w1[q];
    } else {
      out[q] = w0[q];
      out[2 + q] = theirs;
    }
  }
  const int col = odd ? nt + 16 + 4 * (g4 - 1) : nt + 4 * g4;
  __builtin_memcpy(C + r * ldc + col, out, 16);
}

template <bool F32, int BN, int D, bool RELU, class BO, class CS>
__global__ __launch_bounds__(64 * NW<F32>) void astat_kernel(const float *A, int64_t lda, int64_t M, int K, BO bo,
                                                             CS cs, int N) {
  constexpr int TN = BN / 16, NS = D + 1, NWV = astat::NW<F32>, NT_ = 64 * NWV, BM = astat::BM<F32>;
  constexpr bool kHalf = CS::kHalf, kMaskIn = CS::kMask, kBitsOut = CS::kBits == 1;
  static_assert(!CS::kMask || CS::kBits == 2, "masks from ReLU bits only");
  constexpr int SLAB = BO::template bytes<BN>();  // one 32-k slice of a column tile
  constexpr int TILE = KS * SLAB;
  constexpr int NSL = BO::template slots<BN>();
  static_assert(BO::kUnit == 16 && NSL % 64 == 0, "whole 16-byte DMA instructions per slice");
  constexpr int NI = NSL / 64;        // DMA instructions per slice
  constexpr int NIT = KS * NI;        // per tile, dealt round-robin to the waves
  constexpr int KW = (NIT + NWV - 1) / NWV;  // per wave per tile, at most
  constexpr int IW = NIT / NWV;              // and at least
  constexpr int KB = F32 ? 2 : BO::template bytes<1>() / SBK;  // bytes from one k to the next
  // stores per wave per tile, at least: one per pair of bfloat16 tiles (and
  // per odd tile), or one per float32 tile
  constexpr int SW = TM * (kHalf ? (TN + 1) / 2 : TN);
  static_assert(D >= 1 && D <= 3 && D * SW + (D - 1) * IW < 64, "vmcnt range");
  __shared__ __attribute__((aligned(16))) char lds[NS * TILE + side_bytes<CS, BM>()];
  static_assert((NS * TILE + bias_bytes<CS>()) % 16 == 0, "16-byte aligned bit words in LDS");
  float *sbias = reinterpret_cast<float *>(lds + NS * TILE);
  uint16_t *sbits = reinterpret_cast<uint16_t *>(lds + NS * TILE + bias_bytes<CS>());

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q16 = lane & 15, g4 = lane >> 4;
  const int64_t m0 = (int64_t)blockIdx.x * BM;
  const int64_t r0 = m0 + wave * 16 * TM;
  // the block's column tiles: all of them, or its share of a split grid
  const int T0 = (int)((int64_t)(N / BN) * blockIdx.y / gridDim.y);
  const int NT = (int)((int64_t)(N / BN) * (blockIdx.y + 1) / gridDim.y) - T0;
  const int wpr = N / 16;  // ReLU-bit words per row
  const bool full = m0 + BM <= M;

  // The wave's DMA instructions of a tile (q = wave + NWV k: slice q / NI,
  // instruction q % NI of it): per-lane byte offsets from the tile's first
  // table row, and LDS offsets in the slot (the same for every tile: N is a
  // multiple of BN, so no row is clamped).
  uint32_t voff[KW];
  int loff[KW];
  const int nq = (NIT - wave + NWV - 1) / NWV;
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const int q = wave + NWV * k, sl = q / NI, ins = q - sl * NI;
    voff[k] = q < NIT ? bo.template lane_off<BN>(ins * 64 + lane, 0) + uint32_t(sl * SBK * KB) : 0u;
    loff[k] = sl * SLAB + ins * 64 * 16;
  }
  const int64_t tstride = bo.base(BN, 0) - bo.base(0, 0);  // bytes between column tiles
  const char *gtab = bo.base(0, 0) + T0 * tstride;
  auto issue = [&](int t) {
    const char *src = gtab + (int64_t)t * tstride;
    char *dst = lds + (t % NS) * TILE;
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      if (k < nq) {
        uint32_t o = voff[k];
        asm volatile("" : "+v"(o));
        dma_to_lds<16>(src + o, dst + loff[k]);
      }
    }
  };

  // prologue: A into registers, the first tiles and the side data into LDS
  AFrag<F32> a;
  load_a<F32>(A, lda, M, K, r0, q16, g4, a);
#pragma unroll
  for (int t = 0; t < D; ++t)
    if (t < NT) issue(t);
  if constexpr (CS::kBias)
    for (int c = tid; c < N; c += NT_) sbias[c] = cs.bias_n[c];
  if constexpr (kMaskIn) {
    // the block's bit words are one run of memory: 16-byte copies when it
    // is whole and aligned (LDS side: the tiles and the bias are multiples
    // of 16 bytes), else word by word with rows clamped
    const uint16_t *src = cs.mbits + m0 * wpr;
    if (full && (BM * wpr) % 8 == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
      for (int c = tid; c < BM * wpr / 8; c += NT_)
        __builtin_memcpy(reinterpret_cast<uint4 *>(sbits) + c, reinterpret_cast<const uint4 *>(src) + c, 16);
    } else {
      for (int c = tid; c < BM * wpr; c += NT_) {
        const int rr = c / wpr;
        int64_t r = m0 + rr;
        if (r >= M) r = M - 1;
        sbits[c] = cs.mbits[r * wpr + (c - rr * wpr)];
      }
    }
  }
  wait_barrier<0>();

  for (int t = 0; t < NT; ++t) {
    if (t >= D) {
      // after the DMA of tile t this wave issued: the stores of tiles
      // t-D .. t-1 and the DMA of tiles t+1 .. t+D-1 (those that exist)
      const int later = min(D - 1, NT - 1 - t);
      if constexpr (D == 1) {
        if (full) wait_barrier<SW>();
        else wait_barrier<0>();
      } else if constexpr (D == 2) {
        if (full) {
          if (later) wait_barrier<2 * SW + IW>();
          else wait_barrier<2 * SW>();
        } else {
          if (later) wait_barrier<IW>();
          else wait_barrier<0>();
        }
      } else {
        if (full) {
          if (later == 2) wait_barrier<3 * SW + 2 * IW>();
          else if (later == 1) wait_barrier<3 * SW + IW>();
          else wait_barrier<3 * SW>();
        } else {
          if (later == 2) wait_barrier<2 * IW>();
          else if (later == 1) wait_barrier<IW>();
          else wait_barrier<0>();
        }
      }
    } else if (t > 0) {
      // every wave is done reading the slot refilled next (tiles t < D
      // arrived before the prologue's barrier)
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    if (t + D < NT) issue(t + D);

    const char *tile = lds + (t % NS) * TILE;
    floatx4 acc[TM][TN], low[F32 ? TM : 1][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (F32) low[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
    for (int sl = 0; sl < KS; ++sl) {
      const char *sb = tile + sl * SLAB;
      if constexpr (F32) {
        bf16x8 b[TN][3];
#pragma unroll
        for (int j = 0; j < TN; ++j) bo.template frag3<BN>(sb, j, q16, g4, b[j]);
        mma_parts(a.v[sl], b, acc, low, 0);
      } else {
        bf16x8 b[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) b[j] = bo.template frag<BN>(sb, j, q16, g4);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a.v[sl][i], acc[i][j], 0, 0, 0);
      }
    }
    if constexpr (F32) {
      add_parts(acc, low);
      if (any_odd(acc))
        mend_odd<false>(SKc<false>{A, lda, M}, bo, r0, (int64_t)(T0 + t) * BN, M, N, 0, K, acc,
                        [&](int i, int64_t, unsigned) { return nan_group(a, i); });
    }

    // epilogue: bias, ReLU, mask, rounding, bits; then the stores
    const int n0 = (T0 + t) * BN;
    floatx4 cbv[TN];
    if constexpr (CS::kBias) {
#pragma unroll
      for (int j = 0; j < TN; ++j) cbv[j] = *reinterpret_cast<const floatx4 *>(sbias + n0 + 16 * j + 4 * g4);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int rr = wave * 16 * TM + i * 16 + q16;
      const int64_t r = m0 + rr;
      floatx4 v[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        v[j] = acc[i][j];
        unsigned mnib = 15u;
        if constexpr (kMaskIn) mnib = (unsigned)sbits[rr * wpr + n0 / 16 + j] >> (4 * g4);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (CS::kBias) v[j][q] += cbv[j][q];
          if constexpr (RELU) v[j][q] = fmaxf(v[j][q], 0.0f);
          if constexpr (kMaskIn) v[j][q] = (mnib >> q) & 1u ? v[j][q] : 0.0f;
        }
      }
      if constexpr (kHalf) {
        uint32_t h2[TN][2];
        unsigned nib[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          nib[j] = 0;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            // both values rounded (RNE) by one packed conversion
            const uint32_t w = pack2_bf16(v[j][2 * q], v[j][2 * q + 1]);
            h2[j][q] = w;
            if constexpr (kBitsOut)  // the stored (rounded) value is > 0
              nib[j] |= ((__builtin_bit_cast(float, w << 16) > 0.0f ? 1u : 0u) |
                         (__builtin_bit_cast(float, w & 0xffff0000u) > 0.0f ? 2u : 0u))
                        << (2 * q);
          }
        }
        if constexpr (kBitsOut) {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const unsigned w = bits_word(nib[j], g4);
            if (g4 == 0) sbits[rr * wpr + n0 / 16 + j] = (uint16_t)w;
          }
        }
        if (r >= M) continue;
#pragma unroll
        for (int jp = 0; jp < TN / 2; ++jp)
          store_pair_bf16(cs.C, cs.ldc, r, n0 + 32 * jp, g4, h2[2 * jp], h2[2 * jp + 1]);
        if constexpr (TN % 2 != 0) __builtin_memcpy(cs.C + r * cs.ldc + n0 + 16 * (TN - 1) + 4 * g4, h2[TN - 1], 8);
      } else {
        if constexpr (kBitsOut) {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            unsigned nib = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) nib |= (v[j][q] > 0.0f ? 1u : 0u) << q;
            const unsigned w = bits_word(nib, g4);
            if (g4 == 0) sbits[rr * wpr + n0 / 16 + j] = (uint16_t)w;
          }
        }
        if (r >= M) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) __builtin_memcpy(cs.C + r * cs.ldc + n0 + 16 * j + 4 * g4, &v[j], 16);
      }
    }
  }

  if constexpr (kBitsOut) {
    // the block's bit words, rows m0 .. m0 + BM - 1 (those below M): one
    // contiguous run of memory, or its columns' words of each row
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int64_t rows = min((int64_t)BM, M - m0);
    uint16_t *dst = cs.obits + m0 * wpr;
    if (gridDim.y > 1) {
      const int w0 = T0 * (BN / 16), nw = NT * (BN / 16);
      for (int64_t c = tid; c < rows * nw; c += NT_) {
        const int64_t at = c / nw * wpr + w0 + c % nw;
        dst[at] = sbits[at];
      }
      return;
    }
    const int64_t nw = rows * wpr;
    if (((reinterpret_cast<uintptr_t>(dst)) & 15) == 0) {
      const int64_t n16 = nw / 8;
      for (int64_t c = tid; c < n16; c += NT_)
        __builtin_memcpy(dst + 8 * c, reinterpret_cast<const uint4 *>(sbits) + c, 16);
      for (int64_t c = 8 * n16 + tid; c < nw; c += NT_) dst[c] = sbits[c];
    } else {
      for (int64_t c = tid; c < nw; c += NT_) dst[c] = sbits[c];
    }
  }
}

// Which output policies the kernel takes: bias or none, or the ReLU mask
// from bit words (an activation mask would be as large as the output).
template <class CS>
constexpr bool takes() {
  return !CS::kMask || CS::kBits == 2;
}

// DLM_TILED_ONLY=1 in the environment sends these GEMMs to the tiled core
// instead (the same results bit for bit; read at every call, for tests).
inline bool tiled_only() {
  const char *e = std::getenv("DLM_TILED_ONLY");
  return e && e[0] == '1';
}

template <bool F32>
bool ok(const TableGemm &t) {
  constexpr int BN = F32 ? DLM_ASTAT_BN_F32 : DLM_ASTAT_BN_BF16;
  return DLM_ASTAT != 0 && !tiled_only() && t.A != nullptr && t.Ah == nullptr && t.K > SBK * (KS - 1) && t.K <= SBK * KS &&
         t.N % BN == 0 && t.N <= kMaxN && t.N % 16 == 0 && t.M > 0 && (t.M + BM<F32> - 1) / BM<F32> <= 0x7fffffff;
}

template <bool F32, class BO, class CS>
int run(const TableGemm &t, BO bo, CS cs, hipStream_t st) {
  constexpr int BN = F32 ? DLM_ASTAT_BN_F32 : DLM_ASTAT_BN_BF16;
  constexpr int D = F32 ? DLM_ASTAT_D_F32 : DLM_ASTAT_D_BF16;
  const unsigned blocks = (unsigned)((t.M + BM<F32> - 1) / BM<F32>);
  // FP32, whose blocks have a compute unit each: batches with fewer blocks
  // than that share a row block's columns among several (the rows are read
  // once more for each)
  unsigned share = 1;
  if constexpr (F32)
    if (blocks < 256) share = std::min<unsigned>(256 / blocks, unsigned(t.N / BN));
  const dim3 grid(blocks, share), threads(64 * NW<F32>);
  if constexpr (CS::kBias) {  // the forward: ReLU fused or not
    if (t.relu)
      hipLaunchKernelGGL((astat_kernel<F32, BN, D, true, BO, CS>), grid, threads, 0, st, t.A, t.lda, t.M, t.K, bo, cs,
                         t.N);
    else
      hipLaunchKernelGGL((astat_kernel<F32, BN, D, false, BO, CS>), grid, threads, 0, st, t.A, t.lda, t.M, t.K, bo, cs,
                         t.N);
  } else {
    if (t.relu) return -3;  // an input gradient never fuses a ReLU
    hipLaunchKernelGGL((astat_kernel<F32, BN, D, false, BO, CS>), grid, threads, 0, st, t.A, t.lda, t.M, t.K, bo, cs,
                       t.N);
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace astat

// BF16, N > 96 (N = 135/136, and 1440/2880 = 10/20 tiles exactly): one
// configuration; for the K = 135 GEMMs it also amortises a block's fixed
// cost (DMA offsets, first loads, epilogue) over 1.5x the output of 128 x 96
using SCfgNarrow = SCfg<128, 144, 4, 1, 3>;
using SCfgSmall = SCfg<128, 48, 4, 1, 3>;   // N <= 96
// BF16, long reductions onto wide outputs without a mask to load: 64 x 96 per
// wave reads 10 KB of LDS for 24 matrix instructions where 32 x 144 reads 11 KB
// for 18 (8192 x 2880 x 2880 187 -> 175 us; with the mask, whose loads then do
// not fit in registers ahead of the epilogue, 203 -> 228 us).  From bfloat16
// rows only: of float32 ones a ring of three fills 115 KB, one block to a
// compute unit (the same product 213 -> 260 us, 120000 x 720 x 720 314 -> 460)
using SCfgWide = SCfg<256, 96, 4, 1, 3>;
// BF16, too few rows for a block per compute unit: small tiles, and a ring deep
// enough that a block waits for memory once and not at every stage (8192 x 135
// x 2880, 64 blocks: 47 -> 27 us; with a ring of four 36 us).  2000 rows, 2880
// onto 960, 112 blocks: 63 -> 79 us; 1440 onto 720, 80 blocks, 2000 rows gain
using SCfgFew = SCfg<64, 48, 4, 1, 8>;
// FP32: the tile that takes the fewest stage times for the batch at hand.  A
// stage (32 k) of one block took, in us, with up to half of the chip's blocks
// resident and with all of them (blocks per compute unit by LDS):
//   256 x 144, eight waves  2.3  3.0   (one)
//   256 x 96, eight waves   1.8  2.1   (one)
//   64 x 144                1.1  1.85  (two)
//   128 x 48                0.93 1.29  (two)
//   64 x 48                 0.66 0.80  (two)
// (1440 and 2880 inputs onto 135, 1440 and 2880 outputs, 256 to 65536 voxels,
// e.g. 1440 onto 135: 256 voxels 109, 84, 55, 46, 33 us; 30000 voxels 112, 94,
// 82, 97, 102; 65536 voxels 141, 205, 177, 194, 234.)  Large batches run at
// 256 x 144: against the float32 matrix instructions 8192 x 2880 x 1440 591 ->
// 383 us (177 TFLOP/s, 1.06 PFLOP/s of part products), K = 1440 onto 135 at 1M
// voxels 3.30 -> 2.18 ms, the K = 135 kernel above 3.82 -> 2.55 ms.
// Rows that are not whole 16-byte pieces are copied element by element, four
// times the instructions, and a block alone on its compute unit has nothing to
// hide them behind: up to 1280 inputs, where the stages do, those take one of
// the tiles with two blocks, whose stages then took the times in the last
// column (120000 voxels, 45 onto 480: 64 x 144 107 us, 128 x 48 111, 256 x 144
// 185, 256 x 96 151; onto 1440 with a mask to load 406, 462, 587 and 848; 315
// onto 1440 787, 911, 962, 853; 1485 onto 1440 3.50, 3.59, 3.45, 3.10 ms).
struct F32Tile {
  int bm, bn, slots;  // slots: blocks of a chip of 256 compute units
  double half, full, pieces;
};
inline int f32_tile(int64_t M, int N, int K, bool whole) {
  static constexpr F32Tile kTiles[] = {{256, 144, 256, 2.3, 3.0, 3.0},
                                       {256, 96, 256, 1.8, 2.1, 2.1},
                                       {64, 144, 512, 1.1, 1.85, 1.65},
                                       {128, 48, 512, 0.93, 1.29, 1.33},
                                       {64, 48, 512, 0.66, 0.80, 0.80}};
  const bool two = !whole && K < 1280;
  int best = -1;
  double least = 0.0;
  for (int i = two ? 2 : 0; i < 5; ++i) {
    const F32Tile &c = kTiles[i];
    const int64_t blocks = (M + c.bm - 1) / c.bm * ((N + c.bn - 1) / c.bn), rest = blocks % c.slots;
    const double full = two ? c.pieces : c.full;
    const double cost = double(blocks / c.slots) * full + (rest == 0 ? 0.0 : rest <= c.slots / 2 ? c.half : full);
    if (best < 0 || cost < least) {
      best = i;
      least = cost;
    }
  }
  return best;
}

template <int OP, bool F32, class AO, class BO, class CS>
int stream_table_c(AO ao, BO bo, CS cs, const TableGemm &t, hipStream_t st) {
  if constexpr (astat::takes<CS>())
    if (astat::ok<F32>(t)) return astat::run<F32>(t, bo, cs, st);
  if constexpr (F32) {
    auto go = [&](auto cfg) { return run_stream<OP, decltype(cfg), F32>(ao, bo, cs, t.M, t.N, t.K, st); };
    switch (f32_tile(t.M, t.N, t.K, AO::kUnit == 16)) {
      case 0: return go(SCfg<256, 144, 8, 1, 2>{});
      case 1: return go(SCfg<256, 96, 8, 1, 2>{});
      case 2: return go(SCfg<64, 144, 4, 1, 2>{});
      case 3: return go(SCfg<128, 48, 4, 1, 3>{});
      default: return go(SCfg<64, 48, 4, 1, 4>{});
    }
  } else {
    if (t.N <= 96) return run_stream<OP, SCfgSmall, F32>(ao, bo, cs, t.M, t.N, t.K, st);
    if constexpr (!CS::kMask && std::is_same_v<AO, SKb>)
      if (t.N > 144 && t.K > 256 && (t.M + 255) / 256 * ((t.N + 95) / 96) >= 512)
        return run_stream<OP, SCfgWide, F32>(ao, bo, cs, t.M, t.N, t.K, st);
    if ((t.M + 127) / 128 * ((t.N + 143) / 144) <= 96)
      return run_stream<OP, SCfgFew, F32>(ao, bo, cs, t.M, t.N, t.K, st);
    return run_stream<OP, SCfgNarrow, F32>(ao, bo, cs, t.M, t.N, t.K, st);
  }
}

// the forward GEMM adds the folded bias; the input-gradient GEMM may mask
template <int OP, bool F32, class AO, class BO>
int stream_table(AO ao, BO bo, const TableGemm &t, hipStream_t st) {
  const int64_t ldm = t.N / 16;  // ReLU-bit words per row
  if constexpr (!F32) {
    if (t.Ch) {  // bfloat16 output (and mask)
      if constexpr (OP == kOpFoldFwd) {
        if (t.relu_bits_out)
          return stream_table_c<OP, F32>(
              ao, bo, CRowSideH<true, false, 1>{t.Ch, t.ldc, t.relu, t.bias_n, nullptr, nullptr, t.relu_bits_out, ldm},
              t, st);
        return stream_table_c<OP, F32>(ao, bo, CRowSideH<true, false>{t.Ch, t.ldc, t.relu, t.bias_n, nullptr}, t, st);
      } else {
        if (t.relu_bits_in)
          return stream_table_c<OP, F32>(
              ao, bo, CRowSideH<false, true, 2>{t.Ch, t.ldc, t.relu, nullptr, nullptr, t.relu_bits_in, nullptr, ldm},
              t, st);
        if (t.out_mask_h)
          return stream_table_c<OP, F32>(ao, bo, CRowSideH<false, true>{t.Ch, t.ldc, t.relu, nullptr, t.out_mask_h},
                                         t, st);
        return stream_table_c<OP, F32>(ao, bo, CRowSideH<false, false>{t.Ch, t.ldc, t.relu, nullptr, nullptr}, t, st);
      }
    }
  }
  if constexpr (OP == kOpFoldFwd) {
    if (t.relu_bits_out)
      return stream_table_c<OP, F32>(
          ao, bo, CRowSide<true, false, 1>{t.C, t.ldc, t.relu, t.bias_n, nullptr, nullptr, t.relu_bits_out, ldm}, t,
          st);
    return stream_table_c<OP, F32>(ao, bo, CRowSide<true, false>{t.C, t.ldc, t.relu, t.bias_n, nullptr}, t, st);
  } else {
    if (t.relu_bits_in)
      return stream_table_c<OP, F32>(
          ao, bo, CRowSide<false, true, 2>{t.C, t.ldc, t.relu, nullptr, nullptr, t.relu_bits_in, nullptr, ldm}, t, st);
    if (t.out_mask)
      return stream_table_c<OP, F32>(ao, bo, CRowSide<false, true>{t.C, t.ldc, t.relu, nullptr, t.out_mask}, t, st);
    return stream_table_c<OP, F32>(ao, bo, CRowSide<false, false>{t.C, t.ldc, t.relu, nullptr, nullptr}, t, st);
  }
}

template <int OP, bool F32, class AO>
int stream_table_b(AO ao, const TableGemm &t, hipStream_t st) {
  if constexpr (F32) return stream_table<OP, true>(ao, SK3{t.B3, t.ldb_h, t.N, t.B3f, t.K}, t, st);
  else return stream_table<OP, false>(ao, SKh{t.Bh, t.ldb_h, t.N}, t, st);
}

template <int OP, bool F32>
int stream_table_op(const TableGemm &t, hipStream_t st) {
  if constexpr (!F32)
    if (t.Ah) return stream_table_b<OP, F32>(SKb{{t.Ah, t.lda, t.M}}, t, st);
  const bool vec = t.lda % 4 == 0 && t.K % 4 == 0 && aligned16(t.A);
  if (vec) return stream_table_b<OP, F32>(SKc<true>{t.A, t.lda, t.M}, t, st);
  return stream_table_b<OP, F32>(SKc<false>{t.A, t.lda, t.M}, t, st);
}

}  // namespace streaming

using namespace streaming;

// Full-stage DMA offsets are 32-bit: a tile's rows must span < 4 GiB.
constexpr int64_t kMaxStreamLd = int64_t(1) << 22;

bool stream_table_ok(const TableGemm &t, dlm_precision prec) {
  if (t.groups != 1 || t.mask != nullptr || (t.op != kOpFoldFwd && t.op != kOpFoldBwdData)) return false;
  if (t.relu_bits_out || t.relu_bits_in) {  // ReLU bits: one word per 16 columns
    if (t.N % 16 != 0) return false;
    if (t.relu_bits_out && (t.op != kOpFoldFwd || !t.relu)) return false;
    if (t.relu_bits_in && (t.op != kOpFoldBwdData || t.out_mask || t.out_mask_h)) return false;
  }
  if (t.Ah || t.Ch || t.out_mask_h) {  // bfloat16 activations: BF16 only, 16-byte rows
    if (prec != DLM_BF16) return false;
    if (t.Ah && (t.A || t.lda % 8 != 0 || t.K % 8 != 0 || !aligned16(t.Ah))) return false;
    if (t.Ch && (t.C || t.ldc % 8 != 0 || !aligned16(t.Ch))) return false;
    if (t.out_mask_h && (!t.Ch || t.out_mask || !aligned16(t.out_mask_h))) return false;
  }
  if (t.lda >= kMaxStreamLd || t.ldb_f >= kMaxStreamLd || t.ldb_h >= kMaxStreamLd) return false;
  if (t.op == kOpFoldFwd ? (t.bias_n == nullptr || t.out_mask != nullptr) : t.bias_n != nullptr) return false;
  const uint16_t *B = prec == DLM_BF16 ? t.Bh : t.B3;
  if (prec != DLM_BF16 && !t.B3f) return false;
  return B != nullptr && t.ldb_h > 0 && t.ldb_h % SBK == 0 && t.ldb_h >= t.K && aligned16(B);
}

int launch_stream_table(const TableGemm &t, dlm_precision prec, void *stream) {
  if (!stream_table_ok(t, prec)) return -3;
  hipStream_t st = (hipStream_t)stream;
  const bool f32 = prec != DLM_BF16;
  switch (t.op) {
    case kOpFoldFwd: return f32 ? stream_table_op<kOpFoldFwd, true>(t, st) : stream_table_op<kOpFoldFwd, false>(t, st);
    case kOpFoldBwdData:
      return f32 ? stream_table_op<kOpFoldBwdData, true>(t, st) : stream_table_op<kOpFoldBwdData, false>(t, st);
    default: return -3;
  }
}

}  // namespace dlm
