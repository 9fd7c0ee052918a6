// Register-staged matrix-core GEMM for operands that a kernel has to change
// on the way into LDS: split into parts (FP32, parts.h) or rounded to
// bfloat16, masked by a ReLU, transposed, or given a row of ones.
//
//   C[r][n] = sum_k A(r, k) B(n, k)
//
// It runs the weight gradients of the folded LSC layer (both operands
// contiguous along their rows, reduced over voxels) and every GEMM of the
// folded layer on images (subjects x channels x voxels), which it reads and
// writes as they are: the forward and the input gradient with the activations
// contiguous along the voxels, their rows, and the weight gradient with both
// operands contiguous along the voxels, the reduction.
//
// A thread moves 16-byte runs from global memory into registers (dword
// alignment suffices on gfx950), one stage of 32 k ahead; after the barrier
// that ends the last stage's reads it masks and splits or rounds them once
// for the whole block and writes bfloat16 to LDS.  Doing that here, and not
// as each wave reads its fragments, is what makes the part products pay: a
// wave's fragments of a 128 x 144 tile cost it 1936 vector cycles to split
// against 1728 of its matrix instructions, its share of the block's runs 750.
//
// LDS holds each operand as it lies in memory.  Contiguous along the rows
// (k-lines of BR entries): a fragment, eight k of one row per lane, is read
// with two transposing reads (ds_read_b64_tr_b16: 16 lanes read four k-lines
// of 16 rows and each receives one row's four k).  The k-lines are 16 or 48
// entries beyond a multiple of 64 apart, so four of them lie in different
// banks, and lane group g takes k = 4 g .. + 3 and 16 + 4 g .. + 3, so the
// eight lines that half a wave reads at once are neighbours and cover all
// banks.  Where the sum has to be that of the other cores bit for bit (BF16
// forwards: the next layer rounds the result), lane group g takes k = 8 g ..
// + 7 and every eight lines are followed by 64 entries, so that lines 8 apart
// do not meet in the same banks.  Contiguous along k (rows of 32): one 16-byte
// read per lane from rows 40 entries apart, which spreads eight rows over all
// banks.
// One buffer of LDS and two barriers per stage: with 55 KB (FP32) or 18 KB
// (BF16) two or more blocks of a compute unit fill each other's gaps.  (Two
// buffers with the next stage converted between the matrix instructions left
// FP32 one block per compute unit, and one wave's instructions do not overlap
// that well: 2.9 -> 3.9 ms on the wide layers at 1M voxels.)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gemm_common.h"
#include "internal.h"
#include "parts.h"

namespace dlm {
namespace tile {

constexpr int TBK = 32;  // reduction entries per stage

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// LDS entries from one k-line of BR rows to the next.
constexpr int line(int BR) {
  const int m = BR % 64;
  return m <= 16 ? BR - m + 16 : m <= 48 ? BR - m + 48 : BR - m + 80;
}
__device__ __forceinline__ int64_t least(int64_t a, int64_t b) { return a < b ? a : b; }
constexpr int kRowLd = TBK + 8;  // entries from one row of 32 k to the next

// LDS entry of k-line k (ORD: in the order k = 8 g4 .. of a fragment).
template <int BR, bool ORD>
constexpr int line_at(int k) {
  return k * line(BR) + (ORD ? (k >> 3) * 64 : 0);
}

// Eight k (4 g4 .., 16 + 4 g4 ..; ORD: 8 g4 ..) of row 16 rg + q16.
template <int BR, bool ORD>
__device__ __forceinline__ bf16x8 frag_lines(const uint16_t *t, int rg, int q16, int g4) {
  bf16x8 r{};
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __attribute__((address_space(3))) s16x4 *lp;
  const int k = (ORD ? 8 : 4) * g4 + (q16 >> 2);
  const uint16_t *p = t + line_at<BR, ORD>(k) + 16 * rg + 4 * (q16 & 3);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + (ORD ? 4 : 16) * line(BR)));
  r = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#endif
  return r;
}

// Four values zeroed where their bit of `nib` is clear.
__device__ __forceinline__ floatx4 keep4(floatx4 v, unsigned nib) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = (nib >> i) & 1u ? v[i] : 0.0f;
  return v;
}

// Four floats as P bfloat16 parts, 8 bytes each, to LDS `part` entries apart.
template <int P>
__device__ __forceinline__ void put4(uint16_t *d, int part, floatx4 v) {
  float x = v[0], y = v[1], u = v[2], w = v[3];
#pragma unroll
  for (int i = 0; i < P; ++i) {
    uint32_t h[2];
    if (i + 1 < P) {
      h[0] = part2<true>(x, y);
      h[1] = part2<true>(u, w);
    } else {
      h[0] = part2<false>(x, y);
      h[1] = part2<false>(u, w);
    }
    __builtin_memcpy(__builtin_assume_aligned(d + i * part, 8), h, 8);
  }
}

// ---------------------------------------------------------------- operands
// Each gives, for a tile of BR rows: size() of its LDS in entries, items()
// runs per stage, Raw (one run in registers), row_of / k_of of run e, off()
// its place relative to base(r0, k0) (the same in every stage, in entries),
// whole(k0, kend): whether a stage's runs can be loaded without a look at any
// bound, load() for such a stage and load_edge() for the others (zeros at and
// beyond kend), store() to LDS and frag(), run_lines() of NT threads: the k-lines
// from one run of a thread to its next where they lie at the same rows, else 0.  Runs of rows beyond the matrix
// load some valid entries; their results are never stored.  batch(b) moves to
// image b.  lane() and at() are the slow path's reads (parts.h).

// What zeroes an operand: nothing, a float32 array of the operand's own layout
// (zero where it is not positive) or ReLU bits along its contiguous index.
enum Mask : int { kNoMask = 0, kFloatMask, kBitMask };

// float32, contiguous along the rows: element (r, k) at p[k ld + r], r < rows,
// k < lines.  Bits: bit r % 16 of word bits[k lb + r / 16].  ONES: row `rows`
// is a row of ones.
template <int P, int MASK, bool ONES, bool ORD = false>
struct Lines {
  const float *p, *mask;
  int64_t ld;
  int rows, lines;
  int64_t bs = 0;
  const uint16_t *bits = nullptr;
  int64_t lb = 0, bbs = 0;
  template <int BR>
  static constexpr int part() { return line_at<BR, ORD>(TBK); }
  template <int BR>
  static constexpr int size() { return P * part<BR>(); }
  template <int BR>
  static constexpr int items() { return TBK * BR / 4; }
  template <int BR, int NT>
  static constexpr int run_lines() {
    // (the BF16 images' small tiles keep a wave more per SIMD without)
    return (!ORD || P == 3) && NT % (BR / 4) == 0 && items<BR>() % NT == 0 ? NT / (BR / 4) : 0;
  }
  struct Raw {
    floatx4 v, m;
    uint16_t w;
  };
  __device__ void batch(int b) {
    p += b * bs;
    if constexpr (MASK == kBitMask) bits += b * bbs;
  }
  template <int BR>
  __device__ static int row_of(int e) { return 4 * (e % (BR / 4)); }
  template <int BR>
  __device__ static int k_of(int e) { return e / (BR / 4); }
  template <int BR>
  __device__ uint32_t off(int e, int64_t r0) const {
    return (uint32_t)(k_of<BR>(e) * ld + least(r0 + row_of<BR>(e), rows - 1));
  }
  // a run of the last line but one ends inside the last line (ld >= 4)
  __device__ bool whole(int k0, int kend) const { return ld >= 4 && k0 + TBK <= least(kend, lines - 1); }
  template <int BR>
  __device__ void load(Raw &x, int e, uint32_t o, int64_t r0, int k0) const {
    const int64_t base = (int64_t)k0 * ld;
    x.v = ld4(p + base + o);
    if constexpr (MASK == kFloatMask) x.m = ld4(mask + base + o);
    if constexpr (MASK == kBitMask) load_bits<BR>(x, e, r0, k0 + k_of<BR>(e));
  }
  template <int BR>
  __device__ void load_bits(Raw &x, int e, int64_t r0, int k) const {
    const int64_t r = least(r0 + row_of<BR>(e), rows - 1);
    x.w = bits[k * lb + (r >> 4)] >> (r & 12);
  }
  template <int BR>
  __device__ void load_edge(Raw &x, int e, int64_t r0, int k0, int kend) const {
    const int k = k0 + k_of<BR>(e);
    const int64_t base = least(k, kend - 1) * ld, r = r0 + row_of<BR>(e);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t o = base + least(r + i, rows - 1);
      const float v = p[o];
      x.v[i] = k < kend ? v : 0.0f;
      if constexpr (MASK == kFloatMask) x.m[i] = mask[o];
    }
    if constexpr (MASK == kBitMask) load_bits<BR>(x, e, r0, (int)least(k, kend - 1));
  }
  // the run's distance to the ones row
  template <int BR>
  __device__ int ones_at(int e, int64_t r0) const { return (int)least(rows - r0 - row_of<BR>(e), 4); }
  template <int BR>
  __device__ void store(const Raw &x, int e, int one, int left, uint16_t *lds) const {
    floatx4 v = x.v;
    if constexpr (MASK == kFloatMask)
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = x.m[i] > 0.0f ? v[i] : 0.0f;
    if constexpr (MASK == kBitMask) v = keep4(v, x.w);
    if constexpr (ONES)
      if (one >= 0 && one < 4)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = one == i ? (k_of<BR>(e) < left ? 1.0f : 0.0f) : v[i];
    put4<P>(lds + line_at<BR, ORD>(k_of<BR>(e)) + row_of<BR>(e), part<BR>(), v);
  }
  template <int BR>
  __device__ static bf16x8 frag(const uint16_t *lds, int rg, int q16, int g4, int i) {
    return frag_lines<BR, ORD>(lds + i * part<BR>(), rg, q16, g4);
  }
  struct Lane {
    uint32_t off, boff;
    int shift, one;  // one: 0 for the ones row, -1 beyond the matrix
  };
  __device__ Lane lane(int64_t r, int q16, int g) const {
    const int64_t c = least(r + q16, rows - 1);
    return Lane{(uint32_t)(g * ld + c), (uint32_t)(g * lb + (c >> 4)), int(c & 15),
                r + q16 < rows ? 1 : ONES && r + q16 == rows ? 0 : -1};
  }
  __device__ float at(int k, const Lane &l) const {
    float v = (p + (int64_t)k * ld)[l.off];
    if constexpr (MASK == kFloatMask) v = (mask + (int64_t)k * ld)[l.off] > 0.0f ? v : 0.0f;
    if constexpr (MASK == kBitMask) v = (bits + (int64_t)k * lb)[l.boff] >> l.shift & 1 ? v : 0.0f;
    return l.one > 0 ? v : l.one == 0 ? 1.0f : 0.0f;
  }
};

// float32, contiguous along k: element (r, k) at p[r ld + k], r < rows.  Bits:
// bit k % 16 of word bits[r lb + k / 16].
template <int P, int MASK, bool ONES>
struct Rows {
  const float *p;
  int64_t ld;
  int rows;
  int64_t bs = 0;
  const uint16_t *bits = nullptr;
  int64_t lb = 0, bbs = 0;
  static_assert(MASK != kFloatMask, "bits or nothing");
  template <int BR>
  static constexpr int size() { return P * BR * kRowLd; }
  template <int BR>
  static constexpr int items() { return BR * TBK / 4; }
  template <int BR, int NT>
  static constexpr int run_lines() { return 0; }
  struct Raw {
    floatx4 v;
    uint16_t w;
  };
  __device__ void batch(int b) {
    p += b * bs;
    if constexpr (MASK == kBitMask) bits += b * bbs;
  }
  template <int BR>
  __device__ static int row_of(int e) { return e / (TBK / 4); }
  template <int BR>
  __device__ static int k_of(int e) { return 4 * (e % (TBK / 4)); }
  __device__ int64_t base(int64_t r0) const { return least(r0, rows - 1); }
  template <int BR>
  __device__ uint32_t off(int e, int64_t r0) const {
    return (uint32_t)((least(r0 + row_of<BR>(e), rows - 1) - base(r0)) * ld + k_of<BR>(e));
  }
  __device__ bool whole(int k0, int kend) const { return k0 + TBK <= kend; }
  template <int BR>
  __device__ void load_bits(Raw &x, int e, int64_t r0, int k) const {
    x.w = bits[least(r0 + row_of<BR>(e), rows - 1) * lb + (k >> 4)] >> (k & 12);
  }
  template <int BR>
  __device__ void load(Raw &x, int e, uint32_t o, int64_t r0, int k0) const {
    x.v = ld4(p + base(r0) * ld + k0 + o);
    if constexpr (MASK == kBitMask) load_bits<BR>(x, e, r0, k0 + k_of<BR>(e));
  }
  template <int BR>
  __device__ void load_edge(Raw &x, int e, int64_t r0, int k0, int kend) const {
    const int k = k0 + k_of<BR>(e);
    const float *row = p + least(r0 + row_of<BR>(e), rows - 1) * ld;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = row[least(k + i, kend - 1)];
      x.v[i] = k + i < kend ? v : 0.0f;
    }
    if constexpr (MASK == kBitMask) load_bits<BR>(x, e, r0, (int)least(k, kend - 1) & ~3);
  }
  template <int BR>
  __device__ int ones_at(int e, int64_t r0) const { return r0 + row_of<BR>(e) == rows ? 0 : 1; }
  template <int BR>
  __device__ void store(const Raw &x, int e, int one, int left, uint16_t *lds) const {
    floatx4 v = x.v;
    if constexpr (MASK == kBitMask) v = keep4(v, x.w);
    if constexpr (ONES)
      if (one == 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = k_of<BR>(e) + i < left ? 1.0f : 0.0f;
    put4<P>(lds + row_of<BR>(e) * kRowLd + k_of<BR>(e), BR * kRowLd, v);
  }
  template <int BR>
  __device__ static bf16x8 frag(const uint16_t *lds, int rg, int q16, int g4, int i) {
    return *reinterpret_cast<const bf16x8 *>(lds + i * BR * kRowLd + (rg * 16 + q16) * kRowLd + 8 * g4);
  }
  struct Lane {
    const float *first;  // of rows r .. r + 15, the same in all lanes
    const uint16_t *words;
    uint32_t off, boff;
    int g, one;
  };
  __device__ Lane lane(int64_t r, int q16, int g) const {
    const int64_t r0 = base(r), c = least(r + q16, rows - 1) - r0;
    return Lane{p + r0 * ld, bits + r0 * lb, (uint32_t)(c * ld + g), (uint32_t)(c * lb), g,
                r + q16 < rows ? 1 : ONES && r + q16 == rows ? 0 : -1};
  }
  __device__ float at(int k, const Lane &l) const {
    float v = (l.first + k)[l.off];
    if constexpr (MASK == kBitMask) v = (l.words + (k >> 4))[l.boff] >> ((k & 15) + l.g) & 1 ? v : 0.0f;
    return l.one > 0 ? v : l.one == 0 ? 1.0f : 0.0f;
  }
};

// A folded table in P bfloat16 parts: part i of (r, k) at p[r P ld + i ld + k],
// zeros from K to ld (a multiple of 32); one table for every image.  P == 3:
// the values themselves in f, rows of ldf.
template <int P>
struct Table {
  const uint16_t *p;
  int64_t ld;
  int rows;
  const float *f;
  int64_t ldf;
  template <int BR>
  static constexpr int size() { return P * BR * kRowLd; }
  template <int BR>
  static constexpr int items() { return P * BR * TBK / 8; }
  template <int BR, int NT>
  static constexpr int run_lines() { return 0; }
  struct Raw {
    u32x4 v;
  };
  __device__ void batch(int) {}
  template <int BR>
  __device__ static int row_of(int e) { return e % (BR * 4) / 4; }
  template <int BR>
  __device__ static int k_of(int e) { return 8 * (e % 4); }
  template <int BR>
  __device__ uint32_t off(int e, int64_t r0) const {
    return (uint32_t)((least(r0 + row_of<BR>(e), rows - 1) - r0) * P * ld + e / (BR * 4) * ld + k_of<BR>(e));
  }
  __device__ bool whole(int, int) const { return true; }
  template <int BR>
  __device__ void load(Raw &x, int, uint32_t o, int64_t r0, int k0) const {
    // not a memcpy: that kept the runs of some tiles in scratch memory, and a
    // wait for each load right behind it (1440 -> 135 channels, 32 768 voxels,
    // FP32 177 us; 106 in registers)
    x.v = *reinterpret_cast<const u32x4 *>(p + r0 * P * ld + k0 + o);
  }
  template <int BR>
  __device__ void load_edge(Raw &, int, int64_t, int, int) const {}
  template <int BR>
  __device__ int ones_at(int, int64_t) const { return 0; }
  template <int BR>
  __device__ void store(const Raw &x, int e, int, int, uint16_t *lds) const {
    uint16_t *d = lds + e / (BR * 4) * BR * kRowLd + row_of<BR>(e) * kRowLd + k_of<BR>(e);
    *reinterpret_cast<u32x4 *>(d) = x.v;
  }
  template <int BR>
  __device__ static bf16x8 frag(const uint16_t *lds, int rg, int q16, int g4, int i) {
    return *reinterpret_cast<const bf16x8 *>(lds + i * BR * kRowLd + (rg * 16 + q16) * kRowLd + 8 * g4);
  }
  struct Lane {
    const float *first;  // of rows r .. r + 15, the same in all lanes
    uint32_t off;
  };
  __device__ Lane lane(int64_t r, int q16, int g) const {
    const int64_t r0 = least(r, rows - 1);
    return Lane{f + r0 * ldf, (uint32_t)(least(q16, rows - 1 - r0) * ldf + g)};
  }
  __device__ float at(int k, const Lane &l) const { return (l.first + k)[l.off]; }
};

// bfloat16, contiguous along the rows (activations stored in bfloat16; ld and
// rows multiples of 8, 16-byte aligned): a run of eight rows lies wholly
// inside or wholly beyond the matrix.
template <bool ONES>
struct LinesH {
  const uint16_t *p;
  int64_t ld;
  int rows, lines;
  template <int BR>
  static constexpr int size() { return TBK * line(BR); }
  template <int BR>
  static constexpr int items() { return TBK * BR / 8; }
  template <int BR, int NT>
  static constexpr int run_lines() { return 0; }
  struct Raw {
    u32x4 v;
  };
  template <int BR>
  __device__ static int row_of(int e) { return 8 * (e % (BR / 8)); }
  template <int BR>
  __device__ static int k_of(int e) { return e / (BR / 8); }
  template <int BR>
  __device__ uint32_t off(int e, int64_t r0) const {
    return (uint32_t)(k_of<BR>(e) * ld + least(r0 + row_of<BR>(e), rows - 8));
  }
  __device__ void batch(int) {}
  __device__ bool whole(int k0, int kend) const { return k0 + TBK <= kend; }
  template <int BR>
  __device__ void load(Raw &x, int, uint32_t o, int64_t, int k0) const {
    __builtin_memcpy(&x.v, __builtin_assume_aligned(p + (int64_t)k0 * ld + o, 16), 16);
  }
  template <int BR>
  __device__ void load_edge(Raw &x, int e, int64_t r0, int k0, int kend) const {
    const int k = k0 + k_of<BR>(e);
    const int64_t o = (int64_t)min(k, kend - 1) * ld + least(r0 + row_of<BR>(e), rows - 8);
    u32x4 v;
    __builtin_memcpy(&v, __builtin_assume_aligned(p + o, 16), 16);
    x.v = k < kend ? v : u32x4{0u, 0u, 0u, 0u};
  }
  template <int BR>
  __device__ int ones_at(int e, int64_t r0) const { return (int)least(rows - r0 - row_of<BR>(e), 8); }
  template <int BR>
  __device__ void store(const Raw &x, int e, int one, int left, uint16_t *lds) const {
    u32x4 v = x.v;
    if constexpr (ONES)
      if (one == 0) v[0] = k_of<BR>(e) < left ? 0x3f80u : 0u;
    __builtin_memcpy(__builtin_assume_aligned(lds + k_of<BR>(e) * line(BR) + row_of<BR>(e), 16), &v, 16);
  }
  template <int BR>
  __device__ static bf16x8 frag(const uint16_t *lds, int rg, int q16, int g4, int) {
    return frag_lines<BR, false>(lds, rg, q16, g4);
  }
};

// ------------------------------------------------------------------ kernel
template <int BM_, int BN_, int WM_, int WN_>
struct Cfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NW = WM * WN;
  static constexpr int TM = BM / (WM * 16), TN = BN / (WN * 16);
  static_assert(TM * WM * 16 == BM && TN * WN * 16 == BN, "tile shape");
};

// One operand's runs of a stage in the block's registers.
template <int BR, int NT, class OPND>
struct Stage {
  static constexpr int N = OPND::template items<BR>(), PER = (N + NT - 1) / NT;
  // A thread's runs lie at one place of lines kLines apart: one offset for all.
  // (Kept one by one, the FP32 weight gradients had some of them in scratch
  // memory, and a wait for it between the loads of a stage: 1M voxels x 136 x
  // 1440 2.96 -> 2.89 ms, to 3.03 with the check for values below 2^-80.)
  static constexpr int kLines = OPND::template run_lines<BR, NT>(), NOFF = kLines ? 1 : PER;
  typename OPND::Raw raw[PER];
  uint32_t off[NOFF];
  int one[NOFF];
  int64_t r0;
  __device__ static int run(int i) {  // threads without an i-th run repeat the last one
    const int e = threadIdx.x + i * NT;
    return N % NT == 0 || e < N ? e : N - 1;
  }
  __device__ void init(const OPND &op, int64_t r0_) {
    r0 = r0_;
#pragma unroll
    for (int i = 0; i < NOFF; ++i) {
      off[i] = op.template off<BR>(run(i), r0);
      one[i] = op.template ones_at<BR>(run(i), r0);
    }
  }
  __device__ __forceinline__ void load(const OPND &op, int k0, int kend) {
    if (op.whole(k0, kend)) {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int j = kLines ? 0 : i;
        op.template load<BR>(raw[i], run(j), off[j], r0, k0 + i * kLines);
      }
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        op.template load_edge<BR>(raw[i], run(i), r0, k0, kend);
        __builtin_amdgcn_sched_barrier(0);  // one run's registers at a time
      }
    }
  }
  __device__ __forceinline__ void store(const OPND &op, int left, uint16_t *lds) const {  // `left` k of the stage lie in the range
#pragma unroll
    for (int i = 0; i < PER; ++i)
      op.template store<BR>(raw[i], run(i), one[kLines ? 0 : i], left, lds);
  }
};

// SWAP: the A fragment first, so a lane holds four consecutive rows of one
// column (outputs stored along the rows) instead of four columns of a row.
// z runs over images and, with ksplit > 0, over nsl slices of each.
template <int OP, class CF, int P, bool SWAP, class AO, class BO, class CS>
__global__ __launch_bounds__(64 * CF::NW, 2) void tile_kernel(AO ao, BO bo, CS cs, int64_t M, int N, int K, int ksplit,
                                                              int nsl, int nbM, int nbN, int nz) {
  constexpr int BM = CF::BM, BN = CF::BN, TM = CF::TM, TN = CF::TN, NT = 64 * CF::NW;
  constexpr int SA = AO::template size<BM>(), SB = BO::template size<BN>();
  static_assert(SA % 8 == 0 && SB % 8 == 0, "16-byte aligned tiles");
  __shared__ __attribute__((aligned(16))) uint16_t sa[SA], sb[SB];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % CF::WM, wn = wave / CF::WM;
  const int q16 = lane & 15, g4 = lane >> 4;
  const TileMap tm(blockIdx.x, nbM, nbN, nz, ksplit > 0);
  const int64_t m0 = (int64_t)tm.mt * BM;
  const int n0 = tm.nt * BN, z = tm.z;
  const int image = z / nsl;
  const int kbeg = (z - image * nsl) * ksplit, kend = ksplit > 0 ? min(K, kbeg + ksplit) : K;
  ao.batch(image);
  bo.batch(image);

  Stage<BM, NT, AO> xa;
  Stage<BN, NT, BO> xb;
  xa.init(ao, m0);
  xb.init(bo, n0);
  floatx4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (kbeg < kend) {
    xa.load(ao, kbeg, kend);
    xb.load(bo, kbeg, kend);
  }
  unsigned flip = 0;
  for (int k0 = kbeg; k0 < kend; k0 += TBK, flip ^= 0x80008000u) {
    __syncthreads();  // the last stage's fragments have been read
    xa.store(ao, kend - k0, sa);
    xb.store(bo, kend - k0, sb);
    __syncthreads();
    if (k0 + TBK < kend) {
      xa.load(ao, k0 + TBK, kend);
      xb.load(bo, k0 + TBK, kend);
    }
    constexpr int NJ = P == 3 ? 2 : 1;  // B tiles at a time
    bf16x8 a[TM][P];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int p = 0; p < P; ++p) {
        a[i][p] = AO::template frag<BM>(sa, wm * TM + i, q16, g4, p);
        if constexpr (P == 3) a[i][p] = flip_sign(a[i][p], flip);
      }
#pragma unroll
    for (int j = 0; j < TN; j += NJ) {
      bf16x8 b[NJ][P];
#pragma unroll
      for (int u = 0; u < NJ; ++u)
#pragma unroll
        for (int p = 0; p < P; ++p)
          if (j + u < TN) b[u][p] = BO::template frag<BN>(sb, wn * TN + j + u, q16, g4, p);
      if constexpr (P == 3) {
        mma_parts_sum<SWAP>(a, b, acc, j, flip ? -1.0f : 1.0f);
      } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(SWAP ? a[i][0] : b[0][0], SWAP ? b[0][0] : a[i][0],
                                                              acc[i][j], 0, 0, 0);
      }
    }
  }
  const int64_t row0 = m0 + wm * TM * 16;
  const int col0 = n0 + wn * TN * 16;
  if constexpr (P == 3)
    if (any_odd(acc))
      mend_odd<SWAP>(ao, bo, row0, col0, M, N, kbeg, kend, acc,
                     [&](int, int64_t r, unsigned want) { return nan_rows(ao, r, kbeg, kend, want); });
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int64_t r = row0 + 16 * i + (SWAP ? 4 * g4 : q16);
      const int n = col0 + 16 * j + (SWAP ? q16 : 4 * g4);
      cs.store(r, n, z, acc[i][j], r < M && n < N ? (int)least(4, SWAP ? M - r : N - n) : 0);
    }
}

template <int OP, class CF, int P, bool SWAP, class AO, class BO, class CS>
int run(AO ao, BO bo, CS cs, int64_t M, int N, int K, int Z, int ksplit, int nsl, hipStream_t st) {
  if (M <= 0 || N <= 0 || Z <= 0) return 0;
  const int64_t nbM = (M + CF::BM - 1) / CF::BM;
  const int nbN = (N + CF::BN - 1) / CF::BN;
  if (nbM * nbN * Z > 0x7fffffff) return -4;
  hipLaunchKernelGGL((tile_kernel<OP, CF, P, SWAP, AO, BO, CS>), dim3((unsigned)(nbM * nbN * Z)), dim3(64 * CF::NW), 0,
                     st, ao, bo, cs, M, N, K, ksplit, nsl, (int)nbM, nbN, Z);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// -------------------------------------------------------- weight gradients
int split_len(int64_t K, int splits) {
  const int64_t ks = (K + splits - 1) / splits;
  return (int)((ks + TBK - 1) / TBK * TBK);
}

// Partial matrices of slice s: part[s][m][n], n < N1.  The run of `cnt`
// (up to 4) values is along n; SWAP kernels have n on their row side.
template <bool SWAP>
struct CPart {
  float *part;
  int M, N1;
  __device__ __forceinline__ void store(int64_t r, int c, int s, floatx4 v, int cnt) const {
    float *o = part + ((int64_t)s * M + (SWAP ? c : r)) * N1 + (SWAP ? r : c);
    if (cnt == 0) return;
    if (cnt == 4) {
      __builtin_memcpy(o, &v, 16);
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i)
        if (i < cnt) o[i] = v[i];
    }
  }
};

// 144 columns: the narrow layers' 135 or 136 fit one tile, so the wide operand
// is read once.  The larger side is on the rows.
// Measured against the streaming core, which read eight k one by one for a
// fragment and split or rounded them in every wave: FP32 with float32
// instructions 3.65 -> 2.8 ms at 1M voxels x 1440 x 136 (half of the matrix
// cores' cycles, 2.7 before every other stage was negated; the same core with
// part products 4.3 ms), 632 -> 454 us for 8192 x 2880 x 1441; BF16 1.10 ->
// 0.96 ms (3.7 TB/s) and, 8192 x 2881 x 2880 from bfloat16, 294 -> 221 us.
using GradCfg = Cfg<128, 144, 4, 1>;

template <int P, class GO, class AO>
int grad(GO go, AO ao, const GradGemm &x, int ks, hipStream_t st) {
  const int N1 = x.CK + 1;
  if (x.M >= N1)
    return run<kOpFoldGrad, GradCfg, P, false>(go, ao, CPart<false>{x.partial, x.M, N1}, x.M, N1, (int)x.V, x.splits, ks,
                                               x.splits, st);
  return run<kOpFoldGrad, GradCfg, P, true>(ao, go, CPart<true>{x.partial, x.M, N1}, N1, x.M, (int)x.V, x.splits, ks,
                                            x.splits, st);
}

template <int P, class GO>
int grad_act(GO go, const GradGemm &x, int ks, hipStream_t st) {
  const int V = (int)x.V;
  if constexpr (P == 1)
    if (x.ah) return grad<P>(go, LinesH<true>{x.ah, x.CK, x.CK, V}, x, ks, st);
  return grad<P>(go, Lines<P, kNoMask, true>{x.a, nullptr, x.CK, x.CK, V}, x, ks, st);
}

template <int P>
int grad_parts(const GradGemm &x, int ks, hipStream_t st) {
  const int V = (int)x.V;
  if constexpr (P == 1)
    if (x.gh) return grad_act<P>(LinesH<false>{x.gh, x.M, x.M, V}, x, ks, st);
  if (x.mask) return grad_act<P>(Lines<P, kFloatMask, false>{x.g, x.mask, x.M, x.M, V}, x, ks, st);
  return grad_act<P>(Lines<P, kNoMask, false>{x.g, nullptr, x.M, x.M, V}, x, ks, st);
}

// ------------------------------------------------------------------ images
// Output of an image GEMM: rows are voxels, columns channels; element (r, c)
// of image z at C[z bs + c ld + r] = acc + bias[c], optional ReLU, and with
// `bits` the bit (stored value > 0) of it.
struct CImage {
  float *C;
  int64_t ld, bs;
  const float *bias;
  int relu;
  uint16_t *bits;
  int64_t lb, bbs;
  __device__ __forceinline__ void store(int64_t r, int c, int z, floatx4 v, int cnt) const {
    if (cnt > 0) {
      const float b = bias ? bias[c] : 0.0f;
      float *o = C + z * bs + c * ld + r;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (bias) v[i] += b;
        if (relu) v[i] = fmaxf(v[i], 0.0f);
      }
      if (cnt == 4) {
        __builtin_memcpy(o, &v, 16);
      } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
          if (i < cnt) o[i] = v[i];
      }
    }
    if (bits) {  // uniform: every lane takes part in the swaps
      unsigned nib = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) nib |= (i < cnt && v[i] > 0.0f ? 1u : 0u) << i;
      const int g4 = (threadIdx.x & 63) >> 4;
      const unsigned w = bits_word(nib, g4);
      if (cnt > 0 && g4 == 0) bits[z * bbs + c * lb + (r >> 4)] = (uint16_t)w;
    }
  }
};

// Tiles.  Measured on 121360 voxels (BF16) and 32768 (FP32), 135 -> 1440 and
// 1440 -> 135 channels, us, when the rule below was laid: BF16 128 x 96 with
// eight waves 391 and 297 (128 x 144 with four 527 and 342, 256 x 144 498 and
// 290, 64 x 48 462 and 327): its small accumulators leave room for the most
// waves.  FP32 256 x 144 with eight waves 179 and 201 (128 x 144 228 and 179,
// 128 x 48 242 and 178): the part products want the larger tile once it fills
// the chip.  Since then the table's runs of the other tiles have left scratch
// memory; with the fold, 256 x 144 now takes 159 and 156 in FP32, 128 x 144 147
// and 122, 128 x 48 171 and 111, 64 x 48 185 and 129; BF16 128 x 96 385 and 216,
// 256 x 144 366 and 191, 128 x 144 349 and 204.
template <int OP, int P, class AO>
int image_table(AO ao, const ImageGemm &x, hipStream_t st) {
  const Table<P> tab{x.table, x.ldb, x.N, x.values, x.K};
  const int64_t words = (x.P + 15) / 16;
  const CImage cs{x.out, x.P, x.P * x.N, x.bias, x.relu, x.obits, words, words * x.N};
  const int64_t b64 = (x.P + 63) / 64 * x.B, b128 = (x.P + 127) / 128 * x.B, b256 = (x.P + 255) / 256 * x.B;
  auto go = [&](auto cfg) { return run<OP, decltype(cfg), P, true>(ao, tab, cs, x.P, x.N, x.K, x.B, 0, 1, st); };
  // few blocks: the smallest tile
  if (b64 * ((x.N + 47) / 48) < 1024) return go(Cfg<64, 48, 4, 1>{});
  if (P == 1 && x.N > 48) return go(Cfg<128, 96, 4, 2>{});
  if (P == 3 && b256 * ((x.N + 143) / 144) >= 512) return go(Cfg<256, 144, 8, 1>{});
  return b128 * ((x.N + 47) / 48) < 512 ? go(Cfg<64, 48, 4, 1>{}) : go(Cfg<128, 48, 4, 1>{});
}

template <int P>
int image_gemm(const ImageGemm &x, hipStream_t st) {
  const int64_t words = (x.P + 15) / 16;
  if (x.op == kOpFoldFwd)
    return image_table<kOpFoldFwd, P>(Lines<P, kNoMask, false, true>{x.in, nullptr, x.P, (int)x.P, x.K, x.P * x.K}, x,
                                      st);
  if (x.ibits)
    return image_table<kOpFoldBwdData, P>(
        Lines<P, kBitMask, false, true>{x.in, nullptr, x.P, (int)x.P, x.K, x.P * x.K, x.ibits, words, words * x.K}, x,
        st);
  return image_table<kOpFoldBwdData, P>(Lines<P, kNoMask, false, true>{x.in, nullptr, x.P, (int)x.P, x.K, x.P * x.K}, x,
                                        st);
}

template <int P, int MASK>
int image_grad(const ImageGrad &x, int ks, hipStream_t st) {
  const int64_t words = (x.P + 15) / 16;
  const int N1 = x.CK + 1, nz = x.B * x.slices;
  const Rows<P, MASK, false> g{x.g, x.P, x.M, x.P * x.M, x.gbits, words, words * x.M};
  const Rows<P, kNoMask, true> a{x.a, x.P, x.CK, x.P * x.CK};
  if (x.M >= N1)
    return run<kOpFoldGrad, GradCfg, P, false>(g, a, CPart<false>{x.partial, x.M, N1}, x.M, N1, (int)x.P, nz, ks,
                                               x.slices, st);
  return run<kOpFoldGrad, GradCfg, P, true>(a, g, CPart<true>{x.partial, x.M, N1}, N1, x.M, (int)x.P, nz, ks, x.slices,
                                            st);
}

}  // namespace tile

// Voxel slices: blocks for three rounds of the chip (two blocks per compute
// unit) while a slice keeps 512 voxels; wide layers, whose partial matrices
// are large (33 MB for 2880 x 2881), one round.  Batches that leave compute
// units without a block at that take slices down to 128 voxels (both gradients
// of 8 -> 16 channels, order 6, 2000 voxels, masked, FP32: 108 us with three
// slices, 58 so; float32 instructions on small tiles 81).
static int grad_slices(int64_t V, int M, int N1, int most, int target_divisor) {
  using tile::GradCfg;
  const int big = std::max(M, N1), small = std::min(M, N1);
  const int tiles = (big + GradCfg::BM - 1) / GradCfg::BM * ((small + GradCfg::BN - 1) / GradCfg::BN);
  int s = (int)std::min<int64_t>(most, std::max(1, (tiles <= 128 ? 1536 : 512) / (tiles * target_divisor)));
  s = (int)std::min<int64_t>(s, std::max({int64_t(1), V / 512, std::min<int64_t>(V / 128, 256 / tiles)}));
  while (s > 1 && (V + tile::split_len(V, s) - 1) / tile::split_len(V, s) != s) --s;
  return s;
}

int fold_grad_splits(int64_t V, int M, int N1) { return grad_slices(V, M, N1, 128, 1); }

// Slices of each of B images, at most 128 in all (the workspace's partials).
int image_grad_slices(int B, int64_t P, int M, int N1) { return grad_slices(P, M, N1, std::max(1, 128 / B), B); }

// Offsets inside a tile are 32-bit: 143 rows or 31 k-lines of P entries.
bool image_ok(int64_t B, int64_t P) { return B >= 1 && B <= 128 && P >= 1 && P < (int64_t(1) << 24); }

int launch_image_gemm(const ImageGemm &x, dlm_precision prec, void *stream) {
  if (!image_ok(x.B, x.P) || !x.table || (reinterpret_cast<uintptr_t>(x.table) & 15) || x.ldb % 32 != 0) return -3;
  if (prec != DLM_BF16 && !x.values) return -3;
  hipStream_t st = (hipStream_t)stream;
  return prec == DLM_BF16 ? tile::image_gemm<1>(x, st) : tile::image_gemm<3>(x, st);
}

int launch_image_grad(const ImageGrad &x, dlm_precision prec, void *stream) {
  if (!image_ok(x.B, x.P)) return -3;
  const int ks = tile::split_len(x.P, x.slices);
  if ((x.P + ks - 1) / ks != x.slices || x.B * x.slices > 128) return -2;
  hipStream_t st = (hipStream_t)stream;
  using namespace tile;
  if (prec == DLM_BF16) return x.gbits ? image_grad<1, kBitMask>(x, ks, st) : image_grad<1, kNoMask>(x, ks, st);
  return x.gbits ? image_grad<3, kBitMask>(x, ks, st) : image_grad<3, kNoMask>(x, ks, st);
}

int launch_lsc_fold_grad(const GradGemm &x, dlm_precision prec, void *stream) {
  const int ks = tile::split_len(x.V, x.splits);
  if (x.V <= 0 || x.V > 0x7fffffff - ks || (x.V + ks - 1) / ks != x.splits) return -2;
  if ((x.gh || x.ah) && prec != DLM_BF16) return -3;
  if ((x.gh && (x.M % 8 != 0 || (reinterpret_cast<uintptr_t>(x.gh) & 15))) ||
      (x.ah && (x.CK % 8 != 0 || (reinterpret_cast<uintptr_t>(x.ah) & 15))))
    return -3;
  if (x.mask && x.gh) return -3;
  hipStream_t st = (hipStream_t)stream;
  return prec == DLM_BF16 ? tile::grad_parts<1>(x, ks, st) : tile::grad_parts<3>(x, ks, st);
}

}  // namespace dlm
