// Register-staged matrix-core GEMM for operands that a kernel has to change
// on the way into LDS: split into parts (FP32, parts.h) or rounded to
// bfloat16, masked by a ReLU, transposed, or given a row of ones.
//
//   C[r][n] = sum_k A(r, k) B(n, k)
//
// It runs the weight gradients of the folded LSC layer (both operands
// contiguous along their rows, reduced over voxels).
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
// banks (with k = 8 g .. + 7, the instruction's own order, two lane groups met
// in the same banks).  Contiguous along k (rows of 32): two 8-byte reads of
// the same k per lane.
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

// Eight k (4 g4 .., 16 + 4 g4 ..) of row 16 rg + q16 from k-lines.
template <int BR>
__device__ __forceinline__ bf16x8 frag_lines(const uint16_t *t, int rg, int q16, int g4) {
  bf16x8 r{};
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __attribute__((address_space(3))) s16x4 *lp;
  const uint16_t *p = t + (4 * g4 + (q16 >> 2)) * line(BR) + 16 * rg + 4 * (q16 & 3);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + 16 * line(BR)));
  r = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#endif
  return r;
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
// its place in a stage (loop-invariant, in entries), whole(k0, kend): whether
// a stage's runs can be loaded without a look at any bound, load() for such a
// stage and load_edge() for the others (zeros at and beyond kend), store() to
// LDS and frag().  Runs of rows beyond the matrix load some valid entries;
// their results are never stored.  at(r, k) is the value itself.

// float32, contiguous along the rows: element (r, k) at p[k ld + r], r < rows,
// k < lines.  MASK: zero where mask (indexed as p) is not positive.  ONES: row
// `rows` is a row of ones.
template <int P, bool MASK, bool ONES>
struct Lines {
  const float *p, *mask;
  int64_t ld;
  int rows, lines;
  template <int BR>
  static constexpr int size() { return P * TBK * line(BR); }
  template <int BR>
  static constexpr int items() { return TBK * BR / 4; }
  struct Raw {
    floatx4 v, m;
  };
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
  __device__ void load(Raw &x, uint32_t o, int k0) const {
    const int64_t base = (int64_t)k0 * ld;
    x.v = ld4(p + base + o);
    if constexpr (MASK) x.m = ld4(mask + base + o);
  }
  template <int BR>
  __device__ void load_edge(Raw &x, int e, int64_t r0, int k0, int kend) const {
    const int k = k0 + k_of<BR>(e);
    const int64_t base = (int64_t)min(k, kend - 1) * ld, r = r0 + row_of<BR>(e);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t o = base + least(r + i, rows - 1);
      const float v = p[o];
      x.v[i] = k < kend ? v : 0.0f;
      if constexpr (MASK) x.m[i] = mask[o];
    }
  }
  // the run's distance to the ones row
  template <int BR>
  __device__ int ones_at(int e, int64_t r0) const { return (int)least(rows - r0 - row_of<BR>(e), 4); }
  template <int BR>
  __device__ void store(const Raw &x, int e, int one, bool valid, uint16_t *lds) const {
    floatx4 v = x.v;
    if constexpr (MASK)
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = x.m[i] > 0.0f ? v[i] : 0.0f;
    if constexpr (ONES)
      if (one >= 0 && one < 4)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = one == i ? (valid ? 1.0f : 0.0f) : v[i];
    put4<P>(lds + k_of<BR>(e) * line(BR) + row_of<BR>(e), TBK * line(BR), v);
  }
  template <int BR>
  __device__ static bf16x8 frag(const uint16_t *lds, int rg, int q16, int g4, int part) {
    return frag_lines<BR>(lds + part * TBK * line(BR), rg, q16, g4);
  }
  __device__ float at(int64_t r, int k) const {
    if (r >= rows) return ONES && r == rows ? 1.0f : 0.0f;
    const int64_t o = (int64_t)k * ld + r;
    return MASK && !(mask[o] > 0.0f) ? 0.0f : p[o];
  }
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
  __device__ bool whole(int k0, int kend) const { return k0 + TBK <= kend; }
  __device__ void load(Raw &x, uint32_t o, int k0) const {
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
  __device__ void store(const Raw &x, int e, int one, bool valid, uint16_t *lds) const {
    u32x4 v = x.v;
    if constexpr (ONES)
      if (one == 0) v[0] = valid ? 0x3f80u : 0u;
    __builtin_memcpy(__builtin_assume_aligned(lds + k_of<BR>(e) * line(BR) + row_of<BR>(e), 16), &v, 16);
  }
  template <int BR>
  __device__ static bf16x8 frag(const uint16_t *lds, int rg, int q16, int g4, int) {
    return frag_lines<BR>(lds, rg, q16, g4);
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
  typename OPND::Raw raw[PER];
  uint32_t off[PER];
  int one[PER];
  int64_t r0;
  __device__ static int run(int i) {  // threads without an i-th run repeat the last one
    const int e = threadIdx.x + i * NT;
    return N % NT == 0 || e < N ? e : N - 1;
  }
  __device__ void init(const OPND &op, int64_t r0_) {
    r0 = r0_;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      off[i] = op.template off<BR>(run(i), r0);
      one[i] = op.template ones_at<BR>(run(i), r0);
    }
  }
  __device__ void load(const OPND &op, int k0, int kend) {
    if (op.whole(k0, kend)) {
#pragma unroll
      for (int i = 0; i < PER; ++i) op.load(raw[i], off[i], k0);
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        op.template load_edge<BR>(raw[i], run(i), r0, k0, kend);
        __builtin_amdgcn_sched_barrier(0);  // one run's registers at a time
      }
    }
  }
  __device__ void store(const OPND &op, int left, uint16_t *lds) {  // `left` k of the stage lie in the range
#pragma unroll
    for (int i = 0; i < PER; ++i)
      op.template store<BR>(raw[i], run(i), one[i], OPND::template k_of<BR>(run(i)) < left, lds);
  }
};

// SWAP: the A fragment first, so a lane holds four consecutive rows of one
// column (outputs stored along the rows) instead of four columns of a row.
template <int OP, class CF, int P, bool SWAP, class AO, class BO, class CS>
__global__ __launch_bounds__(64 * CF::NW, 2) void tile_kernel(AO ao, BO bo, CS cs, int64_t M, int N, int K,
                                                                    int ksplit, int nbM, int nbN, int nz) {
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
  const int kbeg = ksplit > 0 ? z * ksplit : 0, kend = ksplit > 0 ? min(K, kbeg + ksplit) : K;

  Stage<BM, NT, AO> xa;
  Stage<BN, NT, BO> xb;
  floatx4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  xa.init(ao, m0);
  xb.init(bo, n0);
  if (kbeg < kend) {
    xa.load(ao, kbeg, kend);
    xb.load(bo, kbeg, kend);
  }
  for (int k0 = kbeg; k0 < kend; k0 += TBK) {
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
      for (int p = 0; p < P; ++p) a[i][p] = AO::template frag<BM>(sa, wm * TM + i, q16, g4, p);
#pragma unroll
    for (int j = 0; j < TN; j += NJ) {
      bf16x8 b[NJ][P];
#pragma unroll
      for (int u = 0; u < NJ; ++u)
#pragma unroll
        for (int p = 0; p < P; ++p)
          if (j + u < TN) b[u][p] = BO::template frag<BN>(sb, wn * TN + j + u, q16, g4, p);
      if constexpr (P == 3) {
        mma_parts_sum<SWAP>(a, b, acc, j);
      } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(SWAP ? a[i][0] : b[0][0], SWAP ? b[0][0] : a[i][0],
                                                              acc[i][j], 0, 0, 0);
      }
    }
  }
  const int64_t ra = m0 + wm * TM * 16;
  const int rb = n0 + wn * TN * 16;
  if constexpr (P == 3)
    if (const uint64_t bad = bad_tiles(acc)) redo_tiles<SWAP>(ao, bo, ra, rb, kbeg, kend, bad, acc);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t r = ra + 16 * i + (SWAP ? 4 * g4 : q16);
      const int n = rb + 16 * j + (SWAP ? q16 : 4 * g4);
      if (r < M && n < N) cs.store(r, n, z, acc[i][j], (int)least(4, SWAP ? M - r : N - n));
    }
}

template <int OP, class CF, int P, bool SWAP, class AO, class BO, class CS>
int run(AO ao, BO bo, CS cs, int64_t M, int N, int K, int Z, int ksplit, hipStream_t st) {
  if (M <= 0 || N <= 0 || Z <= 0) return 0;
  const int64_t nbM = (M + CF::BM - 1) / CF::BM;
  const int nbN = (N + CF::BN - 1) / CF::BN;
  if (nbM * nbN * Z > 0x7fffffff) return -4;
  hipLaunchKernelGGL((tile_kernel<OP, CF, P, SWAP, AO, BO, CS>), dim3((unsigned)(nbM * nbN * Z)), dim3(64 * CF::NW), 0,
                     st, ao, bo, cs, M, N, K, ksplit, (int)nbM, nbN, Z);
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
  __device__ void store(int64_t r, int c, int s, floatx4 v, int cnt) const {
    float *o = part + ((int64_t)s * M + (SWAP ? c : r)) * N1 + (SWAP ? r : c);
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
// instructions 3.65 -> 2.73 ms at 1M voxels x 1440 x 136 (0.52 of the matrix
// cores' cycles; the same core with part products 4.3 ms), 632 -> 454 us for
// 8192 x 2880 x 1441; BF16 1.10 -> 0.96 ms (3.7 TB/s) and, 8192 x 2881 x 2880
// from bfloat16, 294 -> 221 us.
using GradCfg = Cfg<128, 144, 4, 1>;

template <int P, class GO, class AO>
int grad(GO go, AO ao, const GradGemm &x, int ks, hipStream_t st) {
  const int N1 = x.CK + 1;
  if (x.M >= N1)
    return run<kOpFoldGrad, GradCfg, P, false>(go, ao, CPart<false>{x.partial, x.M, N1}, x.M, N1, (int)x.V, x.splits, ks,
                                               st);
  return run<kOpFoldGrad, GradCfg, P, true>(ao, go, CPart<true>{x.partial, x.M, N1}, N1, x.M, (int)x.V, x.splits, ks, st);
}

template <int P, class GO>
int grad_act(GO go, const GradGemm &x, int ks, hipStream_t st) {
  const int V = (int)x.V;
  if constexpr (P == 1)
    if (x.ah) return grad<P>(go, LinesH<true>{x.ah, x.CK, x.CK, V}, x, ks, st);
  return grad<P>(go, Lines<P, false, true>{x.a, nullptr, x.CK, x.CK, V}, x, ks, st);
}

template <int P>
int grad_parts(const GradGemm &x, int ks, hipStream_t st) {
  const int V = (int)x.V;
  if constexpr (P == 1)
    if (x.gh) return grad_act<P>(LinesH<false>{x.gh, x.M, x.M, V}, x, ks, st);
  if (x.mask) return grad_act<P>(Lines<P, true, false>{x.g, x.mask, x.M, x.M, V}, x, ks, st);
  return grad_act<P>(Lines<P, false, false>{x.g, nullptr, x.M, x.M, V}, x, ks, st);
}

}  // namespace tile

// Voxel slices: blocks for three rounds of the chip (two blocks per compute
// unit) while a slice keeps 512 voxels; wide layers, whose partial matrices
// are large (33 MB for 2880 x 2881), one round.
int fold_grad_splits(int64_t V, int M, int N1) {
  using tile::GradCfg;
  const int big = std::max(M, N1), small = std::min(M, N1);
  const int tiles = (big + GradCfg::BM - 1) / GradCfg::BM * ((small + GradCfg::BN - 1) / GradCfg::BN);
  int s = (int)std::min<int64_t>(128, std::max(1, (tiles <= 128 ? 1536 : 512) / tiles));
  s = (int)std::min<int64_t>(s, std::max<int64_t>(1, V / 512));
  while (s > 1 && (V + tile::split_len(V, s) - 1) / tile::split_len(V, s) != s) --s;
  return s;
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
