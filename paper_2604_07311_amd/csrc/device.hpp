// Device building blocks of the contraction kernels (gfx950 / CDNA4).
//
// Structure follows the paper's GEMM layering (the BLIS refactoring as loops
// around a micro-kernel with packed operands, Fig. "five loops around the
// micro-kernel"), re-cut for a GPU: the workgroup grid replaces the outer
// cache-blocking loops, the block-scatter gather into LDS replaces packing
// into contiguous panels (Approach, "Supporting tensor computations"), and
// wave-level MFMA tiles replace the register micro-kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "args.hpp"

namespace famlies {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = 256;  // 4 waves of 64 lanes
constexpr int kXcds = 8;       // MI355X: 8 XCDs, 32 CUs each

// Workgroups are dealt round-robin to the XCDs (id % 8).  Renumber them so
// that consecutive logical tile ids land on the same XCD and share its L2.
__device__ __forceinline__ int xcd_remap(int bid, int total) {
  int q = total / kXcds, r = total % kXcds;
  int xcd = bid % kXcds, idx = bid / kXcds;
  return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

// A wave-uniform value in a scalar register (integer division leaves its
// result in a vector register).
__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }

// What workgroup b of a levelled launch runs (args.hpp): the tile (over all
// batch planes), its slices [s0, s1) of nk and the block of partial sums they
// go to (-1: a whole tile, written to C).  Runs of one number are
// neighbours, so the tiles of a moment read the same K range.  Selects, no
// branches: with branches the compiler kept these values in scratch memory.
template <typename Args>
__device__ __forceinline__ void level_work(const Args& a, int b, int nk, int& tile, int& s0, int& s1, int& block) {
  const bool whole = b < a.head, first = !whole && b < a.head + a.rem;
  const int from = whole ? 0 : first ? a.head : a.head + a.rem;
  const int count = whole ? a.head : first ? a.rem : a.rem * a.lev_parts;
  const int v = scalar(xcd_remap(b - from, count));
  const int run = whole || first ? 0 : scalar(v / a.rem), i = v - run * a.rem;
  tile = whole ? v : a.head + i;
  s0 = whole || first ? 0 : a.lev_q + run * a.lev_part;
  s1 = whole ? nk : first ? a.lev_q : min(nk, s0 + a.lev_part);
  block = whole ? -1 : first ? i : a.rem + i * a.lev_parts + run;
}

// Element at `off` from `base`: uint32_t offsets count bytes (an SGPR base
// plus a 32-bit VGPR offset per load); int32_t and int64_t offsets count
// elements (int32_t for operands past 4 GiB but under 2^31 elements: 32-bit
// registers per offset like the byte form).
template <typename T>
__device__ __forceinline__ T* at(T* base, uint32_t off) {
  typedef typename std::conditional<std::is_const<T>::value, const char, char>::type byte;
  return reinterpret_cast<T*>(reinterpret_cast<byte*>(base) + off);
}
template <typename T>
__device__ __forceinline__ T* at(T* base, int32_t off) {
  return base + (int64_t)off;
}
template <typename T>
__device__ __forceinline__ T* at(T* base, int64_t off) {
  return base + off;
}

// Offsets that count bytes (the uint32_t form) rather than elements.
template <typename OffT>
constexpr bool kByteOffsets = std::is_same<OffT, uint32_t>::value;

// Operands always live in global memory.  Loads and stores through these
// helpers say so, so they compile to global (not flat) instructions even when
// the pointer was read from memory, as in the batched kernel: a flat load
// takes a 64-bit VGPR address and is counted by the LDS wait counter too.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* global(const T* p) {
  return (const __attribute__((address_space(1))) T*)p;
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* global(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}
template <typename T, typename OffT>
__device__ __forceinline__ T gload(const T* base, OffT off) {
  return *global(at(base, off));
}

// MFMA shapes.  In every shape the lane index l selects the row (of the left
// operand) and the column (of the right operand) as l % BS, and the group
// l / BS selects the contraction index, the same way for both operands, so
// any consistent assignment of tile k's to (group, step) is valid.
template <typename T>
struct Mfma;

template <>
struct Mfma<double> {  // v_mfma_f64_16x16x4_f64
  static constexpr int BS = 16, KG = 4, NACC = 4;
  using Acc = f64x4;
  __device__ __forceinline__ static Acc mma(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // row of accumulator element r held by lane l (column is l % 16)
  __device__ __forceinline__ static int row(int l, int r) { return (l / 16) + 4 * r; }
};

template <>
struct Mfma<float> {  // v_mfma_f32_32x32x2_f32
  static constexpr int BS = 32, KG = 2, NACC = 16;
  using Acc = f32x16;
  __device__ __forceinline__ static Acc mma(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  __device__ __forceinline__ static int row(int l, int r) {
    return 8 * (r / 4) + 4 * (l / 32) + (r % 4);
  }
};

// Gather of one operand tile (BR rows of the free dimension x BK contracted
// indices) from strided global memory through the block-scatter indexing
// vectors into LDS laid out [row][k] with leading dimension LDK (16-byte
// aligned rows, padded by 16 bytes so that the MFMA operand reads and the
// stores below are free of bank conflicts).
//
// KFAST (the operand's smallest stride is a contracted mode): lanes run along
// k; each thread owns KV consecutive k's (KV = 1 for the plain kernels, 2 for
// the bf16 split, whose stores pack pairs) in E / KV rows.
// Row-fast (otherwise): lanes run along the rows, each thread owns one row and
// a run of E consecutive k's, stored to LDS as 16-byte vectors.
// Rows past the problem edge carry offset 0 (a valid address) and only feed
// accumulator rows that are never stored; k's past the edge are stored as 0.
//
// The phases are split so a K loop can pipeline them: fetch_k() loads the
// contracted-index offsets of a future slice, load() issues the data loads of
// the next slice (nothing waits on them until store()), store() writes the
// slice into LDS, zeroing k >= kend.  Element j of a thread is
// (row j / KV, k j % KV) in the KFAST case and (row 0, k j) otherwise.
// NSLOT > 1 keeps that many slices in flight: each phase takes the slot it
// works on as a template argument.
template <typename T, typename OffT, int BR, int BK, bool KFAST, int KV = 1, int NSLOT = 1, bool SCALARK = false>
struct TileGather {
  static constexpr int E = BR * BK / kThreads;
  static constexpr int kLoads = E;
  static constexpr int KVT = KV;                  // KFAST: consecutive k's per thread
  static constexpr int LDK = BK + 16 / (int)sizeof(T);
  static constexpr int VK = 16 / (int)sizeof(T);  // k's per 16-byte vector
  static constexpr int KT = BK / KV;              // KFAST: threads along k
  static constexpr int RSTEP = kThreads / KT;     // KFAST: row step between a thread's rows
  static constexpr int KPH = kThreads / BR;       // row-fast: threads sharing one row
  static_assert(E >= 1 && E % KV == 0, "tile too small for the workgroup");
  static_assert(KFAST ? (kThreads % KT == 0 && BR % RSTEP == 0)
                      : (kThreads % BR == 0 && BK % KPH == 0 && E % VK == 0),
                "tile shape does not divide the workgroup");

  // SCALARK, row-fast with byte offsets: the run's contracted offsets are the
  // same for the whole wave.  They are fetched with one load, entry j in lane
  // j, and read back into scalar registers, so each data load is a scalar
  // address plus the row's 32-bit offset: one register per slot instead of E.
  // Taken where registers are short: the bf16x3 kernel with one row-gathered
  // operand no longer spills (7 and, under the void mask, 37 registers; ring
  // o=48 v=192 5.51 -> 5.40 ms); in the FP32 kernels, which have them, the
  // address work per load costs more (autograd step 2.33 against 2.42 ms).
  static constexpr bool SK = SCALARK && !KFAST && kByteOffsets<OffT> && E <= 64;

  OffT mn[KFAST ? E / KV : 1];  // row offsets, fixed for the tile
  OffT ko[NSLOT][KFAST ? KV : SK ? 1 : E];  // contracted-index offsets of a slice to load
  T v[NSLOT][E];
  int r0, kk0;  // first row; first k of the thread's run

  __device__ __forceinline__ void init(const OffT* __restrict__ mnoff, int tile_r0, int tid) {
    if constexpr (KFAST) {
      kk0 = (tid % KT) * KV;
      r0 = tid / KT;
#pragma unroll
      for (int i = 0; i < E / KV; ++i) mn[i] = mnoff[tile_r0 + r0 + i * RSTEP];
    } else {
      r0 = tid % BR;
      // The k run is the same for a whole wave, but its offsets are fetched
      // with vector loads on purpose: scalar loads share the LDS wait
      // counter, and every wait for an MFMA operand read would then also wait
      // for the offsets of a slice two steps ahead.
      kk0 = SK ? scalar((tid / BR) * E) : (tid / BR) * E;
      mn[0] = mnoff[tile_r0 + r0];
    }
  }

  // Offsets of slice [k0, k0 + BK); koff must hold k0 + BK entries.  Row-fast
  // runs are read as 16-byte vectors: every indexing vector starts on a
  // 64-byte boundary and k0 + kk0 is a multiple of E.
  static constexpr int OV = 16 / (int)sizeof(OffT);
  template <int S = 0>
  __device__ __forceinline__ void fetch_k(const OffT* __restrict__ koff, int k0) {
    if constexpr (SK) {
      ko[S][0] = koff[k0 + kk0 + threadIdx.x % E];
    } else if constexpr (!KFAST && E % OV == 0) {
      typedef OffT ovec_t __attribute__((ext_vector_type(16 / sizeof(OffT))));
      const ovec_t* src = reinterpret_cast<const ovec_t*>(koff + k0 + kk0);
#pragma unroll
      for (int q = 0; q < E / OV; ++q) {
        const ovec_t w = src[q];
#pragma unroll
        for (int u = 0; u < OV; ++u) ko[S][q * OV + u] = w[u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < (KFAST ? KV : E); ++u) ko[S][u] = koff[k0 + kk0 + u];
    }
  }

  template <int S = 0>
  __device__ __forceinline__ void load(const T* __restrict__ base) {
    if constexpr (SK) {
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const uint32_t so = (uint32_t)__builtin_amdgcn_readlane((int)ko[S][0], j);
        v[S][j] = gload(at(base, so), mn[0]);
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < E; ++j)
      v[S][j] = KFAST ? gload(base, (OffT)(mn[j / KV] + ko[S][j % KV])) : gload(base, (OffT)(mn[0] + ko[S][SK ? 0 : j]));
  }

  __device__ __forceinline__ int krel(int j) const { return kk0 + (KFAST ? j % KV : j); }

  // Value of element j of the slice starting at k0 (0 past kend).
  template <int S = 0>
  __device__ __forceinline__ T value(int j, int k0, int kend) const {
    return k0 + krel(j) < kend ? v[S][j] : T(0);
  }

  // value() where EDGE, the raw element otherwise (slices wholly inside K).
  template <bool EDGE, int S = 0>
  __device__ __forceinline__ T val(int j, int k0, int kend) const {
    return EDGE ? value<S>(j, k0, kend) : v[S][j];
  }

  __device__ __forceinline__ int lds_index(int j, int ldk) const {
    return KFAST ? (r0 + (j / KV) * RSTEP) * ldk + kk0 + j % KV : r0 * ldk + kk0 + j;
  }

  // Store the slice to LDS, zeroing k's past kend.  Only the last slice of a
  // K range can hold such k's, so the test is skipped (a uniform branch) on
  // every other slice.
  template <bool EDGE, int S>
  __device__ __forceinline__ void store_impl(T* __restrict__ lds, int k0, int kend) const {
    if constexpr (KFAST) {
#pragma unroll
      for (int j = 0; j < E; ++j) lds[lds_index(j, LDK)] = val<EDGE, S>(j, k0, kend);
    } else {
      typedef T vec_t __attribute__((ext_vector_type(16 / sizeof(T))));
#pragma unroll
      for (int q = 0; q < E / VK; ++q) {
        vec_t w;
#pragma unroll
        for (int u = 0; u < VK; ++u) w[u] = val<EDGE, S>(q * VK + u, k0, kend);
        *reinterpret_cast<vec_t*>(lds + r0 * LDK + kk0 + q * VK) = w;
      }
    }
  }
  template <int S = 0>
  __device__ __forceinline__ void store(T* __restrict__ lds, int k0, int kend) const {
    if (k0 + BK <= kend)
      store_impl<false, S>(lds, k0, kend);
    else
      store_impl<true, S>(lds, k0, kend);
  }
  // The same with the slice's void mask (bit k: index k of the slice does not
  // count and is stored as 0).
  template <int S = 0>
  __device__ __forceinline__ void store_masked(T* __restrict__ lds, uint32_t voids) {
    store_impl<false, S>(lds, 0, 0);
    if (voids)
      zero(voids, [&](int r, int k) { lds[r * LDK + k] = T(0); });
  }
  // f(row, k) for this thread's elements at the slice's void k's
  template <typename F>
  __device__ __forceinline__ void zero(uint32_t voids, F f) const {
    for (int j = 0; j < E; ++j)
      if ((voids >> krel(j)) & 1u) f(KFAST ? r0 + (j / KV) * RSTEP : r0, krel(j));
  }
};

// Loader for a pre-packed operand (the packing step hoisted out of repeated
// calls: Girder 2, "Enabling optimizations across layers").  The packed
// buffer holds the operand tile by tile in the kernel's order: block
// (tile, kb) is BR x BK elements stored [row][k] densely, zero-filled past the
// problem edges, blocks ordered tile-major (tile * nkb + kb).  A slice is then
// a contiguous run of 16-byte vectors: no indexing vectors, no edge tests.
template <typename T, int BR, int BK, int NSLOT = 1>
struct PackedGather {
  static constexpr int VK = 16 / (int)sizeof(T);
  static constexpr int LDK = BK + VK;
  static constexpr int NV = BR * BK / VK;  // vectors per block
  static constexpr int VPT = NV / kThreads;
  static constexpr int kLoads = VPT;
  static_assert(NV % kThreads == 0 && BK % VK == 0, "packed block does not divide the workgroup");
  typedef T vec_t __attribute__((ext_vector_type(16 / sizeof(T))));
  vec_t v[NSLOT][VPT];
  int tile = 0, kb[NSLOT] = {}, nkb = 1, tid = 0;

  template <typename OffT>
  __device__ __forceinline__ void init(const OffT* /*unused*/, int tile_r0, int t) {
    tile = tile_r0 / BR;
    tid = t;
  }
  template <int S = 0, typename OffT>
  __device__ __forceinline__ void fetch_k(const OffT* /*unused*/, int k0) {
    kb[S] = k0 / BK;
  }
  template <int S = 0>
  __device__ __forceinline__ void load(const T* __restrict__ base) {
    const vec_t* blk = reinterpret_cast<const vec_t*>(base + ((size_t)tile * nkb + kb[S]) * (size_t)(BR * BK));
#pragma unroll
    for (int q = 0; q < VPT; ++q) v[S][q] = *global(blk + tid + q * kThreads);
  }
  template <int S = 0>
  __device__ __forceinline__ void store(T* __restrict__ lds, int /*k0*/, int /*kend*/) const {
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      const int e = (tid + q * kThreads) * VK;
      *reinterpret_cast<vec_t*>(lds + (e / BK) * LDK + e % BK) = v[S][q];
    }
  }
  template <int S = 0>
  __device__ __forceinline__ void store_masked(T* __restrict__ lds, uint32_t /*voids: packed as 0*/) const {
    store<S>(lds, 0, 0);
  }
};

// Loader for a K-gathered operand whose every aligned run of 16 bytes along
// K is contiguous in memory (the block-scatter layout's block strides,
// Approach, "Supporting tensor computations"): each thread reads VK
// consecutive k's of a row with one 16-byte load (at element alignment:
// gfx950 global loads need no more) instead of VK gathered loads, and takes
// one offset per slice.  Runs of any length of at least VK elements get that
// form from the plan's padded contracted order (KRuns): element loads are
// bound by the cache lines they touch per instruction (FP32 ladder v=93 o=27,
// runs of 93 on both sides: 1095 us with element loads, 1002 with runs; bf16x6
// ring o=31 v=115 722 -> 668 us).
//
// With whole slices and nothing to leave out (mode kVecK) a slice is stored
// as it was loaded.  Otherwise (mode kRunK) the plan's void mask -- one bit
// per entry of the contracted order, set for repeated entries and past the
// end of K -- says which entries to store as 0, in both operands; a slice
// without such entries takes the plain store only.  The zeros are written
// over the stored slice, by the threads that stored the elements: branches
// that change the loaded registers cost registers at their joins (bf16x3 with
// a row-gathered partner: 29 spilled with masked registers), and a load with
// a fallback for a partial slice made the compiler wait there for the other
// operand's loads on every step.
template <typename T, typename OffT, int BR, int BK, int NSLOT = 1>
struct VecKGather {
  static constexpr int VK = 16 / (int)sizeof(T);
  // one element in offset units: bytes for the byte form, else 1
  static constexpr int kStep = kByteOffsets<OffT> ? (int)sizeof(T) : 1;
  static constexpr int LDK = BK + VK;
  static constexpr int KT = BK / VK;           // threads along k
  static constexpr int RSTEP = kThreads / KT;  // rows between a thread's runs
  static constexpr int NR = BR / RSTEP;        // runs per thread
  static constexpr int kLoads = NR;
  static_assert(BK % VK == 0 && kThreads % KT == 0 && BR % RSTEP == 0, "tile shape does not divide the workgroup");
  typedef T vec_t __attribute__((ext_vector_type(16 / sizeof(T))));
  typedef T gvec_t __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
  OffT mn[NR];
  OffT ko[NSLOT];
  vec_t v[NSLOT][NR];
  int r0 = 0, kk0 = 0;

  __device__ __forceinline__ void init(const OffT* __restrict__ mnoff, int tile_r0, int tid) {
    kk0 = (tid % KT) * VK;
    r0 = tid / KT;
#pragma unroll
    for (int i = 0; i < NR; ++i) mn[i] = mnoff[tile_r0 + r0 + i * RSTEP];
  }
  template <int S = 0>
  __device__ __forceinline__ void fetch_k(const OffT* __restrict__ koff, int k0) {
    // FP64: named global, the load is scheduled so that the ladder o=32 v=128
    // takes 7.58 instead of 7.71 ms; the FP32 ladder, 3.89 instead of 3.82
    if constexpr (sizeof(T) == 8)
      ko[S] = *global(koff + k0 + kk0);
    else
      ko[S] = koff[k0 + kk0];
  }
  template <int S = 0>
  __device__ __forceinline__ void load(const T* __restrict__ base) {
#pragma unroll
    for (int i = 0; i < NR; ++i) 
      v[S][i] = *reinterpret_cast<const __attribute__((address_space(1))) gvec_t*>(
          global(at(base, (OffT)(mn[i] + ko[S]))));
  }
  template <int S = 0>
  __device__ __forceinline__ void store(T* __restrict__ lds, int /*k0*/, int /*kend*/) const {
#pragma unroll
    for (int i = 0; i < NR; ++i) *reinterpret_cast<vec_t*>(lds + (r0 + i * RSTEP) * LDK + kk0) = v[S][i];
  }
  template <int S = 0>
  __device__ __forceinline__ void store_masked(T* __restrict__ lds, uint32_t voids) {
    store<S>(lds, 0, 0);
    if (voids)
      zero(voids, [&](int r, int k) { lds[r * LDK + k] = T(0); });
  }
  template <typename F>
  __device__ __forceinline__ void zero(uint32_t voids, F f) const {
    for (int u = 0; u < VK; ++u)
      if ((voids >> (kk0 + u)) & 1u)
        for (int i = 0; i < NR; ++i) f(r0 + i * RSTEP, kk0 + u);
  }
};

// Void mask of the BK contracted entries from k0 (a multiple of BK), as a
// wave-uniform value: bit k set where entry k0 + k does not count.
template <int BK>
__device__ __forceinline__ uint32_t void_bits(uint32_t word, int k0) {
  static_assert(32 % BK == 0, "a slice lies in one word of the void mask");
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)word);
  return BK == 32 ? w : (w >> (k0 & 31)) & ((1u << (BK % 32)) - 1u);
}

// Operand loaders by mode: 0 row-gathered, 1 K-gathered, 2 pre-packed,
// 3 K-gathered in 16-byte runs, every slice whole, 4 the same under the
// plan's void mask.
enum { kRowGather = 0, kKGather = 1, kPacked = 2, kVecK = 3, kRunK = 4 };
// Whether both operands of a slice are stored under the void mask: with an
// operand in masked runs, and for an operand gathered by elements beside a
// pre-packed one, whose plan may have the padded contracted order -- the
// packed side holds 0 at a void entry, and the partner's real value there
// must not meet it (0 * Inf).
constexpr bool masked_modes(int xm, int ym) {
  return xm == kRunK || ym == kRunK || (xm == kPacked && (ym == kRowGather || ym == kKGather)) ||
         (ym == kPacked && (xm == kRowGather || xm == kKGather));
}
template <int MODE>
constexpr bool known_mode() {
  static_assert(MODE >= kRowGather && MODE <= kRunK, "unknown loader mode");
  return true;
}
template <typename T, typename OffT, int BR, int BK, int MODE, int KV = 1, int NSLOT = 1,
          bool = known_mode<MODE>()>
using Loader = typename std::conditional<
    MODE == kPacked, PackedGather<T, BR, BK, NSLOT>,
    typename std::conditional<MODE == kVecK || MODE == kRunK, VecKGather<T, OffT, BR, BK, NSLOT>,
                              TileGather<T, OffT, BR, BK, MODE == kKGather, KV, NSLOT>>::type>::type;

}  // namespace famlies
