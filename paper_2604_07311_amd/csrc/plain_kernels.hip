// Plain FP64 / FP32 strided-contraction kernels, the split-K reduction and
// the K == 0 scaling kernel.
//
// One workgroup computes one BM x BN tile of C (in the kernel view
// C(m,n) = sum_k X(m,k) Y(k,n)) over one K range:
//   gather X and Y K-slices through the block-scatter indexing vectors into
//   double-buffered LDS  ->  2x2 waves, each a (BM/2)x(BN/2) MFMA tile
//   ->  alpha/beta scatter-update of C through C's indexing vectors
// (block-scatter mapping, Approach, "Supporting tensor computations"; the
// loops-around-a-micro-kernel structure of Fig. "five loops").
#include "launch.hpp"
#include "tile.hpp"

// Two workgroups per CU (waves per SIMD) for the plain kernels: the FP64 tile
// then keeps its accumulators in VGPRs within 256 registers, and a second
// workgroup hides the other's barrier and global-load latency.
#ifndef FAMLIES_PLAIN_WAVES_PER_EU
#define FAMLIES_PLAIN_WAVES_PER_EU 2
#endif

namespace famlies {

template <typename T, typename OffT, int BM, int BN, int BK, int XM, int YM>
__global__ __launch_bounds__(kThreads, FAMLIES_PLAIN_WAVES_PER_EU) void plain_contract(PlainArgs<OffT> a) {
  // Two slices in flight where the registers allow it: tiles with a
  // row-gathered operand and 32-bit offsets (one load per element along K,
  // so its slice takes longest to arrive), and tiles whose operands are both
  // read in affine 16-byte blocks (few registers per slice; FP64 only with
  // 32-bit offsets).  Measured on the ladder (both affine): FP64 82 -> 87 %,
  // FP32 83 -> 88 %, FP32 with 64-bit offsets 77 -> 85 % of peak.  FP64
  // slices are 8 deep (the FP64 MFMA takes 4 k's, so two steps per slice):
  // half the staging registers of 16-deep slices, which lets the FP64 tile
  // with a row-gathered operand keep two slices in flight too (ring o=48
  // v=192 83.1 -> 85.5 %; ladder 87.0 -> 87.7 %).  With both operands
  // element-gathered along K the deeper pipeline was no faster.
  static constexpr bool kBothRuns = (XM == kVecK || XM == kRunK) && (YM == kVecK || YM == kRunK);
  static constexpr int kDepth = ((sizeof(OffT) == 4 && (XM == kRowGather || YM == kRowGather)) ||
                                 ((sizeof(OffT) == 4 || sizeof(T) == 4) && kBothRuns))
                                    ? 2
                                    : 1;
  using Tile = PlainTile<T, BM, BN, BK, XM, YM, kDepth>;
  __shared__ T smem[Tile::SMEM];
  // Work units in launch order: with a levelled last round, level_work's; without
  // split-K, every tile of every batch plane; with split-K, first the tiles [0, head) over all of K, then each
  // remaining tile once per K slice.  Each range is spread over the XCDs in
  // contiguous blocks, so neighbouring tiles share an L2.
  const int ntiles = a.tiles_m * a.tiles_n;
  TileJob<OffT> j;
  j.kbeg = 0;
  j.kend = a.K;
  int t;            // tile over all batch planes
  int block = -1;   // its block of partial sums, -1: none
  if (BM == 128 && BN == 128 && a.rem > 0) {
    int s0, s1;
    level_work(a, (int)blockIdx.x, (a.K + BK - 1) / BK, t, s0, s1, block);
    j.kbeg = s0 * BK;
    j.kend = min(a.K, s1 * BK);
  } else if (a.splits == 1) {
    t = xcd_remap(blockIdx.x, gridDim.x);
  } else if ((int)blockIdx.x < a.head) {
    t = xcd_remap(blockIdx.x, a.head);
  } else {
    const int ntail = ntiles - a.head;
    const int v = xcd_remap(blockIdx.x - a.head, gridDim.x - a.head);
    const int split = v / ntail;
    t = a.head + v % ntail;
    block = v;
    j.kbeg = split * a.kchunk;
    j.kend = min(a.K, j.kbeg + a.kchunk);
  }
  t = scalar(t);
  block = scalar(block);
  j.kbeg = scalar(j.kbeg);
  j.kend = scalar(j.kend);
  const int l = scalar(t / ntiles), tl = t - l * ntiles;  // batch index, tile of its plane
  // M fastest: neighbours share Y's panel
  const int pn = scalar(tl / a.tiles_m), pm = tl - pn * a.tiles_m;
  // a pre-packed operand holds its batch planes back to back
  j.x = static_cast<const T*>(a.x) +
        (XM == kPacked ? (int64_t)l * a.tiles_m * a.x_nkb * (int64_t)(BM * BK) : a.xl[l]);
  j.y = static_cast<const T*>(a.y) +
        (YM == kPacked ? (int64_t)l * a.tiles_n * a.y_nkb * (int64_t)(BN * BK) : a.yl[l]);
  j.x_nkb = a.x_nkb;
  j.y_nkb = a.y_nkb;
  j.c = static_cast<T*>(a.c) + a.cl[l];
  j.xmn = a.xmn;
  j.xk = a.xk;
  j.yk = a.yk;
  j.ymn = a.ymn;
  j.cm = a.cm;
  j.cn = a.cn;
  j.kvoid = a.kvoid;
  j.M = a.M;
  j.N = a.N;
  j.m0 = pm * BM;
  j.n0 = pn * BN;
  j.alpha = a.alpha;
  j.beta = a.beta;
  // partial sums: a dense BM x BN block of their own
  j.ldw = BN;
  j.work = block < 0 ? nullptr
                     : static_cast<void*>(static_cast<T*>(a.work) + (size_t)block * (size_t)(BM * BN));
  Tile::run(j, smem);
}

// For the split tiles: C = alpha * sum_s W[s] + beta * C, the K slices
// summed in index order so the result does not depend on scheduling.  One
// thread per element of a split tile (bm x bn blocks, row-major).  P: type of
// the partial sums (T; double in the bf16 kernels).
template <typename T, typename P, typename OffT>
__global__ __launch_bounds__(kThreads) void splitk_reduce(PlainArgs<OffT> a, int bm, int bn) {
  // whole workgroups per block (bm * bn is a multiple of 256, bn a power of two)
  const int ntail = a.tiles_m * a.tiles_n - a.head, per = bm * bn, wgs = per / kThreads;
  const int tt = scalar((int)blockIdx.x / wgs), r = ((int)blockIdx.x - tt * wgs) * kThreads + threadIdx.x;
  const int t = a.head + tt, pn = scalar(t / a.tiles_m), pm = t - pn * a.tiles_m;
  const int ri = r >> __builtin_ctz(bn), m = pm * bm + ri, n = pn * bn + (r & (bn - 1));
  if (m >= a.M || n >= a.N) return;
  const P* W = static_cast<const P*>(a.work) + (size_t)tt * per + r;
  P s = P(0);
#pragma unroll 4
  for (int k = 0; k < a.splits; ++k) s += *global(W + (size_t)k * ntail * per);
  T* cp = at(static_cast<T*>(a.c), (OffT)(a.cm[m] + a.cn[n]));
  const P al = static_cast<P>(a.alpha), be = static_cast<P>(a.beta);
  P v = al * s;
  if (be != P(0)) v += be * (P)*cp;
  *cp = (T)v;
}

// The levelled tiles: C = alpha * (their blocks of partial sums in order) +
// beta * C.  P is the type of the partial sums (and of the update): T for the
// plain kernels, double for the bf16 kernels.  A workgroup takes eight rows of
// a tile, its lanes consecutive columns, four rows of four blocks per thread in
// flight; bound by HBM (partial sums read once, C read and written), by latency
// where the tiles are few (75 x 4882, 13 blocks a tile: 11.3 us with 16 rows of
// one block in flight, 9.6).
constexpr int kLevelRows = 8;
template <typename T, typename P, typename OffT>
__global__ __launch_bounds__(kThreads) void level_reduce(PlainArgs<OffT> a, int bm) {
  constexpr int B = 128, RW = kLevelRows, RT = RW / 2;  // B: columns of a tile
  const int i = blockIdx.x / (bm / RW), row0 = (blockIdx.x % (bm / RW)) * RW + threadIdx.x / B;
  const size_t per = (size_t)bm * B;
  const int ntiles = a.tiles_m * a.tiles_n;
  const int t = a.head + i, l = t / ntiles, tl = t % ntiles;
  const int m0 = (tl % a.tiles_m) * bm + row0, n = (tl / a.tiles_m) * B + threadIdx.x % B;
  if (m0 >= a.M || n >= a.N) return;  // past the edges of a ragged tile: nothing to read either
  const P* W = static_cast<const P*>(a.work) + (size_t)row0 * B + threadIdx.x % B;
  P s[RT];
#pragma unroll
  for (int q = 0; q < RT; ++q) s[q] = *global(W + i * per + q * 2 * B);
#pragma unroll 4
  for (int w = 0; w < a.lev_parts; ++w)
#pragma unroll
    for (int q = 0; q < RT; ++q)
      s[q] += *global(W + ((size_t)a.rem + (size_t)i * a.lev_parts + w) * per + q * 2 * B);
  T* C = static_cast<T*>(a.c) + a.cl[l];
  const OffT cn = a.cn[n];
  const P al = static_cast<P>(a.alpha), be = static_cast<P>(a.beta);
  OffT co[RT];
  P c[RT];
#pragma unroll
  for (int q = 0; q < RT; ++q) co[q] = (OffT)(a.cm[m0 + 2 * q < a.M ? m0 + 2 * q : 0] + cn);
  if (be != P(0)) {
#pragma unroll
    for (int q = 0; q < RT; ++q) c[q] = (P)*global(at(C, co[q]));
  }
#pragma unroll
  for (int q = 0; q < RT; ++q)
    if (m0 + 2 * q < a.M) {
      P v = al * s[q];
      if (be != P(0)) v += be * c[q];
      *global(at(C, co[q])) = (T)v;
    }
}

// bf16: the partial sums are FP64.
template <typename OffT>
hipError_t launch_level_reduce(int dtype, bool bf16, const PlainArgs<OffT>& a, int bm, hipStream_t s) {
  const dim3 grid(a.rem * (bm / kLevelRows));
  if (dtype == FAMLIES_F64)
    hipLaunchKernelGGL((level_reduce<double, double, OffT>), grid, dim3(kThreads), 0, s, a, bm);
  else if (bf16)
    hipLaunchKernelGGL((level_reduce<float, double, OffT>), grid, dim3(kThreads), 0, s, a, bm);
  else
    hipLaunchKernelGGL((level_reduce<float, float, OffT>), grid, dim3(kThreads), 0, s, a, bm);
  return hipGetLastError();
}
template hipError_t launch_level_reduce(int, bool, const PlainArgs<uint32_t>&, int, hipStream_t);
template hipError_t launch_level_reduce(int, bool, const PlainArgs<int32_t>&, int, hipStream_t);
template hipError_t launch_level_reduce(int, bool, const PlainArgs<int64_t>&, int, hipStream_t);

template <typename OffT>
hipError_t launch_splitk_reduce(int dtype, bool bf16, const PlainArgs<OffT>& a, int bm, int bn, hipStream_t s) {
  const int64_t red = ((int64_t)a.tiles_m * a.tiles_n - a.head) * bm * bn;
  const dim3 grid((int)((red + kThreads - 1) / kThreads));
  if (dtype == FAMLIES_F64)
    hipLaunchKernelGGL((splitk_reduce<double, double, OffT>), grid, dim3(kThreads), 0, s, a, bm, bn);
  else if (bf16)
    hipLaunchKernelGGL((splitk_reduce<float, double, OffT>), grid, dim3(kThreads), 0, s, a, bm, bn);
  else
    hipLaunchKernelGGL((splitk_reduce<float, float, OffT>), grid, dim3(kThreads), 0, s, a, bm, bn);
  return hipGetLastError();
}
template hipError_t launch_splitk_reduce(int, bool, const PlainArgs<uint32_t>&, int, int, hipStream_t);
template hipError_t launch_splitk_reduce(int, bool, const PlainArgs<int32_t>&, int, int, hipStream_t);
template hipError_t launch_splitk_reduce(int, bool, const PlainArgs<int64_t>&, int, int, hipStream_t);

// K == 0 or alpha == 0: C = beta * C (beta == 0 writes zeros without reading C).
template <typename T, typename OffT>
__global__ __launch_bounds__(kThreads) void scale_c(PlainArgs<OffT> a) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t mn = (int64_t)a.M * a.N;
  if (i >= mn * a.L) return;
  const int l = (int)(i / mn);
  const int64_t r = i % mn;
  const int m = (int)(r / a.N), n = (int)(r % a.N);
  T* cp = at(static_cast<T*>(a.c) + a.cl[l], (OffT)(a.cm[m] + a.cn[n]));
  const T be = static_cast<T>(a.beta);
  *cp = be != T(0) ? be * *cp : T(0);
}

// ------------------------------------------------------------------ dispatch
template <typename T, typename OffT, int BM, int BN, int BK, int XM, int YM>
static void launch_one(const PlainArgs<OffT>& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL((plain_contract<T, OffT, BM, BN, BK, XM, YM>), dim3(grid), dim3(kThreads), 0, s, a);
}

// Gathered operands and whole 16-byte runs (modes 0, 1, 3) with every offset
// form; pre-packed operands and masked runs (modes 2, 4) with byte offsets.
template <typename T, typename OffT, int BM, int BN, int BK>
static hipError_t launch_tile(const PlainArgs<OffT>& a, int xm, int ym, int grid, hipStream_t s) {
#define FAMLIES_MODES(X, Y) \
  case X * 8 + Y: launch_one<T, OffT, BM, BN, BK, X, Y>(a, grid, s); return hipGetLastError();
  switch (xm * 8 + ym) {
    FAMLIES_MODES(0, 0) FAMLIES_MODES(0, 1) FAMLIES_MODES(0, 3)
    FAMLIES_MODES(1, 0) FAMLIES_MODES(1, 1) FAMLIES_MODES(1, 3)
    FAMLIES_MODES(3, 0) FAMLIES_MODES(3, 1) FAMLIES_MODES(3, 3)
    default: break;
  }
  if constexpr (kByteOffsets<OffT>) {
    switch (xm * 8 + ym) {
      FAMLIES_MODES(0, 2) FAMLIES_MODES(1, 2) FAMLIES_MODES(3, 2) FAMLIES_MODES(4, 2)
      FAMLIES_MODES(2, 0) FAMLIES_MODES(2, 1) FAMLIES_MODES(2, 3) FAMLIES_MODES(2, 4) FAMLIES_MODES(2, 2)
      FAMLIES_MODES(4, 0) FAMLIES_MODES(4, 1) FAMLIES_MODES(4, 4) FAMLIES_MODES(0, 4) FAMLIES_MODES(1, 4)
      default: break;
    }
  }
#undef FAMLIES_MODES
  return hipErrorInvalidValue;
}

template <typename T, typename OffT>
static hipError_t launch_plain_t(const PlainArgs<OffT>& a, const PlainLaunch& L, hipStream_t s) {
  const int64_t mn = (int64_t)a.M * a.N;
  if (L.kind == PlainLaunch::kScale) {
    hipLaunchKernelGGL((scale_c<T, OffT>), dim3((int)((mn * a.L + kThreads - 1) / kThreads)), dim3(kThreads),
                       0, s, a);
    return hipGetLastError();
  }
  const int64_t ntiles = (int64_t)a.tiles_m * a.tiles_n;
  const int grid = a.rem > 0 ? a.head + a.rem * (1 + a.lev_parts)
                             : (int)(a.splits == 1 ? ntiles * a.L : a.head + (ntiles - a.head) * a.splits);
  constexpr int BK = sizeof(T) == 8 ? 8 : 32;
  hipError_t e = hipErrorInvalidValue;
  if (L.bm == 128 && L.bn == 128 && L.bk == BK)
    e = launch_tile<T, OffT, 128, 128, BK>(a, L.xm, L.ym, grid, s);
  else if (L.bm == 64 && L.bn == 64 && L.bk == BK)
    e = launch_tile<T, OffT, 64, 64, BK>(a, L.xm, L.ym, grid, s);
  if (e == hipSuccess && a.rem > 0) return launch_level_reduce(sizeof(T) == 8 ? FAMLIES_F64 : FAMLIES_F32, false, a, L.bm, s);
  if (e != hipSuccess || a.splits == 1) return e;
  return launch_splitk_reduce(sizeof(T) == 8 ? FAMLIES_F64 : FAMLIES_F32, false, a, L.bm, L.bn, s);
}

hipError_t launch_plain(int dtype, const PlainArgs<uint32_t>& a, const PlainLaunch& L, hipStream_t s) {
  return dtype == FAMLIES_F64 ? launch_plain_t<double, uint32_t>(a, L, s)
                              : launch_plain_t<float, uint32_t>(a, L, s);
}

hipError_t launch_plain(int dtype, const PlainArgs<int32_t>& a, const PlainLaunch& L, hipStream_t s) {
  return dtype == FAMLIES_F64 ? launch_plain_t<double, int32_t>(a, L, s)
                              : launch_plain_t<float, int32_t>(a, L, s);
}

hipError_t launch_plain(int dtype, const PlainArgs<int64_t>& a, const PlainLaunch& L, hipStream_t s) {
  return dtype == FAMLIES_F64 ? launch_plain_t<double, int64_t>(a, L, s)
                              : launch_plain_t<float, int64_t>(a, L, s);
}

bool plain_tile_supported(int dtype, int bm, int bn, int bk) {
  const int BK = dtype == FAMLIES_F64 ? 8 : 32;
  return bk == BK && ((bm == 128 && bn == 128) || (bm == 64 && bn == 64));
}

}  // namespace famlies
