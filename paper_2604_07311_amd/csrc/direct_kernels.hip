// Small and narrow FP64 / FP32 contractions: operands straight from global
// memory into MFMA registers.
//
// A wave owns a (16 MB) x (16 NB) tile of C (kernel view) over a share of K
// and loads each operand element into the lane that multiplies it, through
// the same block-scatter indexing vectors as the tiled kernels; there is no
// LDS staging and no barrier in the K loop.  The waves of a workgroup either
// share one tile, each taking every wk-th K step (their partial tiles are
// summed through LDS in wave order, so results do not depend on timing), or
// (wk = 1) own a tile each.
//
// What bounds it: with few tiles, the latency of a wave's K steps (so K is
// spread over the four waves and three steps are in flight); with many, L2,
// since every operand element is read once per tile of the other side
// (9 TB/s measured).  Counters: FP64 six modes of 16 6.3 us, matrix cores 3 %
// busy, waves waiting 69 % of their time; FP32 777 x 319 x 437 12.8 us, 7 %,
// 5 TB/s of L2 requests; FP64 16 x 675840 x 64 108 us, HBM at 4.05 TB/s.
//
// In FP32 a wave's chain is no longer than a K range of the tiled plan (three
// accumulators in turn where it would be, ChainCfg).  The LDS-tiled kernel at these sizes pays a barrier and
// a memory round trip per K slice, a second launch to sum its K ranges, and
// 64 x 64 tiles of which a narrow problem fills a quarter or less.  Measured
// per call on MI355X, tiled -> direct: FP64 256^3 12.2 -> 5.6 us, FP64 64 x
// 676 x 676 13.1 -> 7.6, FP32 240^3 10.1 -> 5.2, FP32 144 x 2500 x 2500 with
// runs of 50 48 -> 33, 400 dot products of 5184 167 -> 21, FP64 16 x 675840 x
// 64 132 -> 108.  Sixteen waves per tile were
// slower than four on all but the dot products; 64 x 64 wave tiles (one wave
// per SIMD) lose to the tiled kernel wherever they beat 32 x 32.
#include "launch.hpp"
#include "device.hpp"

namespace famlies {

template <typename T>
struct Mfma16;
template <>
struct Mfma16<double> {  // v_mfma_f64_16x16x4_f64
  using Acc = f64x4;
  __device__ __forceinline__ static Acc mma(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ __forceinline__ static int row(int l, int r) { return (l / 16) + 4 * r; }
};
template <>
struct Mfma16<float> {  // v_mfma_f32_16x16x4_f32
  using Acc = f32x4;
  __device__ __forceinline__ static Acc mma(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ __forceinline__ static int row(int l, int r) { return 4 * (l / 16) + r; }
};

// One operand of a wave: NBK blocks of 16 rows; lane l holds row l % 16 of
// each block and, per K step of 4 U indices, the U consecutive ones of group
// l / 16 (U elements are 16 bytes).  VEC: those U elements are consecutive
// in memory and are read with one load (at element alignment); otherwise one
// load per element.  D steps in flight, one register slot each.
template <typename T, int NBK, bool VEC, int D>
struct DirectOperand {
  static constexpr int U = 16 / (int)sizeof(T);
  static constexpr int NK = VEC ? 1 : U;  // contracted offsets per step
  typedef T vec_t __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
  typedef uint32_t off_t __attribute__((ext_vector_type(NK)));
  uint32_t mn[NBK];
  off_t ko[D];
  T v[D][NBK][U];

  __device__ __forceinline__ void init(const uint32_t* __restrict__ rows, const DirectPacked& p, int row0) {
#pragma unroll
    for (int i = 0; i < NBK; ++i) {
      const uint32_t row = (uint32_t)(row0 + 16 * i);
      mn[i] = p.plane ? (row >> p.shift) * p.tile + (row & ((1u << p.shift) - 1u)) * p.row : rows[row];
    }
  }
  // contracted offsets of this lane's run at k (a multiple of U)
  template <int S>
  __device__ __forceinline__ void fetch(const uint32_t* __restrict__ ks, int k) {
    ko[S] = *reinterpret_cast<const off_t*>(ks + k);
  }
  template <int S>
  __device__ __forceinline__ void load(const T* __restrict__ base) {
#pragma unroll
    for (int i = 0; i < NBK; ++i) {
      if constexpr (VEC) {
        const vec_t w = *reinterpret_cast<const __attribute__((address_space(1))) vec_t*>(global(at(base, mn[i] + ko[S][0])));
#pragma unroll
        for (int u = 0; u < U; ++u) v[S][i][u] = w[u];
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) v[S][i][u] = *global(at(base, mn[i] + ko[S][u]));
      }
    }
  }
};

// CH: accumulator sets a wave takes its K steps in, in turn.  Three where the
// planner needs the chains of additions short (DirectCfg); their registers
// cost a wave per SIMD in the FP64 tiles of four blocks, so not elsewhere.
template <typename T, int MB, int NB, bool XV, bool YV, int NW, int CH>
__global__ __launch_bounds__(64 * NW) void direct_contract(PlainArgs<uint32_t> a, int wk, DirectPacked xp,
                                                           DirectPacked yp) {
  using MF = Mfma16<T>;
  constexpr int U = 16 / (int)sizeof(T), KS = 4 * U, BM = 16 * MB, BN = 16 * NB;
  constexpr int D = 3;
  static_assert(CH == 1 || CH == D, "one chain, or one per register slot");
  __shared__ T part[NW * BM * BN];
  const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int g = lane / 16, r = lane % 16;
  const int ntiles = a.tiles_m * a.tiles_n;
  // units: (batch index, K range, tile), tile fastest; within, the side of
  // fewer tiles, so that the run of tiles of an XCD reads the long operand once
  const int units = ntiles * a.splits * a.L;  // at most 1e9 (the planner's limit)
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int unit = wk == 1 ? wg * NW + wave : wg;
  if (unit >= units) return;  // wk == 1 only: whole waves, and no barrier follows
  const int wki = wk == 1 ? 0 : wave;
  const int ls = unit / ntiles, o = unit - ls * ntiles;
  const int l = ls / a.splits, split = ls % a.splits;
  const bool n_first = a.tiles_n < a.tiles_m;
  const int fewer = n_first ? a.tiles_n : a.tiles_m, oq = o / fewer, rest = o - oq * fewer;
  const int pm = n_first ? oq : rest, pn = n_first ? rest : oq;
  const int t = pn * a.tiles_m + pm;  // blocks of partial sums: M fastest
  const int m0 = pm * BM, n0 = pn * BN;
  const T* X = static_cast<const T*>(a.x) + (xp.plane ? l * xp.plane : a.xl[l]);
  const T* Y = static_cast<const T*>(a.y) + (yp.plane ? l * yp.plane : a.yl[l]);
  const int kbeg = split * a.kchunk, kend = min(a.K, kbeg + a.kchunk);

  DirectOperand<T, MB, XV, D> gx;
  DirectOperand<T, NB, YV, D> gy;
  gx.init(a.xmn, xp, m0 + r);
  gy.init(a.ymn, yp, n0 + r);
  typename MF::Acc acc[CH][MB][NB];
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[c][i][j] = typename MF::Acc{};

  const int ns = (kend - kbeg + KS - 1) / KS;                // K steps of the unit
  const int n = ns > wki ? (ns - wki + wk - 1) / wk : 0;     // this wave's
  const int klast = kbeg + (wki + (n - 1) * wk) * KS;
  // first k of this lane's run in step `it` (clamped: loads past the last
  // step repeat it and are not used)
  auto kof = [&](int it) {
    const int k = kbeg + (wki + it * wk) * KS;
    return (k < klast ? k : klast) + g * U;
  };
  uint32_t vw[D];  // word of the void mask of this lane's run; its bits are picked at the step (not while loading)
  if (n > 0) {
    auto load = [&](auto sc, int it) {
      constexpr int S = decltype(sc)::value;
      vw[S] = *global(a.kvoid + (kof(it) >> 5));
      gx.template load<S>(X);
      gy.template load<S>(Y);
    };
    auto start = [&](auto sc) {
      constexpr int S = decltype(sc)::value;
      gx.template fetch<S>(a.xk, kof(S));
      gy.template fetch<S>(a.yk, kof(S));
      load(sc, S);
    };
    auto ahead = [&](auto sc) {
      constexpr int S = decltype(sc)::value;
      gx.template fetch<S>(a.xk, kof(S + D));
      gy.template fetch<S>(a.yk, kof(S + D));
    };
    start(std::integral_constant<int, 0>{});
    start(std::integral_constant<int, 1>{});
    start(std::integral_constant<int, 2>{});
    ahead(std::integral_constant<int, 0>{});
    ahead(std::integral_constant<int, 1>{});
    ahead(std::integral_constant<int, 2>{});
    auto step = [&](auto sc, int it) {
      constexpr int S = decltype(sc)::value;
      const uint32_t voids = (vw[S] >> (kof(it) & 31)) & ((1u << U) - 1u);
      if (__builtin_amdgcn_ballot_w64(voids != 0)) {
        // entries that do not count: zero in both operands (an Inf or NaN
        // there must not reach the sum)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = !((voids >> u) & 1u);
#pragma unroll
          for (int i = 0; i < MB; ++i) gx.v[S][i][u] = in ? gx.v[S][i][u] : T(0);
#pragma unroll
          for (int j = 0; j < NB; ++j) gy.v[S][j][u] = in ? gy.v[S][j][u] : T(0);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[S % CH][i][j] = MF::mma(gx.v[S][i][u], gy.v[S][j][u], acc[S % CH][i][j]);
      load(sc, it + D);
      gx.template fetch<S>(a.xk, kof(it + 2 * D));
      gy.template fetch<S>(a.yk, kof(it + 2 * D));
    };
    for (int it = 0; it < n; it += D) {
      step(std::integral_constant<int, 0>{}, it);
      if (it + 1 < n) step(std::integral_constant<int, 1>{}, it + 1);
      if (it + 2 < n) step(std::integral_constant<int, 2>{}, it + 2);
    }
  }

#pragma unroll
  for (int c = 1; c < CH; ++c)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[0][i][j] += acc[c][i][j];
  T* __restrict__ C = static_cast<T*>(a.c) + a.cl[l];
  const T al = static_cast<T>(a.alpha), be = static_cast<T>(a.beta);
  T* __restrict__ W = a.splits > 1 ? static_cast<T*>(a.work) + ((size_t)split * ntiles + t) * (size_t)(BM * BN) : nullptr;
  if (wk == 1) {
    // reads (indexing vectors, C) before the first write
    uint32_t cmv[MB][4], cnv[NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) cmv[i][e] = a.cm[m0 + 16 * i + MF::row(lane, e)];
#pragma unroll
    for (int j = 0; j < NB; ++j) cnv[j] = a.cn[n0 + 16 * j + r];
    T cv[MB][NB][4];
    if (be != T(0)) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) cv[i][j][e] = *global(at(C, cmv[i][e] + cnv[j]));
    }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = m0 + 16 * i + MF::row(lane, e), nn = n0 + 16 * j + r;
          if (m < a.M && nn < a.N) {
            T v = al * acc[0][i][j][e];
            if (be != T(0)) v += be * cv[i][j][e];
            *global(at(C, cmv[i][e] + cnv[j])) = v;
          }
        }
    return;
  }
  // partial tiles of the waves, summed in wave order
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        part[wave * (BM * BN) + (16 * i + MF::row(lane, e)) * BN + 16 * j + r] = acc[0][i][j][e];
  __syncthreads();
  constexpr int PER = (BM * BN + 64 * NW - 1) / (64 * NW);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int e = tid + q * 64 * NW;
    if ((BM * BN) % (64 * NW) != 0 && e >= BM * BN) break;
    const int mi = e / BN, ni = e % BN, m = m0 + mi, nn = n0 + ni;
    T s = part[e];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += part[w * (BM * BN) + e];
    if (W) {
      *global(W + e) = s;
    } else if (m < a.M && nn < a.N) {
      auto* cp = global(at(C, a.cm[m] + a.cn[nn]));
      T v = al * s;
      if (be != T(0)) v += be * *cp;
      *cp = v;
    }
  }
}

template <typename T, int MB, int NB, bool XV, bool YV>
static hipError_t launch_nw(const PlainArgs<uint32_t>& a, const DirectCfg& d, const DirectPacked& xp, const DirectPacked& yp,
                            hipStream_t s) {
  const int64_t units = (int64_t)a.tiles_m * a.tiles_n * a.splits * a.L;
  const int grid = (int)(d.wk == 1 ? (units + 3) / 4 : units);
  if (d.chains == 3)
    hipLaunchKernelGGL((direct_contract<T, MB, NB, XV, YV, 4, 3>), dim3(grid), dim3(256), 0, s, a, d.wk, xp, yp);
  else
    hipLaunchKernelGGL((direct_contract<T, MB, NB, XV, YV, 4, 1>), dim3(grid), dim3(256), 0, s, a, d.wk, xp, yp);
  return hipGetLastError();
}

template <typename T, int MB, int NB>
static hipError_t launch_modes(const PlainArgs<uint32_t>& a, const DirectCfg& d, bool xv, bool yv, const DirectPacked& xp,
                               const DirectPacked& yp, hipStream_t s) {
  if (xv && yv) return launch_nw<T, MB, NB, true, true>(a, d, xp, yp, s);
  if (xv) return launch_nw<T, MB, NB, true, false>(a, d, xp, yp, s);
  if (yv) return launch_nw<T, MB, NB, false, true>(a, d, xp, yp, s);
  return launch_nw<T, MB, NB, false, false>(a, d, xp, yp, s);
}

template <typename T>
static hipError_t launch_direct_t(const PlainArgs<uint32_t>& a, const DirectCfg& d, bool xv, bool yv, const DirectPacked& xp,
                                  const DirectPacked& yp, hipStream_t s) {
  if (d.bm == 16 && d.bn == 16) return launch_modes<T, 1, 1>(a, d, xv, yv, xp, yp, s);
  if (d.bm == 32 && d.bn == 32) return launch_modes<T, 2, 2>(a, d, xv, yv, xp, yp, s);
  if (d.bm == 16 && d.bn == 64) return launch_modes<T, 1, 4>(a, d, xv, yv, xp, yp, s);
  if (d.bm == 64 && d.bn == 16) return launch_modes<T, 4, 1>(a, d, xv, yv, xp, yp, s);
  return hipErrorInvalidValue;
}

hipError_t launch_direct(int dtype, const PlainArgs<uint32_t>& a, const DirectCfg& d, bool xv, bool yv,
                         const DirectPacked& xp, const DirectPacked& yp, hipStream_t s) {
  return dtype == FAMLIES_F64 ? launch_direct_t<double>(a, d, xv, yv, xp, yp, s)
                              : launch_direct_t<float>(a, d, xv, yv, xp, yp, s);
}

}  // namespace famlies
