// Split-bf16 contractions of large operands through part planes.
//
// split_contract (split_kernels.hip) splits every operand element while it
// stages a tile, once per tile of the other side, and the conversions, the
// LDS stores and the staging registers share each CU with the matrix
// products.  Here both operands are split once, into NS bf16 part planes laid
// out as the GEMM's LDS image, and the GEMM moves them from global memory
// straight into LDS: no conversions, no staging registers, a 256 x 128 tile
// on eight waves (two per SIMD) with the same accumulators and epilogue (hh
// apart from the lower orders, FP64 combination, FP32 store).  The pass over
// the operands costs 4 + 2 NS bytes per element, so it pays where each
// element meets many tiles (the planner's estimate).  An operand that the
// caller keeps pre-packed is kept as its planes.
//
// Bound by the matrix cores together with the planes' way from the memory-side
// cache: ring o=48 v=192 bf16x3 has them 58 % busy while 25 GB pass L2 (33 %
// hits, 5.4 TB/s; the tile order of an XCD shares one operand's panel only);
// ring o=31 v=115 bf16x6 50 %, 58 % hits.  Measured against split_contract
// (pass included): ring o=48 v=192 bf16x3 5.58 -> 4.50 ms, bf16x6 9.25 -> 8.12
// ms; ring o=31 v=115 bf16x3 418 -> 316 us, bf16x6 (with folds) 719 -> 561 us;
// ladder o=36 v=110 bf16x3 1.82 -> 1.58 ms.  The pass alone: 128 us for the
// 340 MB operand of the large ring.
//
// bf16_planes writes [l][part][tile of 64 rows][64-k block][8-k chunk][row][8
// k]: a chunk of a tile is 1 KB, moved by one wave in one instruction, and a
// fragment read (32 rows of one chunk) is 512 consecutive bytes.
#include "device.hpp"
#include "runtime.hpp"

namespace famlies {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kPlRows = 64, kPlK = 64, kPlChunk = 1024;  // rows and k's of a block, bytes of a chunk
constexpr int kPlBlock = kPlRows * kPlK * 2;              // bytes of a block of one part
constexpr int kPlBM = 256, kPlBN = 128, kPlStepK = 32;

struct PlanesArgs {
  const void* src;       // operand base (its lowest element)
  const uint32_t* rows;  // row offsets (R valid)
  const uint32_t* ks;    // contracted offsets (padded)
  const int64_t* bl;     // batch offsets in elements (L)
  const uint32_t* kvoid;
  unsigned char* planes;
  int32_t R, L, tiles, nkb;  // tiles of 64 rows (padded to the GEMM's tile)
};

// One workgroup splits one block of 64 rows x 64 k's.  RUNS: lanes along k,
// 16-byte loads of four k's (element alignment); else lanes along k (KF) or
// rows with one load per element.  Bound by HBM (read once, 2 NS bytes per
// element written in whole KB).
template <int NS, bool KF, bool RUNS>
__device__ __forceinline__ void split_block(const PlanesArgs& a, int id, unsigned char* lds) {
  const int tid = threadIdx.x;
  const int kb = scalar(id % a.nkb), lt = scalar(id / a.nkb);
  const int tile = scalar(lt % a.tiles), l = scalar(lt / a.tiles);
  const int row0 = tile * kPlRows, k0 = kb * kPlK;
  const float* base = static_cast<const float*>(a.src) + a.bl[l];
  typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
  float v[4][4];
  int r[4], k[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {  // four runs of four k's
    r[j] = KF ? tid / 16 + 16 * j : tid % 64;
    k[j] = KF ? 4 * (tid % 16) : 4 * (tid / 64 + 4 * j);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool in = row0 + r[j] < a.R;
    const uint32_t ro = a.rows[in ? row0 + r[j] : 0];
    if constexpr (RUNS) {
      const f32x4u w = *reinterpret_cast<const __attribute__((address_space(1))) f32x4u*>(
          global(at(base, ro + a.ks[k0 + k[j]])));
#pragma unroll
      for (int c = 0; c < 4; ++c) v[j][c] = w[c];
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) v[j][c] = *global(at(base, ro + a.ks[k0 + k[j] + c]));
    }
    const uint32_t voids = in ? (a.kvoid[(k0 + k[j]) >> 5] >> ((k0 + k[j]) & 31)) & 15u : 15u;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[j][c] = (voids >> c) & 1u ? 0.0f : v[j][c];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f32x2 lo = {v[j][0], v[j][1]}, hi = {v[j][2], v[j][3]};
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const bf16x2 hl = __builtin_convertvector(lo, bf16x2), hh = __builtin_convertvector(hi, bf16x2);
      const u32x2 w = {__builtin_bit_cast(uint32_t, hl), __builtin_bit_cast(uint32_t, hh)};
      *reinterpret_cast<u32x2*>(lds + t * kPlBlock + (k[j] / 8) * kPlChunk + r[j] * 16 + (k[j] % 8) * 2) = w;
      if (t + 1 < NS) {
        lo = lo - __builtin_convertvector(hl, f32x2);
        hi = hi - __builtin_convertvector(hh, f32x2);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    unsigned char* dst = a.planes + ((((int64_t)l * NS + t) * a.tiles + tile) * a.nkb + kb) * (int64_t)kPlBlock;
#pragma unroll
    for (int q = 0; q < kPlBlock / (16 * kThreads); ++q) {
      const int o = (tid + q * kThreads) * 16;
      *global(reinterpret_cast<u32x4*>(dst + o)) = *reinterpret_cast<const u32x4*>(lds + t * kPlBlock + o);
    }
  }
}

// mode: 0 row-gathered, 1 K-gathered, 2 in 16-byte runs along K
template <int NS>
__global__ __launch_bounds__(kThreads) void bf16_planes(PlanesArgs a, int mode) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[NS * kPlBlock];
  if (mode == 2)
    split_block<NS, true, true>(a, (int)blockIdx.x, lds);
  else if (mode == 1)
    split_block<NS, true, false>(a, (int)blockIdx.x, lds);
  else
    split_block<NS, false, false>(a, (int)blockIdx.x, lds);
}

// LDS stages: three for two parts (two steps of loads in flight: a step is
// about 0.7 us of products), two for three parts (72 KB each).
template <int NS>
constexpr int kPlStages = NS == 2 ? 3 : 2;

static_assert(planes_turn(2) == 2 * kPlStages<2> && planes_turn(3) == 2 * kPlStages<3>, "steps of the K loop");
constexpr int kPlFold = kPlBM * kPlBN;  // elements of a workgroup's running sums

// FOLD: every `fold` steps (whole turns) the hh accumulators move into
// running sums in `sums`, so that no chain of additions is longer than the K
// ranges of the plan's split_contract launch (ChainCfg; bf16x6 with K in one
// chain had 1.5 to 2.2 times the error).  The addition is exact: its rounding
// error, taken by the two-sum of Knuth and Moeller, goes to the accumulators
// of the lower orders, which are of that size.  Two sets of accumulators and
// the fragments leave no registers for a third, and the workgroup's 128 KB go
// through L2, 13 us per fold and round (ring o=35 v=105, three ranges: 579 us
// in one chain, 619 with two folds).  K ranges in workgroups of their own with
// FP64 partial sums, as split_contract has them, move three times the bytes
// and fill their rounds less well: 723 us.
template <int NS, bool FOLD>
__global__ __launch_bounds__(512, 2) void planes_contract(PlainArgs<uint32_t> a, const unsigned char* xp,
                                                          const unsigned char* yp, int xt, int yt, int nkb, int fold,
                                                          float* sums) {
  constexpr int NW = 8, TX = kPlBM / kPlRows, TY = kPlBN / kPlRows;
  constexpr int STEP = kPlStepK / 8 * kPlChunk;  // bytes per tile of 64 rows and part
  constexpr int PART = (TX + TY) * STEP, STAGE = NS * PART;
  constexpr int PIECES = STAGE / kPlChunk, PER = PIECES / NW;  // 1 KB loads per step, per wave
  static_assert(PIECES % NW == 0, "pieces per wave");
  constexpr int NST = kPlStages<NS>;
  // one array per stage: loads into one do not alias reads of another
  __shared__ __attribute__((aligned(1024))) unsigned char s0[STAGE];
  __shared__ __attribute__((aligned(1024))) unsigned char s1[STAGE];
  __shared__ __attribute__((aligned(1024))) unsigned char s2[NST == 3 ? STAGE : 1024];
  const int tid = threadIdx.x, lane = tid % 64, wave = scalar(tid / 64);
  const int wm = wave % 4, wn = wave / 4;
  const int ntiles = a.tiles_m * a.tiles_n, nk = (a.K + kPlStepK - 1) / kPlStepK;
  int t, block = -1, st0 = 0, st1 = nk;  // t: tile over all batch planes
  if (a.rem > 0) {
    level_work(a, (int)blockIdx.x, nk, t, st0, st1, block);
  } else {
    t = scalar(xcd_remap(blockIdx.x, gridDim.x));
  }
  const int l = scalar(t / ntiles), tl = t - l * ntiles;
  const int pn = scalar(tl / a.tiles_m), pm = tl - pn * a.tiles_m;  // M fastest: neighbours share Y's panel
  const int m0 = pm * kPlBM, n0 = pn * kPlBN;
  // loads of step st (clamped: every step issues the same number, so a fixed
  // count of outstanding ones is the wait for the step before)
  auto fetch = [&](unsigned char* buf, int st) {
    st = st < st1 ? st : st1 - 1;
    const int64_t in = (int64_t)(st >> 1) * kPlBlock + (st & 1) * STEP + lane * 16;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int q = wave * PER + i;
      const int p = q / (PIECES / NS), piece = q % (PIECES / NS), tile = piece / (STEP / kPlChunk),
                chunk = piece % (STEP / kPlChunk);
      const bool x = tile < TX;
      const int64_t row = ((int64_t)l * NS + p) * (x ? xt : yt) + (x ? pm * TX + tile : pn * TY + tile - TX);
      const unsigned char* src = (x ? xp : yp) + row * nkb * kPlBlock;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + in + chunk * kPlChunk),
                                       (__attribute__((address_space(3))) void*)(buf + q * kPlChunk), 16, 0, 0);
    }
  };
  constexpr int NA = 2;  // hh; the lower orders together (as in split_contract)
  f32x16 acc[NA][2][2];
#pragma unroll
  for (int o = 0; o < NA; ++o)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[o][i][j] = f32x16{};
  const int g = lane / 32, r = lane % 32;
  // The fragments of half a step (16 contracted indices) and their products.
  // Two sets of them alternate, so that every read is issued a half step of
  // products before it is needed: with one set the eight waves, in step after
  // each barrier, waited for LDS together.
  struct Frag {
    bf16x8 x[NS][2], y[NS][2];
  };
  auto read = [&](Frag& f, const unsigned char* buf, int s) {
    const unsigned char* bx = buf + wm * STEP + g * kPlChunk + r * 16 + 2 * s * kPlChunk;
    const unsigned char* by = buf + (TX + wn) * STEP + g * kPlChunk + r * 16 + 2 * s * kPlChunk;
#pragma unroll
    for (int p = 0; p < NS; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f.x[p][i] = *reinterpret_cast<const bf16x8*>(bx + p * PART + i * 512);
        f.y[p][i] = *reinterpret_cast<const bf16x8*>(by + p * PART + i * 512);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](const Frag& f) {
#pragma unroll
    for (int pa = 0; pa < NS; ++pa)
#pragma unroll
      for (int pb = 0; pa + pb < NS; ++pb)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            f32x16& c = acc[pa + pb < NA ? pa + pb : NA - 1][i][j];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.x[pa][i], f.y[pb][j], c, 0, 0, 0);
          }
  };
  // Join of the waves in the middle of a step: the loads of the next step
  // have arrived (all but the `keep` newest), every wave has read this stage
  // and sees the next.  (s_waitcnt: vmcnt in bits 3:0 and 15:14, expcnt 6:4,
  // lgkmcnt 11:8.)
  auto join = [&](auto keepc) {
    constexpr int keep = decltype(keepc)::value;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((keep & 15) | ((keep >> 4) << 14) | (7 << 4));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4* S = reinterpret_cast<f32x4*>(sums + (size_t)blockIdx.x * kPlFold);
  // hh into the running sums: 0 the first time, 1 again, 2 at the end (the
  // total stays in the accumulators)
  auto fold_sums = [&](auto howc) {
    constexpr int how = decltype(howc)::value;
    // recomputed here: kept over the K loop, the addresses went to scratch
    uint32_t lane_at = (uint32_t)tid * 16u;
    asm volatile("" : "+v"(lane_at));
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          auto* sum = global(at(S + ((i * 2 + j) * 4 + q) * 512, lane_at));
          f32x4 v;
#pragma unroll
          for (int c = 0; c < 4; ++c) v[c] = acc[0][i][j][4 * q + c];
          if constexpr (how > 0) {
            const f32x4 h = *sum;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const float t = h[c] + v[c], b = t - h[c], e = (h[c] - (t - b)) + (v[c] - b);
              acc[1][i][j][4 * q + c] += __builtin_isfinite(t) ? e : 0.0f;
              v[c] = t;
            }
          }
          if constexpr (how < 2) *sum = v;
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[0][i][j][4 * q + c] = how < 2 ? 0.0f : v[c];
        }
  };
  if (st0 < st1) {
    bool folded = false;
    Frag fa, fb;
    fetch(s0, st0);
    fetch(s1, st0 + 1);
    if constexpr (NST == 3) fetch(s2, st0 + 2);
    join(std::integral_constant<int, (NST - 1) * PER>{});
    // step st: its second half's fragments, products of the first, join, the
    // loads of step st + NST into the stage just left, the next step's first
    // fragments, products of the second half; false after the last step
    auto step = [&](unsigned char* cur, const unsigned char* next, int st) {
      read(fb, cur, 1);
      multiply(fa);
      join(std::integral_constant<int, (NST - 2) * PER>{});
      fetch(cur, st + NST);
      read(fa, next, 0);
      multiply(fb);
      return st + 1 < st1;
    };
    // Several rounds of the stages per turn: at the head of a loop the
    // compiler waits for every load before it reads LDS.
    if constexpr (!FOLD) {  // (apart: with the loop below bf16x3 was 4 % slower)
      read(fa, s0, 0);
      if constexpr (NST == 3) {
        for (int st = st0;; st += 6)
          if (!step(s0, s1, st) || !step(s1, s2, st + 1) || !step(s2, s0, st + 2) || !step(s0, s1, st + 3) ||
              !step(s1, s2, st + 4) || !step(s2, s0, st + 5))
            break;
      } else {
        for (int st = st0;; st += 4)
          if (!step(s0, s1, st) || !step(s1, s0, st + 1) || !step(s0, s1, st + 2) || !step(s1, s0, st + 3)) break;
      }
    } else {
      // a turn; false after the last step
      auto turn = [&](int st) {
        if constexpr (NST == 3)
          return step(s0, s1, st) && step(s1, s2, st + 1) && step(s2, s0, st + 2) && step(s0, s1, st + 3) &&
                 step(s1, s2, st + 4) && step(s2, s0, st + 5);
        else
          return step(s0, s1, st) && step(s1, s0, st + 1) && step(s0, s1, st + 2) && step(s1, s0, st + 3);
      };
      // From fold to fold: the first fragments are read again after it, so that
      // none are held through it (with them, 48 registers went to scratch).
      int end = st0 + fold;
      for (int st = st0;;) {
        read(fa, s0, 0);
        bool more;
        do {
          more = turn(st);
          st += planes_turn(NS);
        } while (more && st < end);
        if (!more) break;
        if (end == st0 + fold)
          fold_sums(std::integral_constant<int, 0>{});
        else
          fold_sums(std::integral_constant<int, 1>{});
        end += fold;
      }
      folded = end > st0 + fold;
    }
    __builtin_amdgcn_s_waitcnt(0);  // the clamped loads of the last steps have landed
    if constexpr (FOLD)
      if (folded) fold_sums(std::integral_constant<int, 2>{});
  }
  auto total = [&](int i, int j, int e) { return (double)acc[1][i][j][e] + (double)acc[0][i][j][e]; };
  if (block >= 0) {
    double* W = static_cast<double*>(a.work) + (size_t)block * (size_t)(kPlBM * kPlBN) + (wm * 64) * kPlBN + wn * 64 + r;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          *global(W + (i * 32 + Mfma<float>::row(lane, e)) * kPlBN + j * 32) = total(i, j, e);
    return;
  }
  // eight rows of a column block at a time: offsets and C read together, past
  // the edge row 0 / column 0 (a valid element, never written back)
  float* C = static_cast<float*>(a.c) + a.cl[l];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = n0 + wn * 64 + j * 32 + r;
    const uint32_t cn = a.cn[n < a.N ? n : 0];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e0 = 0; e0 < 16; e0 += 8) {
        uint32_t co[8];
        float cv[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int m = m0 + wm * 64 + i * 32 + Mfma<float>::row(lane, e0 + q);
          co[q] = a.cm[m < a.M ? m : 0] + cn;
        }
        if (a.beta != 0.0) {
#pragma unroll
          for (int q = 0; q < 8; ++q) cv[q] = *global(at(C, co[q]));
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int m = m0 + wm * 64 + i * 32 + Mfma<float>::row(lane, e0 + q);
          if (m < a.M && n < a.N) {
            double v = a.alpha * total(i, j, e0 + q);
            if (a.beta != 0.0) v += a.beta * (double)cv[q];
            *global(at(C, co[q])) = (float)v;
          }
        }
      }
  }
}

// Workspace: X planes | Y planes | blocks of partial sums (levelled rounds) |
// running sums of every workgroup (folds).
struct PlanesLayout {
  int64_t nkb, xt, yt, x, y;
  PlanesLayout(int ns, int64_t M, int64_t N, int64_t K, int64_t L) {
    nkb = (K + kPlK - 1) / kPlK;
    xt = (M + kPlBM - 1) / kPlBM * (kPlBM / kPlRows);
    yt = (N + kPlBN - 1) / kPlBN * (kPlBN / kPlRows);
    x = L * ns * xt * nkb * kPlBlock;
    y = L * ns * yt * nkb * kPlBlock;
  }
};

// Workgroups of the launch.
static int64_t planes_grid(int64_t tiles, const LevelCfg& lv) {
  return lv.rem > 0 ? lv.head + (int64_t)lv.rem * (1 + lv.parts) : tiles;
}

size_t planes_work_bytes(int ns, int64_t M, int64_t N, int64_t K, int64_t L, const LevelCfg& lv, int fold) {
  const PlanesLayout lay(ns, M, N, K, L);
  const int64_t tiles = (lay.xt / (kPlBM / kPlRows)) * (lay.yt / (kPlBN / kPlRows)) * L;
  return (size_t)(lay.x + lay.y) + (size_t)lv.blocks() * (size_t)(kPlBM * kPlBN) * 8 +
         (fold > 0 ? (size_t)planes_grid(tiles, lv) * kPlFold * 4 : 0);
}

size_t planes_pack_bytes(int ns, int64_t M, int64_t N, int64_t K, int64_t L, bool x) {
  const PlanesLayout lay(ns, M, N, K, L);
  return (size_t)(x ? lay.x : lay.y);
}

template <int NS>
static hipError_t launch_planes_ns(const PlainArgs<uint32_t>& a0, int xmode, int ymode, bool pack_only, int fold,
                                   hipStream_t s) {
  PlainArgs<uint32_t> a = a0;
  const PlanesLayout lay(NS, a.M, a.N, a.K, a.L);
  unsigned char* xp = static_cast<unsigned char*>(a.work);
  unsigned char* yp = pack_only ? xp : xp + lay.x;  // packing writes one operand, to the start of `work`
  if (!pack_only) a.work = yp + lay.y;
  const PlanesArgs sx{a.x, a.xmn, a.xk, a.xl, a.kvoid, xp, a.M, a.L, (int)lay.xt, (int)lay.nkb};
  const PlanesArgs sy{a.y, a.ymn, a.yk, a.yl, a.kvoid, yp, a.N, a.L, (int)lay.yt, (int)lay.nkb};
  if (xmode != 3)
    hipLaunchKernelGGL(bf16_planes<NS>, dim3((int)((int64_t)sx.L * sx.tiles * sx.nkb)), dim3(kThreads), 0, s, sx,
                       xmode);
  if (ymode != 3)
    hipLaunchKernelGGL(bf16_planes<NS>, dim3((int)((int64_t)sy.L * sy.tiles * sy.nkb)), dim3(kThreads), 0, s, sy,
                       ymode);
  if (pack_only) return hipGetLastError();
  const unsigned char* xq = xmode == 3 ? static_cast<const unsigned char*>(a.x) : xp;
  const unsigned char* yq = ymode == 3 ? static_cast<const unsigned char*>(a.y) : yp;
  LevelCfg lv;
  lv.head = a.head;
  lv.rem = a.rem;
  lv.parts = a.lev_parts;
  const int grid = (int)planes_grid((int64_t)a.tiles_m * a.tiles_n * a.L, lv);
  float* sums = reinterpret_cast<float*>(static_cast<char*>(a.work) + (size_t)lv.blocks() * (kPlBM * kPlBN) * 8);
  if (fold > 0)
    hipLaunchKernelGGL((planes_contract<NS, true>), dim3(grid), dim3(512), 0, s, a, xq, yq, (int)lay.xt, (int)lay.yt,
                       (int)lay.nkb, fold, sums);
  else
    hipLaunchKernelGGL((planes_contract<NS, false>), dim3(grid), dim3(512), 0, s, a, xq, yq, (int)lay.xt,
                       (int)lay.yt, (int)lay.nkb, fold, sums);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && a.rem > 0) e = launch_level_reduce(FAMLIES_F32, true, a, kPlBM, s);
  return e;
}

// xmode / ymode: 0 row-gathered, 1 K-gathered, 2 in 16-byte runs along K, 3
// planes written before (a.x / a.y point to them)
hipError_t launch_planes(const PlainArgs<uint32_t>& a, int ns, int xmode, int ymode, int fold, hipStream_t s) {
  return ns == 2 ? launch_planes_ns<2>(a, xmode, ymode, false, fold, s)
                 : launch_planes_ns<3>(a, xmode, ymode, false, fold, s);
}

hipError_t launch_planes_pack(const PlainArgs<uint32_t>& a, int ns, bool x, int mode, hipStream_t s) {
  const int xm = x ? mode : 3, ym = x ? 3 : mode;
  return ns == 2 ? launch_planes_ns<2>(a, xm, ym, true, 0, s) : launch_planes_ns<3>(a, xm, ym, true, 0, s);
}

}  // namespace famlies
