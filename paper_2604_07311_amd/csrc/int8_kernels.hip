// FP64 contraction emulated on 8-bit integer products (INT8 MFMA).
//
// A new precision placed inside the GEMM the way the paper places
// transformations in the packing step ("Supporting new and mixed
// precisions"; Introduction, "Challenges"): the operands are sliced while
// they are packed, and the GEMM runs on the slices.  The slicing is the
// error-free splitting of Ozaki, Ogita, Oishi and Rump in the integer form of
// Ootomo, Ozaki and Yokota:
//   1. every row of X's GEMM view (and column of Y's) is scaled by a power
//      of two, 2^-e with e the smallest integer such that
//      max|v| <= (127/128) 2^e;
//   2. each scaled value is cut into S signed digits by exact rounding to
//      nearest (d_t = rint(2^7 r), r <- 2^7 r - d_t; |d_1| <= 127 since the
//      scale keeps |v| <= 127/128, |d_t| <= 64 after it);
//   3. for every digit pair (t, u) with t + u <= S + 1 the digit products are
//      summed exactly in int32 on v_mfma_i32_32x32x32_i8, pairs of one
//      diagonal t + u into one accumulator (exact while the sum stays below
//      2^31, so long K runs in chunks flushed to FP64);
//   4. C = alpha 2^(ex+ey) sum_d 2^-7d S_d + beta C, in FP64.
//
// int8_rowmax, int8_digits: the row maxima -> exponents, then the digits ->
//   digit planes, for both operands in one launch each.  Planes are stored
//   tile-major, [l][t][tile of 64 rows][64-k block][16-k chunk][row][16 k]
//   (int8), which is at once the LDS image int8_gemm multiplies from: a wave
//   moves 1 KB straight into LDS per instruction and every fragment read (32
//   rows of one chunk) is 512 consecutive bytes.
// int8_gemm: one workgroup per 128 x 128 (up to six slices) or 128 x 64 tile
//   of C, waves of 64 x 32; the S planes of X and Y for 32 contracted indices
//   sit in one of two or three LDS buffers (the next one or two steps' are
//   loaded meanwhile) and every wave keeps one int32 accumulator set per digit
//   diagonal (S sets of 32 registers).  S is 3 to 7.
#include "launch.hpp"
#include "runtime.hpp"
#include "tile.hpp"

namespace famlies {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int kI8K = 64;          // contracted indices of a plane block
constexpr int kI8Rows = 64;       // rows of a plane tile, and of a slicing workgroup
constexpr int kI8Chunk = 16;      // contracted indices (bytes) of a chunk
constexpr int kI8Block = kI8K * kI8Rows;  // bytes of one block of one plane
constexpr int kI8BM = 128;
constexpr int kExpNonFinite = 0x7fffffff;  // exponent of a row holding Inf or NaN

// K slices whose digit products stay exact in int32: one diagonal sums at
// most S pairs of products |d_t d_u| <= 127^2 per contracted index.
constexpr int int8_chunk_slices(int S) { return (int)(2147483647LL / (64LL * S * 127 * 127)); }

template <typename OffT>
struct SliceArgs {
  const void* src;      // operand base (its lowest element in the uint32 form)
  const OffT* rows;     // row offsets (R valid)
  const OffT* ks;       // contracted offsets (K valid)
  const int64_t* bl;    // batch offsets in elements (L)
  const uint32_t* kvoid;  // void mask of the contracted order (null: nothing to leave out below K)
  int8_t* planes;       // [L][S][tiles][nkb][4 chunks][64 rows][16]
  int32_t* exps;        // [L][tiles * 64]
  double* pmax;         // partial row maxima [L][ksplit][tiles * 64] (+Inf: a non-finite value)
  int32_t R, K, L;
  int32_t tiles, nkb;   // tiles of 64 rows
  int32_t ksplit, kbper;  // K ranges per tile, 64-blocks per range
  int32_t grid() const { return L * tiles * ksplit; }
};

// ---------------------------------------------------------------- slicing
// Two kernels over (tile of 64 rows, K range) workgroups, X's first, then
// Y's, so that a long K spreads over many workgroups and small operands do
// not pay a launch each: int8_rowmax writes each range's row maxima,
// int8_digits reduces them for its rows (the first range's workgroup also
// writes the exponents) and cuts its range into digit planes.  The partial
// maxima are reduced in range order: no atomics, deterministic.  Both are
// bound by HBM: the operand is read twice and S bytes per element written.
//
// Operand read modes: lanes along rows (row-gathered), lanes along k with
// one load per element (K-gathered), or lanes along k with 16-byte loads of
// pairs (every aligned pair of the contracted order contiguous, at element
// alignment; W of the ladder v=96 o=24 took 440 us in the element mode).
constexpr int kSliceRows = 0, kSliceK = 1, kSliceKVec = 2;

// Step 1: the smallest e with m <= (127/128) 2^e (0 for m == 0), so that
// every scaled value's first digit rint(2^7 v) stays within [-127, 127].
__device__ __forceinline__ int slice_exponent(double m) {
  if (m == 0.0) return 0;
  int e;
  const double f = frexp(m, &e);
  return f <= 127.0 / 128.0 ? e : e + 1;
}

// One workgroup's view of a slicing job: 64 rows from row0, K blocks
// [kb0, kb1).  Thread layout: 16 elements each, 4 rows x 4 consecutive k
// (lanes along k, 16 lanes per row) or 1 row x 4 runs of 4 consecutive k
// (lanes along rows).
template <typename OffT, int MODE>
struct SliceTile {
  static constexpr bool KF = MODE != kSliceRows;
  const SliceArgs<OffT>& a;
  OffT* srow;  // LDS: the 64 row offsets
  OffT* sk;    // LDS: one block's 64 contracted offsets
  const double* base;
  int tid, l, tile, row0, kb0, kb1, kq, rg, rr, kg;
  __device__ SliceTile(const SliceArgs<OffT>& args, int block, OffT* sr, OffT* skk) : a(args), srow(sr), sk(skk) {
    tid = threadIdx.x;
    const int per_l = a.tiles * a.ksplit;
    l = block / per_l;
    const int w = block % per_l;
    tile = w / a.ksplit;
    row0 = tile * kI8Rows;
    kb0 = (w % a.ksplit) * a.kbper;
    kb1 = min(a.nkb, kb0 + a.kbper);
    base = static_cast<const double*>(a.src) + a.bl[l];
    kq = KF ? tid % 16 : 0;
    rg = KF ? tid / 16 : 0;
    rr = KF ? 0 : tid % 64;
    kg = KF ? 0 : tid / 64;
    if (tid < kI8Rows) srow[tid] = row0 + tid < a.R ? a.rows[row0 + tid] : (OffT)0;
  }
  __device__ int row_of(int j) const { return KF ? rg + 16 * j : rr; }
  __device__ int kin(int j) const { return KF ? 4 * kq : 4 * (kg + 4 * j); }  // first of 4 k's in the block
  // stage block kb's offsets in LDS (barriers on both sides)
  __device__ void stage_k(int kb) {
    __syncthreads();
    if (tid < kI8K) sk[tid] = kb * kI8K + tid < a.K ? a.ks[kb * kI8K + tid] : (OffT)0;
    __syncthreads();
  }
  // which of the 4 k's of group j do not count (bits)
  __device__ uint32_t voids(int kb, int j) const {
    const int k = kb * kI8K + kin(j);
    if (a.kvoid) return (a.kvoid[k >> 5] >> (k & 31)) & 15u;
    return k + 4 <= a.K ? 0u : k >= a.K ? 15u : (15u << (a.K - k)) & 15u;
  }
  __device__ void load(int kb, double (&v)[4][4]) const {
    uint32_t out = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = row_of(j), k0 = kin(j);
      const bool rok = row0 + r < a.R;
      const OffT ro = srow[r];
      if (!KF || j == 0) out = voids(kb, j);
      if constexpr (MODE == kSliceKVec) {
        typedef double f64x2 __attribute__((ext_vector_type(2), aligned(8)));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f64x2 w = *reinterpret_cast<const __attribute__((address_space(1))) f64x2*>(
            global(at(base, (OffT)(ro + sk[k0 + 2 * h]))));
          v[j][2 * h] = w[0];
          v[j][2 * h + 1] = w[1];
        }
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[j][c] = *global(at(base, (OffT)(ro + sk[k0 + c])));
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) v[j][c] = rok && !((out >> c) & 1u) ? v[j][c] : 0.0;
    }
  }
};

// Partial row maxima of one K range (+Inf marks a row holding Inf or NaN).
template <typename OffT, int MODE>
__device__ __forceinline__ void slice_rowmax(const SliceArgs<OffT>& a, int block, OffT* srow, OffT* sk,
                                             double (*smax)[kI8Rows]) {
  SliceTile<OffT, MODE> st(a, block, srow, sk);
  constexpr bool KF = SliceTile<OffT, MODE>::KF;
  double m[4] = {0.0, 0.0, 0.0, 0.0};
  for (int kb = st.kb0; kb < st.kb1; ++kb) {
    st.stage_k(kb);
    double v[4][4];
    st.load(kb, v);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double x = v[j][c];
        m[KF ? j : 0] = __builtin_isfinite(x) ? fmax(m[KF ? j : 0], fabs(x)) : __builtin_inf();
      }
  }
  const int64_t rows_pad = (int64_t)a.tiles * kI8Rows;
  double* out = a.pmax + ((int64_t)st.l * a.ksplit + st.kb0 / a.kbper) * rows_pad + st.row0;
  if constexpr (KF) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int sh = 1; sh < 16; sh <<= 1) m[j] = fmax(m[j], __shfl_xor(m[j], sh, 16));
      if (st.kq == 0) out[st.row_of(j)] = m[j];
    }
  } else {
    smax[st.kg][st.rr] = m[0];
    __syncthreads();
    if (st.tid < kI8Rows)
      out[st.tid] = fmax(fmax(smax[0][st.tid], smax[1][st.tid]), fmax(smax[2][st.tid], smax[3][st.tid]));
  }
}

template <typename OffT, int MX, int MY>
__global__ __launch_bounds__(kThreads) void int8_rowmax(SliceArgs<OffT> x, SliceArgs<OffT> y, int xgrid) {
  __shared__ OffT srow[kI8Rows], sk[kI8K];
  __shared__ double smax[4][kI8Rows];
  if ((int)blockIdx.x < xgrid)
    slice_rowmax<OffT, MX>(x, (int)blockIdx.x, srow, sk, smax);
  else
    slice_rowmax<OffT, MY>(y, (int)blockIdx.x - xgrid, srow, sk, smax);
}

// Exponents from the partial maxima, then the digits of one K range (step 2:
// exact rounding to nearest), staged in LDS as [chunk][row][16] and written
// out as the planes hold them.
constexpr int kI8DigPitch = kI8Rows * kI8Chunk + 16;  // bytes between chunks: spreads the stores' banks
template <typename OffT, int S, int MODE>
__device__ __forceinline__ void slice_digits(const SliceArgs<OffT>& a, int block, unsigned char* dig, OffT* srow,
                                             OffT* sk, int* sexp) {
  SliceTile<OffT, MODE> st(a, block, srow, sk);
  const int tid = st.tid;
  const int64_t rows_pad = (int64_t)a.tiles * kI8Rows;
  if (tid < kI8Rows) {
    const double* pm = a.pmax + (int64_t)st.l * a.ksplit * rows_pad + st.row0 + tid;
    double m = 0.0;
    for (int q = 0; q < a.ksplit; ++q) m = fmax(m, pm[q * rows_pad]);
    const int e = m == __builtin_inf() ? kExpNonFinite : slice_exponent(m);
    sexp[tid] = e;
    if (st.kb0 == 0) a.exps[(int64_t)st.l * rows_pad + st.row0 + tid] = e;
  }
  for (int kb = st.kb0; kb < st.kb1; ++kb) {
    st.stage_k(kb);  // its first barrier also orders sexp and the previous block's dig reads
    double v[4][4];
    st.load(kb, v);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = st.row_of(j);
      const int e = sexp[r];
      uint32_t packed[S];
#pragma unroll
      for (int t = 0; t < S; ++t) packed[t] = 0u;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        double rem = e == kExpNonFinite ? 0.0 : ldexp(v[j][c], -e);
#pragma unroll
        for (int t = 0; t < S; ++t) {
          const double y = rem * 128.0;  // exact
          const double q = rint(y);      // nearest, ties to even
          rem = y - q;                   // exact
          packed[t] |= ((uint32_t)(int)q & 0xffu) << (8 * c);
        }
      }
      const int k0 = st.kin(j);
#pragma unroll
      for (int t = 0; t < S; ++t)
        *reinterpret_cast<uint32_t*>(&dig[(t * 4 + k0 / kI8Chunk) * kI8DigPitch + r * kI8Chunk + k0 % kI8Chunk]) =
            packed[t];
    }
    __syncthreads();
    // 4 chunks x 64 rows x 16 bytes per plane, one 16-byte piece per thread
    const int cc = tid / kI8Rows, cr = tid % kI8Rows;
#pragma unroll
    for (int t = 0; t < S; ++t) {
      const i32x4 w = *reinterpret_cast<const i32x4*>(&dig[(t * 4 + cc) * kI8DigPitch + cr * kI8Chunk]);
      const int64_t blk = (((int64_t)st.l * S + t) * a.tiles + st.tile) * a.nkb + kb;
      *global(reinterpret_cast<i32x4*>(a.planes + blk * kI8Block + tid * 16)) = w;
    }
  }
}

template <typename OffT, int S, int MX, int MY>
__global__ __launch_bounds__(kThreads) void int8_digits(SliceArgs<OffT> x, SliceArgs<OffT> y, int xgrid) {
  __shared__ __attribute__((aligned(16))) unsigned char dig[S * 4 * kI8DigPitch];
  __shared__ OffT srow[kI8Rows], sk[kI8K];
  __shared__ int sexp[kI8Rows];
  if ((int)blockIdx.x < xgrid)
    slice_digits<OffT, S, MX>(x, (int)blockIdx.x, dig, srow, sk, sexp);
  else
    slice_digits<OffT, S, MY>(y, (int)blockIdx.x - xgrid, dig, srow, sk, sexp);
}

// K ranges per row block: enough workgroups to fill the chip (about 2048)
// with ranges of whole 64-blocks.
__host__ __device__ inline void slice_split(int64_t rblocks_l, int nkb, int* ksplit, int* kbper) {
  int64_t want = (2048 + rblocks_l - 1) / rblocks_l;
  if (want < 1) want = 1;
  if (want > nkb) want = nkb;
  *kbper = (int)((nkb + want - 1) / want);
  *ksplit = (nkb + *kbper - 1) / *kbper;
}

// ---------------------------------------------------------------- GEMM
template <typename OffT>
struct Int8GemmArgs {
  PlainArgs<OffT> p;         // C, its indexing vectors, sizes, alpha, beta
  const int8_t* xp;          // X digit planes (tiles of 64 rows, an even number)
  const int8_t* yp;          // Y digit planes
  const int32_t* xe;         // X row exponents
  const int32_t* ye;         // Y column exponents
  int32_t xt, yt;            // plane tiles of X, Y per batch index
  int32_t nkb;               // blocks of the planes
  int32_t kb0, kb1;          // the blocks this launch sums (at most one exact int32 chunk)
  int32_t kbper;             // blocks per K range (p.splits ranges; > 1: partial sums to p.work)
};

// 32 x 32 accumulator layout of the 32x32 MFMA shapes: element r of lane l
// is row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
__device__ __forceinline__ int acc_row(int l, int r) { return 8 * (r / 4) + 4 * (l / 32) + (r % 4); }

// Contracted indices of a step: two chunks.  One step of one plane and tile
// is 2 KB, of which a wave moves 1 KB (64 lanes x 16 bytes) per instruction.
constexpr int kI8Step = 32;
constexpr int kI8StepBytes = kI8Step * kI8Rows;
constexpr int kI8Piece = 1024;

template <int BN>
constexpr int int8_waves() { return 2 * (BN / 32); }

// What bounds it: with 128 x 64 tiles (four waves) the planes' L2 traffic,
// 27 bytes per clock and CU where L2 gives about 15 (measured 9 TB/s over the
// chip); 128 x 128 tiles (eight waves, two per SIMD, S sets of 32 of their
// 256 registers) take two thirds of it per product.  The planes go from
// global memory straight into LDS, which frees the registers the second wave
// needs: six slices, ladder o=24 v=96, matrix cores 67 % busy, 80 % L2 hits.
// Seven slices' sets do not fit two waves and stay at 128 x 64: one
// wave per SIMD, with nothing else to run while it waits.
//
// NST: buffers.  With two, a step's loads have the time of one step before
// they are needed, which at one wave per SIMD is too little: seven slices,
// ring o=31 v=93, 901 us a launch, with three 695 (with the planes staged
// through registers 818).  Fewer slices gain from three on long K (three
// slices, 700 x 3100 x 9000: 408 -> 345 us a call; six, ring o=23 v=71: 130 ->
// 122) and lose up to 3 % on short K, where the two steps loaded past the last
// count (ten steps).
template <typename OffT, int S, int BN, int NST>
__global__ __launch_bounds__(64 * int8_waves<BN>(), int8_waves<BN>() / 4) void int8_gemm(Int8GemmArgs<OffT> g) {
  constexpr int NW = int8_waves<BN>();
  constexpr int TX = kI8BM / kI8Rows, TY = BN / kI8Rows;     // plane tiles per C tile
  constexpr int PLANE = (TX + TY) * kI8StepBytes;            // LDS bytes per plane and step
  constexpr int PIECES = PLANE / kI8Piece;                   // per plane
  // one array per buffer: the loads into one then do not alias the reads of
  // the other, so nothing waits for them before the step's end
  __shared__ __attribute__((aligned(1024))) unsigned char buf0[S * PLANE];
  __shared__ __attribute__((aligned(1024))) unsigned char buf1[S * PLANE];
  __shared__ __attribute__((aligned(1024))) unsigned char buf2[NST == 3 ? S * PLANE : 16];
  const PlainArgs<OffT>& a = g.p;
  const int tid = threadIdx.x, lane = tid % 64, wave = scalar(tid / 64);
  const int wm = wave % 2, wn = wave / 2;  // wave tile: rows 64 wm .., columns 32 wn ..
  const int ntiles = a.tiles_m * a.tiles_n;
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int ls = scalar(lid / ntiles), t = lid - ls * ntiles;
  const int l = scalar(ls / a.splits), split = ls - l * a.splits;
  const int pn = scalar(t / a.tiles_m), pm = t - pn * a.tiles_m;  // M fastest: neighbours share Y's panel
  const int64_t tstride = (int64_t)g.nkb * kI8Block;         // between tiles of a plane
  constexpr int kSteps = kI8K / kI8Step;
  const int st0 = kSteps * (g.kb0 + split * g.kbper);
  const int st1 = kSteps * min(g.kb1, g.kb0 + (split + 1) * g.kbper);
  // loads of step st: piece q = wave + i NW of the S * PIECES pieces; within a
  // plane pieces run tile by tile (X's, then Y's), two chunks each.  A Y tile
  // past the last re-reads the last (its columns are not stored).
  // With three buffers steps past the last re-read it and every wave issues
  // PER loads (the last piece again), so that a count of them is a wait.
  constexpr int PER = (S * PIECES + NW - 1) / NW;
  auto fetch = [&](unsigned char* buf, int st) {
    if constexpr (NST == 3) st = st < st1 ? st : st1 - 1;
    const int64_t in = (int64_t)(st / kSteps) * kI8Block + (st % kSteps) * kI8StepBytes + lane * 16;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      int q = wave + i * NW;
      if constexpr (NST == 3)
        q = min(q, S * PIECES - 1);
      else if ((S * PIECES) % NW != 0 && q >= S * PIECES)
        break;
      const int t2 = q / PIECES, piece = q % PIECES, tl = piece / 2, half = piece % 2;
      const int8_t* src;
      if (tl < TX)
        src = g.xp + (((int64_t)l * S + t2) * g.xt + pm * TX + tl) * tstride;
      else
        src = g.yp + (((int64_t)l * S + t2) * g.yt + min(pn * TY + tl - TX, g.yt - 1)) * tstride;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(src + in + half * kI8Piece),
          (__attribute__((address_space(3))) void*)(buf + t2 * PLANE + piece * kI8Piece), 16, 0, 0);
    }
  };
  i32x16 acc[S][2];
#pragma unroll
  for (int d = 0; d < S; ++d)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[d][b][r] = 0;
  const int fr = lane % 32, fc = (lane / 32) * kI8Piece;  // operand fragment: row / column, chunk
  auto multiply = [&](const unsigned char* buf) {
    const unsigned char* bx = buf + wm * kI8StepBytes + fc + fr * kI8Chunk;
    const unsigned char* by = buf + (TX + wn / 2) * kI8StepBytes + fc + ((wn % 2) * 32 + fr) * kI8Chunk;
    i32x4 yf[S];
#pragma unroll
    for (int u = 0; u < S; ++u) yf[u] = *reinterpret_cast<const i32x4*>(by + u * PLANE);
#pragma unroll
    for (int t2 = 0; t2 < S; ++t2) {
      const i32x4 x0 = *reinterpret_cast<const i32x4*>(bx + t2 * PLANE);
      const i32x4 x1 = *reinterpret_cast<const i32x4*>(bx + t2 * PLANE + 32 * kI8Chunk);
      // pairs (t2, u) with t2 + u <= S - 1 (0-based digits): diagonal d = t2 + u
#pragma unroll
      for (int u = 0; u + t2 < S; ++u) {
        acc[t2 + u][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x0, yf[u], acc[t2 + u][0], 0, 0, 0);
        acc[t2 + u][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x1, yf[u], acc[t2 + u][1], 0, 0, 0);
      }
    }
  };
  if constexpr (NST == 2) {
    // Steps alternate between the buffers: load the next step into the other
    // one, multiply this one, wait for the loads, barrier (every wave is then
    // done with this buffer and sees the other).
    auto step = [&](unsigned char* cur, unsigned char* nxt, int st) {
      if (st + 1 < st1) fetch(nxt, st + 1);
      multiply(cur);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
    };
    if (st0 < st1) {
      fetch(buf0, st0);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      for (int st = st0; st < st1; st += 2) {
        step(buf0, buf1, st);
        if (st + 1 < st1) step(buf1, buf0, st + 1);
      }
    }
  } else if (st0 < st1) {
    // Steps go round the buffers: load the step after the next into the one
    // that the step before this left, multiply this one, wait for the next
    // step's loads (all but the newest PER; s_waitcnt: vmcnt in bits 3:0 and
    // 15:14, expcnt 6:4, lgkmcnt 11:8), barrier.
    auto join = [&](auto keepc) {
      constexpr int keep = decltype(keepc)::value;
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt((keep & 15) | ((keep >> 4) << 14) | (7 << 4));
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    auto step = [&](unsigned char* cur, unsigned char* free, int st) {
      fetch(free, st + 2);
      multiply(cur);
      join(std::integral_constant<int, PER>{});
      return st + 1 < st1;
    };
    fetch(buf0, st0);
    fetch(buf1, st0 + 1);
    join(std::integral_constant<int, PER>{});
    // two rounds per turn: at the head of a loop the compiler waits for every
    // load before it reads LDS
    for (int st = st0;; st += 6)
      if (!step(buf0, buf2, st) || !step(buf1, buf0, st + 1) || !step(buf2, buf1, st + 2) ||
          !step(buf0, buf2, st + 3) || !step(buf1, buf0, st + 4) || !step(buf2, buf1, st + 5))
        break;
    __builtin_amdgcn_s_waitcnt(0);  // the loads past the last step have landed
  }
  // C update from the exact int32 sums of this launch's K chunk:
  // C = alpha 2^(ex+ey) sum_d 2^-7d S_d + beta C, the sum over diagonals from
  // the lightest to the heaviest (a later chunk runs with beta = 1); with K
  // ranges, 2^(ex+ey) sum_d 2^-7d S_d of this range to its block of `work`.
  const int ncol = pn * BN + wn * 32 + fr;
  if (ncol >= a.N) return;
  const int ey = g.ye[(int64_t)l * g.yt * kI8Rows + ncol];
  const int mrow0 = pm * kI8BM + wm * 64;
  const int32_t* xe = g.xe + (int64_t)l * g.xt * kI8Rows;
  double* C = static_cast<double*>(a.c) + a.cl[l];
  const OffT cn = a.cn[ncol];
  double* W = a.splits > 1 ? static_cast<double*>(a.work) +
                                 ((size_t)split * ntiles + t) * (size_t)(kI8BM * BN) + (wm * 64) * BN + wn * 32 + fr
                           : nullptr;
  // eight rows at a time: their exponents, offsets and C values are read
  // together (rows past the edge read row 0 and are not stored)
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r0 = 0; r0 < 16; r0 += 8) {
      int ex[8];
      OffT co[8];
      double c[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int m = mrow0 + 32 * b + acc_row(lane, r0 + q), mc = m < a.M ? m : 0;
        ex[q] = xe[mc];
        co[q] = (OffT)(a.cm[mc] + cn);
      }
      if (!W && a.beta != 0.0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) c[q] = *global(at(C, co[q]));
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int mi = 32 * b + acc_row(lane, r0 + q);
        double v = 0.0;
#pragma unroll
        for (int d = S - 1; d >= 0; --d) v += ldexp((double)acc[d][b][r0 + q], -7 * (d + 2));
        v = (ex[q] == kExpNonFinite || ey == kExpNonFinite) ? __builtin_nan("") : ldexp(v, ex[q] + ey);
        if (mrow0 + mi >= a.M) continue;
        if (W) {
          *global(W + mi * BN) = v;
        } else {
          double out = a.alpha * v;
          if (a.beta != 0.0) out += a.beta * c[q];
          *global(at(C, co[q])) = out;
        }
      }
    }
}

// ---------------------------------------------------------------- launch
// Workspace layout of an INT8 plan: X planes | Y planes | X exponents |
// Y exponents | X partial maxima | Y partial maxima | partial sums (K ranges).
struct Int8Layout {
  int64_t nkb, tx, ty, xsplit, xper, ysplit, yper;
  int64_t xplanes, yplanes, xexp, yexp, xmax, ymax, part;  // bytes
  Int8Layout(int S, int64_t M, int64_t N, int64_t K, int64_t L, int bn, int splits) {
    nkb = (K + kI8K - 1) / kI8K;
    const int64_t tm = (M + kI8BM - 1) / kI8BM, tn = (N + bn - 1) / bn;
    tx = tm * (kI8BM / kI8Rows);
    ty = (N + kI8Rows - 1) / kI8Rows;
    int a, b;
    slice_split(L * tx, (int)nkb, &a, &b);
    xsplit = a;
    xper = b;
    slice_split(L * ty, (int)nkb, &a, &b);
    ysplit = a;
    yper = b;
    xplanes = L * S * tx * nkb * kI8Block;
    yplanes = L * S * ty * nkb * kI8Block;
    xexp = L * tx * kI8Rows * 4;
    yexp = L * ty * kI8Rows * 4;
    xmax = L * xsplit * tx * kI8Rows * 8;
    ymax = L * ysplit * ty * kI8Rows * 8;
    part = splits > 1 ? (int64_t)splits * tm * tn * kI8BM * bn * 8 : 0;
  }
  int64_t total() const { return xplanes + yplanes + xexp + yexp + xmax + ymax + part; }
};

template <typename OffT, int S, int MX, int MY>
static void launch_slice(const SliceArgs<OffT>& x, const SliceArgs<OffT>& y, hipStream_t s) {
  const dim3 grid(x.grid() + y.grid());
  hipLaunchKernelGGL((int8_rowmax<OffT, MX, MY>), grid, dim3(kThreads), 0, s, x, y, x.grid());
  hipLaunchKernelGGL((int8_digits<OffT, S, MX, MY>), grid, dim3(kThreads), 0, s, x, y, x.grid());
}

template <typename OffT, int S, int MX>
static void launch_slice_y(const SliceArgs<OffT>& x, const SliceArgs<OffT>& y, int ymode, hipStream_t s) {
  if (ymode == kSliceKVec)
    launch_slice<OffT, S, MX, kSliceKVec>(x, y, s);
  else if (ymode == kSliceK)
    launch_slice<OffT, S, MX, kSliceK>(x, y, s);
  else
    launch_slice<OffT, S, MX, kSliceRows>(x, y, s);
}

template <typename OffT, int S, int BN>
static hipError_t launch_gemm(const Int8GemmArgs<OffT>& g, hipStream_t s) {
  const int grid = g.p.L * g.p.tiles_m * g.p.tiles_n * g.p.splits;
  const int steps = (g.p.splits > 1 ? g.kbper : g.kb1 - g.kb0) * (kI8K / kI8Step);  // of a workgroup
  if (S == 7 || steps >= 16)
    hipLaunchKernelGGL((int8_gemm<OffT, S, BN, 3>), dim3(grid), dim3(64 * int8_waves<BN>()), 0, s, g);
  else
    hipLaunchKernelGGL((int8_gemm<OffT, S, BN, S == 7 ? 3 : 2>), dim3(grid), dim3(64 * int8_waves<BN>()), 0, s, g);
  return hipGetLastError();
}

template <typename OffT, int S>
static hipError_t launch_int8_s(const PlainArgs<OffT>& a, int bn, int xmode, int ymode, const uint32_t* kvoid,
                                hipStream_t s) {
  const Int8Layout lay(S, a.M, a.N, a.K, a.L, bn, a.splits);
  const int nkb = (int)lay.nkb;
  int8_t* xp = static_cast<int8_t*>(a.work);
  int8_t* yp = xp + lay.xplanes;
  int32_t* xe = reinterpret_cast<int32_t*>(yp + lay.yplanes);
  int32_t* ye = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(xe) + lay.xexp);
  double* xm = reinterpret_cast<double*>(reinterpret_cast<char*>(ye) + lay.yexp);
  double* ym = reinterpret_cast<double*>(reinterpret_cast<char*>(xm) + lay.xmax);
  double* part = reinterpret_cast<double*>(reinterpret_cast<char*>(ym) + lay.ymax);
  const SliceArgs<OffT> sx{a.x, a.xmn, a.xk, a.xl, kvoid, xp, xe, xm, a.M, a.K, a.L, (int)lay.tx, nkb,
                           (int)lay.xsplit, (int)lay.xper};
  const SliceArgs<OffT> sy{a.y, a.ymn, a.yk, a.yl, kvoid, yp, ye, ym, a.N, a.K, a.L, (int)lay.ty, nkb,
                           (int)lay.ysplit, (int)lay.yper};
  if (xmode == kSliceKVec)
    launch_slice_y<OffT, S, kSliceKVec>(sx, sy, ymode, s);
  else if (xmode == kSliceK)
    launch_slice_y<OffT, S, kSliceK>(sx, sy, ymode, s);
  else
    launch_slice_y<OffT, S, kSliceRows>(sx, sy, ymode, s);
  // one launch per K chunk whose int32 sums stay exact, ordered on the stream
  // (K ranges only where one chunk holds all of K)
  const int chunk = int8_chunk_slices(S);
  for (int kb0 = 0; kb0 < nkb; kb0 += chunk) {
    const int kb1 = min(nkb, kb0 + chunk);
    Int8GemmArgs<OffT> g{a, xp, yp, xe, ye, (int)lay.tx, (int)lay.ty, nkb, kb0, kb1,
                         (kb1 - kb0 + a.splits - 1) / a.splits};
    g.p.work = part;
    if (kb0 > 0) g.p.beta = 1.0;  // later chunks add to C
    hipError_t e = hipErrorInvalidValue;
    if constexpr (S <= 6)
      if (bn == 128) e = launch_gemm<OffT, S, 128>(g, s);
    if (bn == 64) e = launch_gemm<OffT, S, 64>(g, s);
    if (e == hipSuccess && a.splits > 1) e = launch_splitk_reduce(FAMLIES_F64, false, g.p, kI8BM, bn, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

template <typename OffT>
static hipError_t launch_int8_t(const PlainArgs<OffT>& a, int slices, int bn, int xmode, int ymode,
                                const uint32_t* kvoid, hipStream_t s) {
  switch (slices) {
    case 3: return launch_int8_s<OffT, 3>(a, bn, xmode, ymode, kvoid, s);
    case 4: return launch_int8_s<OffT, 4>(a, bn, xmode, ymode, kvoid, s);
    case 5: return launch_int8_s<OffT, 5>(a, bn, xmode, ymode, kvoid, s);
    case 6: return launch_int8_s<OffT, 6>(a, bn, xmode, ymode, kvoid, s);
    case 7: return launch_int8_s<OffT, 7>(a, bn, xmode, ymode, kvoid, s);
    default: return hipErrorInvalidValue;
  }
}

// xmode / ymode: 0 row-gathered, 1 K-gathered, 2 K-gathered in 16-byte pairs
hipError_t launch_int8(const PlainArgs<uint32_t>& a, int slices, int bn, int xmode, int ymode, hipStream_t s) {
  return launch_int8_t(a, slices, bn, xmode, ymode, a.kvoid, s);
}
hipError_t launch_int8(const PlainArgs<int64_t>& a, int slices, int bn, int xmode, int ymode, hipStream_t s) {
  return launch_int8_t<int64_t>(a, slices, bn, xmode, ymode, nullptr, s);
}

size_t int8_work_bytes(int slices, int64_t M, int64_t N, int64_t K, int64_t L, int bn, int splits) {
  return (size_t)Int8Layout(slices, M, N, K, L, bn, splits).total();
}

// Exact int32 chunk of K, in contracted indices.
int64_t int8_exact_k(int slices) { return (int64_t)int8_chunk_slices(slices) * kI8K; }

}  // namespace famlies
