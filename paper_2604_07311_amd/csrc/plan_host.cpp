// Host-side planning that touches no device: error state, tile choice,
// split-K settlement, the plan summary and the planner dry run
// (famlies_analyze).  Kept apart from the HIP sources so that it can be
// built and run on its own under the host sanitizers.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "famlies.h"
#include "internal.hpp"
#include "runtime.hpp"

namespace famlies {

static thread_local std::string g_err;
void set_error(const std::string& msg) { g_err = msg; }

famlies_status fail(famlies_status st, const std::string& msg) {
  g_err = msg;
  return st;
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Step a4: tile shape and split-K.  A tile-table entry for the problem's
// size class wins.  Otherwise a small cost model picks the tile edge (128 or
// 64) and the number of K slices: the workgroups are dealt to the CUs two at
// a time (two share a CU at half rate each; a lone one runs at about 0.65 of
// the CU), so the busiest CU's time is
//     pairs * 2w + (odd ? w / 0.65 : 0),  w = work of one workgroup,
// a 64-edge tile does its flops at about 0.75 of the 128-edge rate, and each
// extra K slice costs a pass over the split tiles' partial sums (at HBM
// rate, measured in the same units).  Splitting is either whole (every tile
// in K slices) or of the tail only: when the tiles fill some rounds of two
// workgroups per CU and part of one more, the whole rounds run unsplit and
// only the tiles of the last round are cut into K slices, so that round
// spreads over every CU instead of leaving most of them idle.  The model
// only ranks candidates; it is not a timing.
TileCfg choose_tiles(const famlies_handle_s* h, const Analysis& an, bool* from_table, bool use_table) {
  TileCfg t;
  const int bk = an.dtype == FAMLIES_F64 ? 8 : 32;
  t.bk = bk;
  if (from_table) *from_table = false;
  if (an.M == 0 || an.N == 0 || an.K == 0) return t;
  if (h && use_table && h->table.lookup_plain(an, &t)) {
    if (!t.planner()) {
      if (from_table) *from_table = true;
      return t;
    }
    t = TileCfg();
    t.bk = bk;
  }
  const int cus = h ? h->num_cus : 256;
  // CU throughput in flop/s and HBM bandwidth in bytes/s (MI355X-class)
  const double cu_rate = (an.dtype == FAMLIES_F64 ? 78.6e12 : 157.3e12) / 256.0;
  const double hbm = 8.0e12 * cus / 256.0;
  const double es = an.esize;
  double best = 1e300;
  TileCfg pick = t;
  for (int bt : {128, 64}) {
    const int64_t tiles = ceil_div(an.M, bt) * ceil_div(an.N, bt) * an.L;
    const double eff = bt == 128 ? 1.0 : 0.75;
    for (int split : {1, 2, 3, 4, 6, 8, 12, 16}) {
      if (split > 1 && (an.L > 1 || an.K / split < 2 * bk)) continue;
      const int64_t units = tiles * split;
      const int64_t q = ceil_div(units, cus);  // workgroups on the busiest CU
      const double w = 2.0 * bt * bt * ((double)an.K / split) / (cu_rate * eff);
      double time = (double)(q / 2) * 2.0 * w + (q % 2 ? w / 0.65 : 0.0);
      if (split > 1) time += (double)split * an.M * an.N * es * 2.0 / hbm + 4e-6;
      if (time < best * 0.9) {  // prefer fewer slices / larger tiles unless clearly faster
        best = time;
        pick.bm = pick.bn = bt;
        pick.split = split;
        pick.tail = 0;
      }
    }
    // tail split: whole rounds unsplit, the last partial round in K slices
    const int64_t slots = 2 * (int64_t)cus, rem = tiles % slots;
    if (an.L == 1 && tiles > slots && rem > 0) {
      const double w = 2.0 * bt * bt * (double)an.K / (cu_rate * eff);
      const double head = (double)(tiles / slots) * 2.0 * w;
      for (int split : {2, 3, 4, 6, 8}) {
        if (an.K / split < 2 * bk) continue;
        const int64_t q = ceil_div(rem * split, cus);
        const double ws = w / split;
        const double time = head + (double)(q / 2) * 2.0 * ws + (q % 2 ? ws / 0.65 : 0.0) +
                            (double)split * rem * bt * bt * es * 2.0 / hbm + 4e-6;
        if (time < best * 0.95) {  // only the tail pays for partial sums
          best = time;
          pick.bm = pick.bn = bt;
          pick.split = split;
          pick.tail = (int)rem;
        }
      }
    }
  }
  return pick;
}

// Whether the FP64 rows of X or Y lie whole cache lines apart.
static bool line_strides(const std::vector<Mode>& rows, bool x) {
  for (const Mode& m : rows)
    if ((x ? m.sx : m.sy) % 16) return false;
  return !rows.empty();
}

// The direct kernel reads every operand element once per tile of the other
// side, so it is bound by L2 (about 9 TB/s measured over its shapes: 32 x 32
// tiles 107 to 2147 MB in 17.8 to 241 us) where there are many tiles, and by
// the latency of one wave's K steps where there are few; the LDS-tiled kernel
// pays a barrier and a memory round trip per K slice and, with split-K, a
// second launch.  Both are estimated in microseconds from constants measured
// on MI355X and the smaller wins.  Examples, tiled -> direct: FP64 256^3
// 12.2 -> 5.6 us, FP64 144 x 1444 x 1444 33 -> 24, FP32 900^3 (runs of 30)
// 39 -> 27, FP64 16 x 675840 x 64 132 -> 108; the other way FP32 256 x 4096 x
// 4096 takes 78 tiled and 125 direct, so direct is not considered above 4
// GFLOP except for narrow problems.
//
// Chains (ChainCfg): a wave that takes K in one accumulator, against the tiled
// kernel's K ranges, had up to 1.5 times the error in FP32 (ladder v=36 o=9,
// 2.1e-7 -> 3.2e-7); with three, and no chain longer than the ranges', it has
// no more.
DirectCfg choose_direct(const famlies_handle_s* h, const Analysis& an, const TileCfg& t, const ChainCfg& chain,
                        double level_us) {
  DirectCfg none;
  if (an.M == 0 || an.N == 0 || an.K == 0) return none;
  const double flops = 2.0 * (double)an.M * (double)an.N * (double)an.K * (double)an.L;
  const bool narrow = std::min(an.M, an.N) <= 32;
  if (flops > 4e9 && !narrow) return none;
  const double es = an.esize, cus = h ? h->num_cus : 256;
  const int u = 16 / an.esize, ks = 4 * u;
  const int64_t kr = padded_k_length(an, u), K = kr ? kr : an.K;
  // an operand gathered along K but not in 16-byte runs touches a cache line
  // per element, one gathered by rows without unit stride two lines for one
  const bool xrun = kr && an.P[0].sx == 1, yrun = kr && an.P[0].sy == 1;
  const bool xlines = an.x_kfast && !xrun, ylines = an.y_kfast && !yrun;
  const double xw = xlines ? 2.5 : !an.x_kfast && !an.I.empty() && an.I[0].sx != 1 ? 2.0 : 1.0;
  const double yw = ylines ? 2.5 : !an.y_kfast && !an.J.empty() && an.J[0].sy != 1 ? 2.0 : 1.0;
  // FP64 rows read along K and whole cache lines apart (the longer side's)
  const bool by_lines = es == 8 && (an.M >= an.N ? xrun && line_strides(an.I, true) : yrun && line_strides(an.J, false));
  const double unique = ((double)an.M * an.K + (double)an.N * an.K + (double)an.M * an.N) * (double)an.L * es;
  const double hbm_us = unique / 4.3e6;

  // the tiled kernel
  const int64_t tiles = ceil_div(an.M, t.bm) * ceil_div(an.N, t.bn) * an.L;
  const int64_t split_tiles = t.split > 1 ? (t.tail ? t.tail : tiles) : 0;
  const double units = (double)(tiles - split_tiles) + (double)split_tiles * t.split;
  const double slices = (double)ceil_div(ceil_div(an.K, split_tiles == tiles ? t.split : 1), an.esize == 8 ? 8 : 32);
  const bool full = units > cus;  // two workgroups share a CU
  const double slice_us = t.bm == 64 ? (an.esize == 8 ? (full ? 0.72 : 0.45) : (full ? 1.5 : 0.92))
                                     : (an.esize == 8 ? 1.9 : xlines || ylines ? 5.0 : 3.8);
  double tiled = 3.5 + std::max(std::max(1.0, units / (2.0 * cus)) * slices * slice_us, hbm_us);
  if (t.split > 1) tiled += 4.0 + (double)(t.split + 1) * (double)split_tiles * t.bm * t.bn * es / 4.0e6;

  tiled = std::min(tiled, level_us);
  DirectCfg best = none;
  double crowded_us = 0.0;
  double best_us = 0.88 * tiled;  // the estimates are good to about a tenth
  const int shapes[4][2] = {{16, 16}, {32, 32}, {16, 64}, {64, 16}};
  for (const auto& sh : shapes)
    for (int wk : {1, 4})
      for (int split : {1, 4, 16, 64}) {
        if (split > 1 && (an.L > 1 || wk == 1 || K / split < 16 * ks)) continue;
        const double n = (double)ceil_div(an.M, sh[0]) * (double)ceil_div(an.N, sh[1]) * (double)an.L * split;
        if (n * wk > 1e9) continue;
        const double steps = (double)ceil_div(ceil_div(K, split), ks);
        const double rows = xw * (double)std::min<int64_t>(an.M, sh[0]) + yw * (double)std::min<int64_t>(an.N, sh[1]);
        const double l2_us = n * rows * steps * ks * es / 9.0e6;
        // 16 x 64 and 64 x 16 load five blocks of rows per step, 32 x 32 four; where
        // that fills as well and both operands come in runs, the difference shows
        // (FP32 2000 x 64 x 800 12.6 us in 16 x 64 tiles)
        const bool five = sh[0] != sh[1] && xrun && yrun && std::min(an.M, an.N) > 32;
        const double step_us = sh[0] * sh[1] == 256 ? (an.esize == 8 ? 0.20 : 0.27) : five ? 0.54 : 0.43;
        const double mfma_us = n * sh[0] * sh[1] * steps * ks * 2.0 / (an.esize == 8 ? 6.0e7 : 1.2e8);
        // narrow tiles touch memory in short segments: FP64 16 x 675840 x 64
        // takes 130 us in 16 x 16 tiles, 120 in 32 x 32, 108 in 16 x 64; with
        // its 64 side on the short side a tile is as narrow as 16 x 16 and does
        // four times the products (FP64 500000 x 16 x 64:
        // 175 us in 16 x 64 tiles, 74 in 64 x 16, tiled 114)
        const int64_t reach = std::max(std::min<int64_t>(sh[0], an.M), std::min<int64_t>(sh[1], an.N));
        const double mem_us = hbm_us * (reach <= 16 ? 1.25 : reach <= 32 ? 1.1 : 1.0);
        // elements gathered along K: up to 64 lines per load, which the larger
        // tiles wait for (FP32 300^3 strided on both sides: 17.7 us in 32 x 32
        // tiles, 9.8 in 16 x 16, tiled 11.1)
        const double lines = 64.0 * u * ((xlines ? sh[0] : 0) + (ylines ? sh[1] : 0)) / 16.0;
        const double line_us = std::ceil(n / cus) * steps * lines / (sh[0] * sh[1] == 256 ? 3.0e3 : 1.5e3);
        const double bound = std::max(
            std::max(std::max(std::ceil(steps / wk) * step_us, mfma_us), std::max(l2_us, mem_us)), line_us);
        double us = 4.0 + bound;
        if (wk > 1) us += 0.0012 * n;  // the waves' partial tiles through LDS
        if (split > 1) us += 4.0 + (double)(split + 1) * (double)an.M * (double)an.N * es / 4.0e6;
        const int64_t of_wave = ceil_div((int64_t)steps, wk);
        const int chains = std::min(of_wave * ks, K) <= chain.length ? 1 : 3;
        if (chains == 3 && ceil_div(of_wave, 3) * ks > chain.length) continue;
        if (us < best_us) {
          best_us = us;
          const double wgs = n * wk / (4.0 * cus), rm = (double)std::min<int64_t>(an.M, sh[0]),
                       rn = (double)std::min<int64_t>(an.N, sh[1]);
          crowded_us = us;
          if (by_lines && wgs > 1.0)
            crowded_us += std::max(0.0, l2_us * std::max(1.0, std::ceil(wgs - 0.1) / wgs) *
                                                (std::ceil(rm / 16) + std::ceil(rn / 16)) * 16 / (rm + rn) - bound);
          best.bm = sh[0];
          best.bn = sh[1];
          best.wk = wk;
          best.split = split;
          best.chains = chains;
        }
      }
  // FP64 rows whole cache lines apart crowd some of L2's channels: the CUs that
  // run a workgroup more than others do not catch up, and rows past an edge
  // cost as much as others (6000 x 64 x 800, 376 workgroups on 256 CUs: 30 us,
  // tiled 23; 51 x 5324 x 784 26.5 and 23; but 100 x 4000 x 700, 500 of them
  // and rows 43.75 lines apart, 21.5, tiled 27)
  if (crowded_us > 0.9 * tiled) return none;
  return best;
}

// Times of the 128 x 128 kernels in microseconds, from constants measured on
// MI355X: per K slice with two workgroups on every CU, per workgroup outside
// its slices (first loads, C update or partial sums), per byte of partial sums
// written and read.  A CU with a single workgroup runs it at about 0.65 of
// the CU's rate.  Two ways to cut the last round's tiles are weighed: evenly
// into 2 to 8 runs, or a long first part beside shorter runs on the slots
// that are free; the second moves fewer bytes, but its workgroups are at
// different places of K and share less in L2 (6 % charged): FP32 ladder v=93
// o=27 (408 tiles), unsplit 1104 us, five even runs 924, uneven 945.  Where
// the tile choice cuts every tile along K the runs keep its chains (ChainCfg),
// which costs a little of that; measured against K ranges of every tile with
// a plain reduction: that ladder 1092 -> 958 us, FP32 ring o=31 v=115 896 ->
// 814.
namespace {
struct RoundModel {
  int bm, bn;
  int64_t slots;               // workgroups in a round
  double slice, unit, block;   // us per slice, us per workgroup besides, bytes of a block of partial sums
  double lone;                 // time of a slice in a round of at most half the slots
  // units of n workgroups of s slices each
  double rounds(int64_t n, double s) const {
    const int64_t last = n % slots;
    return (double)(n / slots) * (s * slice + unit) +
           (last == 0 ? 0.0 : (2 * last > slots ? 1.0 : lone) * s * slice + unit);
  }
};
constexpr double kPassRate = 7.0e6;  // bytes of partial sums per us, written then read

// The fastest levelled round for `tiles` tiles of nk slices below *best us
// (which it lowers).  The last `cut` tiles run in parts of at most `chain`
// slices each: where they are more than the last round's, all of them are
// levelled, evenly.
LevelCfg level_round(const RoundModel& m, int64_t tiles, int64_t nk, int64_t cut, int64_t chain, double* best) {
  LevelCfg lv;
  const bool all = cut > tiles % m.slots;
  const int64_t rem = all ? tiles : tiles % m.slots, full = all ? 0 : tiles / m.slots;
  if (rem == 0 || tiles >= ((int64_t)1 << 30)) return lv;
  auto consider = [&](double time, int64_t q, int64_t part, int64_t parts) {
    if (cut > 0 && std::max(q, part) > chain) return;
    time += (double)full * ((double)nk * m.slice + m.unit) + 4.0 +
            (double)(rem * (2 * (1 + parts) + 2)) * m.block / kPassRate;
    if (time >= *best) return;
    *best = time;
    lv.head = (int)(tiles - rem);
    lv.rem = (int)rem;
    lv.q = (int)q;
    lv.part = (int)part;
    lv.parts = (int)parts;
  };
  const int64_t free_slots = m.slots - rem;
  for (int64_t parts = 1; parts <= (cut > 0 ? 15 : 7); ++parts) {
    if (nk / (parts + 1) < 4 || rem * (parts + 1) > (1 << 24)) break;
    const int64_t even = ceil_div(nk, parts + 1);
    if (nk - parts * even >= 1) consider(m.rounds(rem * (parts + 1), (double)even), nk - parts * even, even, parts);
    if (free_slots <= 0) continue;
    // the runs take `turns` each on the free slots, the first part is as long
    // as those together
    const int64_t turns = ceil_div(rem * parts, free_slots);
    const int64_t part =
        (int64_t)(((double)nk * m.slice - (double)(turns - 1) * m.unit) / (m.slice * (double)(turns + parts)));
    const int64_t q = nk - parts * part;
    if (part < 4 || q <= part) continue;
    consider(1.06 * std::max((double)q * m.slice + m.unit, (double)turns * ((double)part * m.slice + m.unit)), q, part,
             parts);
  }
  return lv;
}
}  // namespace

ChainCfg plan_chain(const Analysis& an, const TileCfg& t, int64_t kd, int64_t ntiles, int kchunk) {
  ChainCfg c;
  c.length = std::max<int64_t>(kd, 1);
  if (t.split <= 1) return c;
  c.length = kchunk;
  c.cut = t.tail ? t.tail : ntiles * an.L;
  // bf16x3 drops the product of the low parts, an error that does not shrink
  // with shorter chains: at 12544 entries in one chain and in four ranges it
  // is the same (3.8e-6; the chain's own share is 3e-7).
  if (split_parts(an.compute) == 2 && kd <= 12544) {
    c.length = kd;
    c.cut = 0;
  }
  return c;
}

LevelCfg choose_level(const famlies_handle_s* h, const Analysis& an, const TileCfg& t, int64_t kd,
                      const ChainCfg& chain, bool* unsplit, double* us) {
  *unsplit = false;
  if (t.bm == 256) {  // one workgroup per CU; measured at 4096^3 with unit strides on neither side, 1090 us
    const RoundModel tall{256, 128, h ? h->num_cus : 256, 4.2, 9.0, 256.0 * 128.0 * 8.0, 1.0};
    *us = tall.rounds(ceil_div(an.M, 256) * ceil_div(an.N, 128) * an.L, (double)ceil_div(kd, t.bk));
    return LevelCfg();
  }
  if (t.bm != 128 || t.bn != 128 || an.M == 0 || an.N == 0 || an.K == 0) return LevelCfg();
  const int ns = split_parts(an.compute);
  // a slice of the bf16 kernels (16-deep in bf16x6, 32-deep in bf16x3) by how
  // the operands are gathered: rows, and elements along K without unit stride,
  // take staging registers and load instructions (bf16x3 with two such operands
  // of a kind has one workgroup per CU).  Measured at 1024 x 4096 x 4096.
  const bool runs = padded_k_length(an, 16 / an.esize) != 0;
  const int strided = (an.x_kfast && !(runs && an.P[0].sx == 1)) + (an.y_kfast && !(runs && an.P[0].sy == 1));
  const int rows = !an.x_kfast + !an.y_kfast;
  const bool alone = ns == 2 && (strided == 2 || rows == 2);
  const double bf16 = ns == 3 ? (strided == 2 ? 2.25 : strided ? 1.6 : rows == 2 ? 1.85 : 1.5)
                              : strided == 2 ? 2.15 : rows == 2 ? 1.15 : strided ? 2.4 : rows ? 1.85 : 1.55;
  const RoundModel m{128, 128, (alone ? 1 : 2) * (int64_t)(h ? h->num_cus : 256),
                     ns ? bf16 : an.esize == 8 ? 1.95 : 3.8, 9.0, 128.0 * 128.0 * (ns ? 8.0 : (double)an.esize),
                     alone ? 1.0 : 0.77};
  const int64_t tiles = ceil_div(an.M, 128) * ceil_div(an.N, 128) * an.L, nk = ceil_div(kd, t.bk);
  const double whole = m.rounds(tiles, (double)nk);
  double now = whole;
  if (t.split > 1) {
    const int64_t cut = t.tail ? t.tail : tiles;
    now = m.rounds(tiles - cut, (double)nk) + m.rounds(cut * t.split, (double)ceil_div(nk, t.split)) + 4.0 +
          (double)(2 * t.split + 2) * (double)cut * m.block / 4.2e6;  // splitk_reduce, one element per thread
    if (whole < now && chain.cut == 0) {
      *unsplit = true;
      now = whole;
    }
  }
  // 5 % for the estimates' error; 2 % against K ranges, whose launch differs
  // from parts of the same length only in the reduction
  double best = (chain.cut ? 0.98 : 0.95) * now;
  const LevelCfg lv = level_round(m, tiles, nk, chain.cut, chain.length / t.bk, &best);
  if (lv.rem) *unsplit = false;
  *us = lv.rem ? best : now;
  return lv;
}

// bf16x3 on large problems: a 256 x 128 tile (128 x 64 per wave) halves the
// LDS bytes per MFMA of the 128 x 128 tile (bf16x6 stays at 128 x 128 with
// 16-deep slices, two workgroups per CU).  It has registers for one slice in
// flight and one workgroup per CU, so it is taken only when both operands are
// element-gathered along K: a row-gathered operand keeps the 128 x 128 tile
// with two slices in flight (ring o=48 v=192: 186 -> 201 TFLOP/s
// FP32-equivalent), and an operand in runs the 128 x 128 tile at two
// workgroups per CU (ladder v=128 o=32: 284 -> 307).  Where the operands meet
// enough tiles part planes, which gather each element once, replace it
// (choose_planes).
bool tall_tile(const Analysis& an, const TileCfg& t, int64_t runs) {
  if (split_parts(an.compute) != 2 || an.M < 1024 || an.N < 512 || t.split != 1 || !an.x_kfast || !an.y_kfast)
    return false;
  std::vector<int64_t> v[9];
  bool xv = false, yv = false;
  all_offsets(an, v);
  vec_flags(an, 32, index_bits_for(an), v, &xv, &yv);
  return !(xv || (runs && an.P[0].sx == 1)) && !(yv || (runs && an.P[0].sy == 1));
}

// The pass over the operands at 5.5 TB/s and tiles of twice the size, one per
// CU, against the estimate of the kernel that splits while staging.  Taken 7 %
// or more below it; measured on either side of the line: bf16x3 ladder o=27
// v=93 489 us split while staging (estimated 530 through planes), ladder o=36
// v=110 1824 -> 1582, ring o=32 v=112 363 -> 308.
//
// A plan that splits every tile along K keeps its chains here by folds
// (ChainCfg): 13 us per fold and round (bf16x6 ring o=31 v=115: 526 us without
// them, 561 with, 719 split while staging).
bool choose_planes(const famlies_handle_s* h, const Analysis& an, int64_t kd, const ChainCfg& chain, double split_us,
                   LevelCfg* lv, int* fold) {
  *fold = 0;
  if (split_us >= 1e30) return false;  // 64 x 64 tiles: operands that small are read too few times over
  const int ns = split_parts(an.compute);
  const int64_t tiles = ceil_div(an.M, 256) * ceil_div(an.N, 128) * an.L, nk = ceil_div(kd, 32);
  const double pass = (double)(an.M + an.N) * (double)kd * (double)an.L * (4.0 + 2.0 * ns) / 5.5e6 + 11.0;
  if (chain.cut > 0) {
    *fold = planes_fold_steps(ns, chain.length);
    if (*fold == 0) return false;
  }
  const double slice = (ns == 2 ? 1.4 : 2.3) + (*fold ? 13.0 / *fold : 0.0);
  const RoundModel m{256, 128, h ? h->num_cus : 256, slice, 11.0, 256.0 * 128.0 * 8.0, 1.0};
  double best = 0.93 * split_us - pass;
  *lv = LevelCfg();
  bool take = false;
  if (m.rounds(tiles, (double)nk) < best) {
    best = m.rounds(tiles, (double)nk);
    take = true;
  }
  const LevelCfg c = level_round(m, tiles, nk, 0, 0, &best);
  if (c.rem) {
    *lv = c;
    take = true;
  }
  return take;
}

bool contiguous_k_runs(const std::vector<int64_t>& ks, int64_t K, int u) {
  if (K < 1 || K % u) return false;
  for (int64_t b = 0; b < K; b += u)
    for (int j = 1; j < u; ++j)
      if (ks[(size_t)(b + j)] != ks[(size_t)b] + j) return false;
  return true;
}

// Settle split-K: K slices of whole BK-blocks, and the number of tiles
// computed whole first (*head; every tile when there is no split).
void finalize_split(TileCfg* t, int64_t K, int64_t ntiles, int* kchunk, int* head) {
  *head = (int)std::min<int64_t>(ntiles, INT32_MAX);
  if (t->split <= 1 || K <= t->bk) {
    t->split = 1;
    t->tail = 0;
    *kchunk = (int)std::max<int64_t>(K, 1);
    return;
  }
  int64_t chunk = ceil_div(ceil_div(K, t->split), t->bk) * t->bk;
  t->split = (int)ceil_div(K, chunk);
  *kchunk = (int)chunk;
  if (t->split <= 1) {
    t->split = 1;
    t->tail = 0;
    *kchunk = (int)K;
    return;
  }
  if (t->tail <= 0 || t->tail >= ntiles) t->tail = 0;  // every tile split
  *head = t->tail ? (int)(ntiles - t->tail) : 0;
}

void fill_info(const Analysis& an, const TileCfg& t, int index_bits, int kernel,
                      famlies_plan_info* info) {
  std::memset(info, 0, sizeof *info);
  info->m = an.M;
  info->n = an.N;
  info->k = an.K;
  info->batch = an.L;
  info->n_batch = (int32_t)an.Lm.size();
  info->n_trace = an.n_trace;
  info->n_diag = an.n_diag;
  info->swapped = an.swapped;
  info->x_kfast = an.x_kfast;
  info->y_kfast = an.y_kfast;
  info->n_i = (int32_t)an.I.size();
  info->n_j = (int32_t)an.J.size();
  info->n_p = (int32_t)an.P.size();
  info->tile_m = t.bm;
  info->tile_n = t.bn;
  info->tile_k = t.bk;
  info->split_k = t.split;
  info->split_tiles = t.split > 1 ? (t.tail ? t.tail : (int32_t)(ceil_div(an.M, t.bm) * ceil_div(an.N, t.bn))) : 0;
  info->index_bits = index_bits;
  info->kernel = kernel;
  info->flops = 2.0 * (double)an.L * (double)an.M * (double)an.N * (double)an.K;
}

// 32: uint32 byte offsets from each operand's lowest element (every operand
// spans less than 4 GiB over its non-batch modes); 64: int64 element offsets.
int index_bits_for(const Analysis& an) {
  const int64_t lim = ((int64_t)1 << 32) - 64;
  const int64_t es = an.esize;
  return ((an.x_span + 1) * es < lim && (an.y_span + 1) * es < lim && (an.c_span + 1) * es < lim) ? 32 : 64;
}

void index_form(const Analysis& an, int force, int* bits, bool* elem32) {
  // int32 element offsets: rebased row offsets lie in [0, span] and K
  // offsets in [-span, span], every sum in [0, span]: all below 2^31
  const int64_t lim = ((int64_t)1 << 31) - 64;
  const bool e32 = !int8_slices(an.compute) && an.x_span + 1 < lim && an.y_span + 1 < lim && an.c_span + 1 < lim;
  *elem32 = false;
  if (force == 64) {
    *bits = 64;
  } else if (force == kForceElem32 && e32) {
    *bits = 32;
    *elem32 = true;
  } else if (index_bits_for(an) == 32) {
    *bits = 32;
  } else if (e32) {
    *bits = 32;
    *elem32 = true;
  } else {
    *bits = 64;
  }
}

// Upload the indexing vectors (padded to the tile grid) into one device
// buffer: six OffT vectors (X rows, X k, Y k, Y cols, C rows, C cols), then
// the three int64 batch-offset vectors.  In the uint32 form every row vector
// is rebased by its operand's lowest offset and all six are scaled to bytes;
// sums row + col then land in [0, span) (unsigned wrap-around is exact).
// Block strides of the block-scatter layout (Approach, "Supporting tensor
// computations"): an operand gathered along K can be read with 16-byte loads
// when BK divides K (every slice whole), in every BK-block of K its indexing
// vector steps by exactly one element, and every run start (row offset +
// block start + batch offset, in elements from the base pointer) is a
// multiple of the 16-byte vector.
bool affine_k_blocks(const std::vector<int64_t>& rows, int64_t nrows, const std::vector<int64_t>& ks,
                            int64_t K, int bk, const std::vector<int64_t>& batch, int64_t L, int64_t vk) {
  if (K < 1 || K % bk) return false;
  for (int64_t b = 0; b < K; b += bk) {
    const int64_t s0 = ks[(size_t)b];
    if (s0 % vk) return false;
    for (int64_t k = b + 1; k < std::min<int64_t>(K, b + bk); ++k)
      if (ks[(size_t)k] != s0 + (k - b)) return false;
  }
  for (int64_t m = 0; m < nrows; ++m)
    if (rows[(size_t)m] % vk) return false;
  for (int64_t l = 0; l < L; ++l)
    if (batch[(size_t)l] % vk) return false;
  return true;
}

// Affine-block flags of X and Y for a plan with K-slice depth bk; v holds
// the nine indexing vectors in upload() order.
void vec_flags(const Analysis& an, int bk, int /*index_bits*/, const std::vector<int64_t>* v, bool* xv,
                      bool* yv) {
  *xv = *yv = false;
  const int64_t vk = 16 / an.esize;
  *xv = an.x_kfast && affine_k_blocks(v[0], an.M, v[1], an.K, bk, v[6], an.L, vk);
  *yv = an.y_kfast && affine_k_blocks(v[3], an.N, v[2], an.K, bk, v[7], an.L, vk);
}

void all_offsets(const Analysis& an, std::vector<int64_t>* v) {
  const std::vector<Mode>* groups[9] = {&an.I, &an.P, &an.P, &an.J, &an.I, &an.J, &an.Lm, &an.Lm, &an.Lm};
  const int which[9] = {0, 0, 1, 1, 2, 2, 0, 1, 2};
  const int64_t len[9] = {an.M, an.K, an.K, an.N, an.M, an.N, an.L, an.L, an.L};
  for (int i = 0; i < 9; ++i) offsets(*groups[i], which[i], len[i], len[i], v[i]);
}

int kernel_code(const Analysis& an, bool xv, bool yv) {
  if (int8_slices(an.compute)) return 8 + int8_slices(an.compute);
  return 1 + split_parts(an.compute) + (xv ? 16 : 0) + (yv ? 32 : 0);
}

TileCfg int8_tile(int slices, int64_t n) {
  TileCfg t;
  t.bm = 128;
  t.bn = slices <= 6 && n > 64 ? 128 : 64;
  t.bk = 64;
  t.split = 1;
  t.tail = 0;
  return t;
}

// One workgroup per CU: K ranges even out the rounds of tiles.  A step of 32
// contracted indices takes about 0.04 S (S + 1) us, a workgroup 8 us besides
// (first loads, recombination), partial sums pass at 6 TB/s.  FP64 ladder v=38
// o=12 at six slices (24 tiles): GEMM 70 us unsplit.
int int8_split(const famlies_handle_s* h, const Analysis& an, const TileCfg& t, int64_t kd) {
  const int64_t cus = h ? h->num_cus : 256;
  const int64_t tiles = ceil_div(an.M, t.bm) * ceil_div(an.N, t.bn), blocks = ceil_div(kd, t.bk);
  const int S = int8_slices(an.compute);
  const double block_us = 0.08 * S * (S + 1) * t.bn / 128.0;
  double best = 1e300;
  int pick = 1;
  for (int s = 1; s <= 16 && s <= blocks; ++s) {
    double us = (double)ceil_div(tiles * s, cus) * ((double)ceil_div(blocks, s) * block_us + 8.0);
    if (s > 1) us += 4.0 + (double)(2 * s + 2) * (double)tiles * t.bm * t.bn * 8.0 / 6.0e6;
    if (us < 0.95 * best) {
      best = us;
      pick = s;
    }
  }
  return pick;
}

bool log_enabled() {
  static const bool on = [] {
    const char* v = std::getenv("FAMLIES_LOG");
    return v && *v && std::strcmp(v, "0") != 0;
  }();
  return on;
}

// One line on stderr: what the planner decided (orientation, loaders, tile,
// split, index form -- index_bits 32: uint32 bytes, -32: int32 elements, 64:
// int64 elements -- and workspace).
void log_decision(const char* what, const Analysis& an, const TileCfg& cfg, const DirectCfg& d,
                  const LevelCfg& lv, bool planes, int fold, int index_bits, bool x_vec, bool y_vec,
                  size_t work_bytes, bool table_hit) {
  static const char* loader[4] = {"rows", "k-gather", "packed", "k-affine"};
  const int xm = an.x_kfast ? (x_vec ? 3 : 1) : 0, ym = an.y_kfast ? (y_vec ? 3 : 1) : 0;
  static const char* int8_names[8] = {"", "", "", "int8x3", "int8x4", "int8x5", "int8x6", "int8x7"};
  const char* comp = an.compute == FAMLIES_BF16X3   ? "bf16x3"
                     : an.compute == FAMLIES_BF16X6 ? "bf16x6"
                     : int8_slices(an.compute)      ? int8_names[int8_slices(an.compute)]
                                                    : "native";
  char direct[112] = "";
  if (d.bm)
    std::snprintf(direct, sizeof direct, " direct=%dx%d/%d waves/split %d/chains %d", d.bm, d.bn, d.wk, d.split,
                  d.chains);
  if (lv.rem)
    std::snprintf(direct, sizeof direct, " level=%d whole, %d x %d + %d x %d slices", lv.head, lv.rem, lv.q, lv.parts,
                  lv.part);
  char through[64] = "";
  if (planes) std::snprintf(through, sizeof through, fold ? " planes 256x128 fold=%d steps" : " planes 256x128", fold);
  std::fprintf(stderr,
               "[famlies] %s %s/%s M=%lld N=%lld K=%lld L=%lld swapped=%d groups=%zu/%zu/%zu/%zu "
               "trace=%d diag=%d X=%s Y=%s tile=%dx%dx%d split=%d split_tiles=%d index=%s "
               "workspace=%zu B%s%s%s\n",
               what, an.dtype == FAMLIES_F64 ? "f64" : "f32", comp, (long long)an.M, (long long)an.N,
               (long long)an.K, (long long)an.L, an.swapped ? 1 : 0, an.I.size(), an.J.size(), an.P.size(),
               an.Lm.size(), an.n_trace, an.n_diag, loader[xm], loader[ym], cfg.bm, cfg.bn, cfg.bk, cfg.split,
               cfg.split > 1 ? (cfg.tail ? cfg.tail : -1) : 0,
               index_bits == 32 ? "u32-bytes" : index_bits == -32 ? "i32-elements" : "i64-elements", work_bytes,
               table_hit ? " (tile table)" : "", through, direct);
}

}  // namespace famlies

using namespace famlies;

extern "C" {

const char* famlies_last_error(void) { return g_err.c_str(); }

static famlies_status analyze_impl(int dtype, int compute, const famlies_tensor* A, const famlies_tensor* B,
                                   const famlies_tensor* C, famlies_plan_info* info, int64_t* offs,
                                   int64_t offs_len) {
  if (!info) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_analyze: null info");
  Analysis an;
  std::string err;
  int st = analyze(dtype, compute, A, B, C, &an, &err);
  if (st != FAMLIES_OK) return fail(st, err);
  if (an.M > kMaxGemmDim || an.N > kMaxGemmDim || an.K > kMaxGemmDim || an.L > kMaxGemmDim)
    return fail(FAMLIES_ERR_UNSUPPORTED, "a GEMM dimension exceeds 2^31 - 1024");
  TileCfg t = int8_slices(an.compute) ? int8_tile(int8_slices(an.compute), an.N) : choose_tiles(nullptr, an);
  if (split_parts(an.compute) && t.tail) {  // as in make_plan: no split for the bf16 kernels
    t.split = 1;
    t.tail = 0;
  }
  if (split_parts(an.compute)) t.bk = split_slice_k(split_parts(an.compute));
  int kchunk = 0, head = 0;
  int ib = 64;
  bool e32 = false;
  index_form(an, 0, &ib, &e32);
  const int64_t runs =  // as in make_plan: the padded contracted order
      ib != 32 || e32 ? 0 : padded_k_length(an, 16 / an.esize);
  const int64_t kd = runs && runs <= kMaxGemmDim ? runs : an.K, ntiles = ceil_div(an.M, t.bm) * ceil_div(an.N, t.bn);
  finalize_split(&t, kd, ntiles, &kchunk, &head);
  const ChainCfg chain = plan_chain(an, t, kd, ntiles, kchunk);
  std::vector<int64_t> v[9];
  bool xv = false, yv = false;
  if (an.M > 0 && an.N > 0) {
    all_offsets(an, v);
    vec_flags(an, t.bk, ib, v, &xv, &yv);
  }
  fill_info(an, t, ib, kernel_code(an, xv, yv), info);
  info->index_elements = ib == 64 || e32;
  // what a plan would run instead of the tile choice reported above
  DirectCfg d;
  LevelCfg lv, plv;
  bool planes = false;
  int fold = 0;
  if (!int8_slices(an.compute)) {
    bool unsplit = false;
    double level_us = 1e30;
    TileCfg run = t;
    if (an.M > 0 && an.N > 0 && tall_tile(an, t, runs)) run.bm = 256;
    lv = choose_level(nullptr, an, run, kd, chain, &unsplit, &level_us);
    if (split_parts(an.compute) && ib == 32 && !e32) planes = choose_planes(nullptr, an, kd, chain, level_us, &plv, &fold);
    if (planes) lv = plv;
    if (!split_parts(an.compute) && ib == 32 && !e32) d = choose_direct(nullptr, an, t, chain, level_us);
    if (d.bm) lv = LevelCfg();
  }
  if (log_enabled()) log_decision("analyze", an, t, d, lv, planes, fold, e32 ? -32 : ib, xv, yv, 0, false);
  if (offs) {
    const int64_t need = 2 * an.M + 2 * an.K + 2 * an.N + 3 * an.L;
    if (offs_len < need) return fail(FAMLIES_ERR_INVALID_ARG, "famlies_analyze: offsets buffer too short");
    if (an.M == 0 || an.N == 0) all_offsets(an, v);
    int64_t pos = 0;
    for (int i = 0; i < 9; ++i) {
      std::copy(v[i].begin(), v[i].end(), offs + pos);
      pos += (int64_t)v[i].size();
    }
  }
  return FAMLIES_OK;
}

famlies_status famlies_analyze(int dtype, int compute, const famlies_tensor* A, const famlies_tensor* B,
                               const famlies_tensor* C, famlies_plan_info* info, int64_t* offs,
                               int64_t offs_len) {
  return no_throw("famlies_analyze", [&] { return analyze_impl(dtype, compute, A, B, C, info, offs, offs_len); });
}

}  // extern "C"
