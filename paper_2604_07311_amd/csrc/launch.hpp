// Host-side launch interface between the C ABI and the kernel files.
#pragma once

#include <hip/hip_runtime.h>

#include "args.hpp"
#include "famlies.h"
#include "internal.hpp"

namespace famlies {

struct PlainLaunch {
  enum Kind { kMain = 0, kScale = 1 } kind = kMain;
  int bm = 128, bn = 128, bk = 16;
  int xm = 1, ym = 1;  // operand loader modes: 0 row-gathered, 1 K-gathered, 2 pre-packed
};

hipError_t launch_plain(int dtype, const PlainArgs<uint32_t>& a, const PlainLaunch& L, hipStream_t s);
hipError_t launch_plain(int dtype, const PlainArgs<int32_t>& a, const PlainLaunch& L, hipStream_t s);
hipError_t launch_plain(int dtype, const PlainArgs<int64_t>& a, const PlainLaunch& L, hipStream_t s);
// A pre-packed operand of the direct kernel: elements of a batch plane (0: not
// packed), rows of a tile (their logarithm), bytes of a tile of rows over all
// of K and between rows of a block.
struct DirectPacked {
  int64_t plane = 0;
  int32_t shift = 0;
  uint32_t tile = 0, row = 0;
};
hipError_t launch_direct(int dtype, const PlainArgs<uint32_t>& a, const DirectCfg& d, bool xv, bool yv,
                         const DirectPacked& xp, const DirectPacked& yp, hipStream_t s);
// C = alpha * sum over K ranges of W + beta * C for the split tiles (bm x bn blocks of partial sums).
// bf16: the partial sums are FP64 (split-bf16 kernels).
template <typename OffT>
hipError_t launch_splitk_reduce(int dtype, bool bf16, const PlainArgs<OffT>& a, int bm, int bn, hipStream_t s);
// C from the blocks (bm x 128) of partial sums of a levelled launch.
template <typename OffT>
hipError_t launch_level_reduce(int dtype, bool bf16, const PlainArgs<OffT>& a, int bm, hipStream_t s);
bool plain_tile_supported(int dtype, int bm, int bn, int bk);

}  // namespace famlies
