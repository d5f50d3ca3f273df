// Per-tile GEMM bodies shared by the single-matrix kernels (gemm.hip) and the
// grouped batched kernels (batched.hip).  Defined in gemm_tiles.inc, included by
// both translation units.
#pragma once

#include "zf_internal.h"

namespace zf {

// 16-bit elements of one 32-wide K stage of a BM x BN tile: both halves of both operands,
// or one half (or one plane of bytes) for the single-product modes.
constexpr int x3_stage(int bm, int bn, int pm) {
  return ((pm & PM_HH) != 0 || pm == PM_I8 ? 1 : 2) * (bm + bn) * 32;
}
// Shared memory of a tile with an NS-stage ring, in 16-bit elements: the ring, which later
// holds the epilogue's 32-row strips (FP32 accumulators, then FP64 values).
constexpr int x3_lds(int bm, int bn, int pm, int ns) {
  return ns * x3_stage(bm, bn, pm) > 192 * (bn + 1) ? ns * x3_stage(bm, bn, pm) : 192 * (bn + 1);
}

template <int BM, int BN, int BK, int WM, int WN>
struct X3Cfg {
  static constexpr int NT = WM * WN * 64;
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int FM = WTM / 32, FN = WTN / 32;
  static constexpr int STAGE = (BM + BN) * 2 * BK;  // 16-bit elements per pipeline stage
  static constexpr int SP = BN + 1;                  // epilogue strip pitch (elements)
  // the two stage buffers also hold the epilogue's 32-row strips: FP32 accumulators
  // then FP64 values, 32 SP (4 + 8) bytes = 192 SP 16-bit elements
  static constexpr int STAGE_ELEMS = (2 * STAGE > 192 * SP) ? STAGE : 96 * SP;
  static_assert(BK == 32, "the LDS swizzle assumes 64-byte tile rows");
  static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0, "wave tile");
};

// FP64 tile of edge T (64 or 32): 4 waves, each a quarter of the tile.  The 64-wide tile
// runs four blocks per CU on a two-stage ring, the 32-wide one, for small grids, hides the
// load latency behind a four-stage ring.
template <int T>
struct F64Cfg {
  static constexpr int WM = 2, WN = 2, NT = 256;
  static constexpr int NS = T == 32 ? 4 : 2;
  static constexpr int LDS = NS * 2 * T * 16;  // doubles
};

}  // namespace zf
