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
// Shared memory the epilogue takes per wave, in 16-bit elements: a 32 x 33 block of doubles.
constexpr int kEpiWave = 32 * 33 * 4;
// Shared memory of a tile with an NS-stage ring and nw waves, in 16-bit elements: the ring,
// whose place the epilogue takes after the main loop.
constexpr int x3_lds(int bm, int bn, int pm, int ns, int nw) {
  return ns * x3_stage(bm, bn, pm) > nw * kEpiWave ? ns * x3_stage(bm, bn, pm) : nw * kEpiWave;
}

template <int BM, int BN, int BK, int WM, int WN>
struct X3Cfg {
  static constexpr int NT = WM * WN * 64;
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int FM = WTM / 32, FN = WTN / 32;
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
