// Matrix-core GEMMs of the refinement sweep (gfx950).
//
// Both kernels compute an "NT" product C[i][j] = sum_k A[i][k] * B[j][k] with A
// (M x K) and B (N x K) row-major, i.e. both operands contiguous along the
// contracted index.  The sweep keeps every operand in that form: S and the
// iterates delta, Q are symmetric, and Z is stored both row-major and
// transposed, so no kernel ever needs a transposing load.  Z's transposed pair
// is K-blocked (kb_offset: 32-wide K blocks, each a row-major panel), which the
// BF16x3 main loop reads through its per-operand K-block stride and which the
// update's transposed epilogue writes as one contiguous 2 KB run per 32 x 32 block.
//
//   gemm_x3  : (h)(h) + (h)(l) + (l)(h) of Sec. III.B (Eqs. SZn, Xn, Xsq): each
//              operand is a BF16 hi/lo pair, the three products accumulate into
//              one FP32 accumulator on v_mfma_f32_32x32x16_bf16.
//   gemm_f64 : FP64 products on v_mfma_f64_16x16x4_f64 (the "double" scheme).
//
// Symmetric mode computes only the tiles with tile_row <= tile_col of a product
// known to be symmetric (Z^T S Z, delta * delta and polynomials of delta) and
// mirrors them, which halves those GEMMs.  Inside a diagonal tile the upper
// triangle is written and mirrored, so the stored matrix is exactly symmetric.
//
// The epilogue forms out = alpha * D + beta * acc + gamma * I in FP64 and writes
// any of: FP32, FP64, a BF16 hi/lo split (Sec. III.A), each in normal and/or
// transposed layout, plus a per-tile FP64 sum of out^2 for the Frobenius norm
// of the stop test (Sec. IV.A).
#include <stdlib.h>

#include "zf_internal.h"
#include "gemm_tiles.inc"

namespace zf {
// SYM is a template parameter so that the two modes are distinct kernels (and show
// up separately in a kernel trace).
template <int BM, int BN, int WM, int WN, bool SYM, int PM, int NS, int OCC>
__global__ void __launch_bounds__(WM* WN * 64, OCC)
    gemm_x3_kernel(const u16* __restrict__ Ahi, const u16* __restrict__ Alo, int lda,
                   const u16* __restrict__ Bhi, const u16* __restrict__ Blo, int ldb, int M,
                   int N, int K, int tiles_n, int gm, EpiParams ep, int ksa, int ksb) {
  __shared__ __attribute__((aligned(16))) u16 lds[x3_lds(BM, BN, PM, NS, WM * WN)];
  __shared__ double red[WM * WN];
  if (ep.gate && *ep.gate) return;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  int ti, tj;
  tile_coords(bid, tiles_n, SYM, ti, tj, gm);
  const int mode = SYM ? (ti == tj ? 2 : 1) : 0;
  int m0 = ti * BM, n0 = tj * BN, m_lo = 0, n_lo = 0;
  if constexpr (BM == 192) {  // may not divide the order: the last tiles move back inside
    m_lo = m0;
    n_lo = n0;
    m0 = m0 < M - BM ? m0 : M - BM;
    n0 = n0 < N - BN ? n0 : N - BN;
  }
  x3_tile<BM, BN, WM, WN, PM, NS>(Ahi, Alo, lda, Bhi, Blo, ldb, K, m0, n0, mode, ep,
                                  tile_index(ti, tj, tiles_n, SYM), lds, red, ksa, ksb, m_lo,
                                  n_lo);
}

// FP32 matrix-core GEMM ("single"): f32_mainloop + the shared epilogue.
template <int BM, int BN, int WM, int WN, bool SYM>
__global__ void __launch_bounds__(WM* WN * 64)
    gemm_f32_kernel(const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb,
                    int K, int tiles_n, int gm, EpiParams ep) {
  using C = X3Cfg<BM, BN, 32, WM, WN>;
  // two stages of 16 floats per row: as many bytes as a single-product 16-bit stage
  __shared__ __attribute__((aligned(16))) u16 lds[x3_lds(BM, BN, PM_HH, 2, WM * WN)];
  __shared__ double red[C::NT / 64];
  if (ep.gate && *ep.gate) return;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  int ti, tj;
  tile_coords(bid, tiles_n, SYM, ti, tj, gm);
  const int mode = SYM ? (ti == tj ? 2 : 1) : 0;
  X3Acc<BM, BN, 32, WM, WN> acc;
#pragma unroll
  for (int a = 0; a < C::FM; ++a)
#pragma unroll
    for (int b = 0; b < C::FN; ++b) acc[a][b] = f32x16{};
  f32_mainloop<BM, BN, WM, WN>(A, lda, B, ldb, 0, K, ti * BM, tj * BN, lds, acc);
  x3_epilogue<BM, BN, 32, WM, WN, PAIR_BF16>(acc, ti * BM, tj * BN, mode, ep, tile_index(ti, tj, tiles_n, SYM),
                                  lds, red);
}

// ---------------------------------------------------------------------------
// FP64 kernel
// ---------------------------------------------------------------------------
// The tiles are 64 wide, except those whose row-major number is nbig or more: each of these is
// four 32-wide ones (f64_whole_tiles), done by the last blocks, as every CU should have its
// share of the large tiles before the small ones fill in.
template <bool SYM>
__global__ void __launch_bounds__(256, 4)
    gemm_f64_kernel(const double* __restrict__ A, int lda, const double* __restrict__ B, int ldb,
                    int K, int tiles, int nbig, int tiles_n, int gm, EpiParams ep) {
  using C64 = F64Cfg<64>;
  using C32 = F64Cfg<32>;
  static_assert(C64::LDS == C32::LDS && C64::NT == 256 && C32::NT == 256, "one block shape");
  __shared__ __attribute__((aligned(16))) double lds[C64::LDS];
  __shared__ double red[4];
  if (ep.gate && *ep.gate) return;
  const int bid = blockIdx.x;
  int ti, tj, sub = 0;
  if (bid < nbig) {  // in bands or groups where they are the whole grid
    tile_coords(xcd_remap(bid, nbig), tiles_n, SYM, ti, tj, nbig == tiles ? gm : 1);
  } else {
    const int j = xcd_remap(bid - nbig, gridDim.x - nbig);
    tile_coords(nbig + j / 4, tiles_n, SYM, ti, tj, 1);
    sub = j % 4;
  }
  const int t = tile_index(ti, tj, tiles_n, SYM);
  if (t < nbig) {
    f64_tile<64, 64, C64::WM, C64::WN, C64::NS>(A, lda, B, ldb, K, ti * 64, tj * 64,
                                                SYM ? (ti == tj ? 2 : 1) : 0, ep, t, lds, red);
    return;
  }
  const int pidx = nbig + 4 * (t - nbig) + sub;
  const int si = 2 * ti + (sub >> 1), sj = 2 * tj + (sub & 1);
  if (SYM && si > sj) {  // below the diagonal: written from its mirror
    if (ep.partials) block_norm_store<256>(0.0, ep, pidx, red);
    return;
  }
  f64_tile<32, 32, C32::WM, C32::WN, C32::NS>(A, lda, B, ldb, K, si * 32, sj * 32,
                                              SYM ? (si == sj ? 2 : 1) : 0, ep, pidx, lds, red);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static bool dims_ok(int M, int N, int K, bool sym) {
  return M > 0 && N > 0 && K > 0 && M % kTile == 0 && N % kTile == 0 && K % kTile == 0 &&
         (!sym || M == N);
}

static int grid_blocks(int M, int N, int t, bool sym) {
  const int tm = (M + t - 1) / t, tn = (N + t - 1) / t;
  return sym ? tm * (tm + 1) / 2 : tm * tn;
}

// Forced tile edge (tuning), 0 for none: ZF_X3_TILE / ZF_X3_SYM_TILE where it divides.
static int forced_edge(int M, int N, bool sym) {
  const char* env = getenv(sym ? "ZF_X3_SYM_TILE" : "ZF_X3_TILE");
  const int want = env ? atoi(env) : 0;
  return (want == 64 || want == 128 || want == 256) && M % want == 0 && N % want == 0 ? want : 0;
}

// Tile edge of a launch.  Per flop the 256-wide tile is the fastest (operand traffic), but
// it, the 192- and the 128-wide one take a CU for themselves, so the number of full rounds
// over the 256 CUs decides.  Estimated time of a launch in rounds of 256-wide tiles:
//   256: 1 per round; 192: 0.6; 128: 0.34 (0.25 of the work); 64: 0.11 (1 + tiles per CU),
//   as up to four of these share a CU.
// The 192-wide tile need not divide the order.  Per round and column of the contraction,
// measured over N = 1024 to 5120 (overlap matrices, mixed solve): 256 58-65 ns, 192 34-42,
// 128 18-21, 64 14 + 7 per tile and CU; the low ends are for rounds that leave CUs idle,
// where the clock stays higher.  Times per launch by edge, 256 / 192 / 128 wide, us:
//   full N = 3072 179 / 125 / 168, N = 3584 218 / 250 / 257, N = 4096 266 / 311 / 321,
//   N = 4352 504 / 445 / 408, N = 5120 615 / 576 / 643;
//   symmetric N = 3072 154 / 103 / 111, N = 4096 210 / 170 / 221, N = 5120 314 / 377 / 383.
// 64 against 128 wide: full N = 1024 14 / 22, N = 1536 33 / 32; symmetric N = 1536 25 / 32,
// N = 2304 52 / 48.
// The single-product modes take the same edges: a third of the products on half the operand
// bytes leaves the edges' order as it is.  (h)(h) solves with every edge forced in turn, N =
// 500 to 6000: the rule's choice is within 2% of the best one but for full N = 2500 (192 wide
// 952 us a solve, 128 wide 897).
int x3_tile_edge(int M, int N, bool sym) {
  const char* env = getenv(sym ? "ZF_X3_SYM_TILE" : "ZF_X3_TILE");
  if (env && atoi(env) == 192 && M >= 192 && N >= 192) return 192;
  if (const int want = forced_edge(M, N, sym)) return want;
  auto rounds = [&](int t) { return (grid_blocks(M, N, t, sym) + 255) / 256; };
  int edge = 64;
  double best = 0.11 * (1 + rounds(64));
  auto offer = [&](int t, double cost) {
    if (cost < best) {
      best = cost;
      edge = t;
    }
  };
  if (M % 128 == 0 && N % 128 == 0) offer(128, 0.34 * rounds(128));
  if (M >= 192 && N >= 192) offer(192, 0.6 * rounds(192));
  if (M % 256 == 0 && N % 256 == 0) offer(256, 1.0 * rounds(256));
  return edge;
}

int x3_blocks(int M, int N, bool sym) { return grid_blocks(M, N, x3_tile_edge(M, N, sym), sym); }


// FP64 tiles of a launch that stay 64 wide.  A 64-wide tile keeps its CU's matrix cores at 0.9
// of their rate, a 32-wide one at 0.7 (twice the operand traffic per flop), but a quarter of
// the size spreads a small number of tiles over more CUs.  So full rounds over the 256 CUs
// stay whole, and the tiles beyond them are quartered where that gives at most three
// 32-wide tiles a CU (1.2 / 4 of a 64-wide one's time each), which is up to 192 of them, and
// where a round weighs enough: from six on, the blocks' own drift evens the rest out.
// Measured per launch, all 64 / all 32 / this rule, us: full N = 512 23 / 11 / 11, N = 1024
// 42 / 41 / 41, N = 1536 143 / 122 / 110, N = 2500 514 / 567 / 514; symmetric N = 1024 41 /
// 35 / 35, N = 1536 100 / 80 / 68, N = 2048 187 / 161 / 144, N = 2500 298 / 300 / 251,
// N = 3000 528 / 500 / 432, N = 4096 1110 / 1248 / 1110.
// ZF_F64_TILE / ZF_F64_SYM_TILE force all 64 or all 32 (tuning).
static int f64_whole_tiles(int M, int N, bool sym) {
  const int tiles = grid_blocks(M, N, 64, sym);
  const char* env = getenv(sym ? "ZF_F64_SYM_TILE" : "ZF_F64_TILE");
  const int want = env ? atoi(env) : 0;
  if (want == 32) return 0;
  if (want == 64) return tiles;
  const int rest = tiles % 256;
  return rest <= 192 && tiles < 6 * 256 ? tiles - rest : tiles;
}

// Row-group height of the full-grid tile order: 4 (a run of 32 tiles on one XCD then
// covers 4 x 8 tiles, 12 operand panels instead of 18); ZF_TILE_GROUP overrides.
static int tile_group(int M, int t) {
  const char* env = getenv("ZF_TILE_GROUP");
  const int gm = env ? atoi(env) : 4, tm = (M + t - 1) / t;
  if (!env && tm % 4 != 0) return tm % 3 == 0 ? 3 : tm % 5 == 0 ? 5 : tm % 2 == 0 ? 2 : 1;
  return (gm > 1 && tm % gm == 0) ? gm : 1;
}

// Band height of the symmetric-grid tile order: 4 (a run of 17 of the 136 tiles of
// an N = 4096 triangle then spans about 4 x 5 tiles instead of one tile row; the
// symmetric BF16x3 GEMM measured 308 -> 303 us); ZF_SYM_TILE_GROUP overrides (1: row
// by row).
static int sym_group() {
  const char* env = getenv("ZF_SYM_TILE_GROUP");
  const int g = env ? atoi(env) : 4;
  return g >= 1 ? g : 1;
}

int f64_blocks(int M, int N, bool sym) {
  const int tiles = grid_blocks(M, N, 64, sym);
  return tiles + 3 * (tiles - f64_whole_tiles(M, N, sym));
}

double f64_elements(int M, int N, bool sym) {
  return 64.0 * 64.0 * grid_blocks(M, N, 64, sym);
}

int max_blocks(int M, int N) { return grid_blocks(M, N, 32, false); }

template <int BM, int BN, int WM, int WN, int PM, int NS, int OCC>
static void x3_launch(const u16* Ahi, const u16* Alo, int lda, const u16* Bhi, const u16* Blo,
                      int ldb, int M, int N, int K, bool sym, int blocks, const EpiParams& ep,
                      hipStream_t st, int ksa, int ksb) {
  if (sym)
    hipLaunchKernelGGL((gemm_x3_kernel<BM, BN, WM, WN, true, PM, NS, OCC>), dim3(blocks),
                       dim3(WM * WN * 64), 0, st, Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, (N + BN - 1) / BN, sym_group(), ep,
                       ksa, ksb);
  else
    hipLaunchKernelGGL((gemm_x3_kernel<BM, BN, WM, WN, false, PM, NS, OCC>), dim3(blocks),
                       dim3(WM * WN * 64), 0, st, Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, (N + BN - 1) / BN,
                       tile_group(M, BM), ep, ksa, ksb);
}

template <int BM, int BN, int WM, int WN>
static void f32_launch(const float* A, int lda, const float* B, int ldb, int M, int N, int K,
                       bool sym, int blocks, const EpiParams& ep, hipStream_t st) {
  if (sym)
    hipLaunchKernelGGL((gemm_f32_kernel<BM, BN, WM, WN, true>), dim3(blocks), dim3(WM * WN * 64),
                       0, st, A, lda, B, ldb, K, N / BN, sym_group(), ep);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<BM, BN, WM, WN, false>), dim3(blocks), dim3(WM * WN * 64),
                       0, st, A, lda, B, ldb, K, N / BN, tile_group(M, BM), ep);
}

template <int PM>
static void x3_dispatch(const u16* Ahi, const u16* Alo, int lda, const u16* Bhi, const u16* Blo,
                        int ldb, int M, int N, int K, bool sym, int tile, int blocks,
                        const EpiParams& ep, hipStream_t st, int ksa, int ksb) {
  // 8 waves of 128 x 64.  The three-product kernels fill all 256 registers and keep three values
  // in scratch memory, stored ahead of the main loop and read back behind it.
  if (tile == 256)
    x3_launch<256, 256, 2, 4, PM, 2, 1>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, blocks, ep, st,
                                        ksa, ksb);
  else if (tile == 192)  // 4 waves of 96 x 96, loads two stages ahead
    x3_launch<192, 192, 2, 2, PM, 3, 1>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, blocks, ep, st,
                                        ksa, ksb);
  else if (tile == 128)  // 8 waves of 32 x 64, one block per CU, loads three stages ahead
    x3_launch<128, 128, 4, 2, PM, 4, 1>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, blocks, ep, st,
                                        ksa, ksb);
  else if (blocks > 512 && blocks <= 1024)  // one round at four blocks per CU
    x3_launch<64, 64, 2, 2, PM, 2, 4>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, blocks, ep, st,
                                      ksa, ksb);
  else
    x3_launch<64, 64, 2, 2, PM, 4, 2>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, blocks, ep, st,
                                      ksa, ksb);
}

hipError_t launch_gemm_x3(const u16* Ahi, const u16* Alo, int lda, const u16* Bhi, const u16* Blo,
                          int ldb, int M, int N, int K, bool sym, const EpiParams& ep,
                          hipStream_t st, int pm, int ksa, int ksb) {
  if (!dims_ok(M, N, K, sym) || pm < 0 || pm > 3) return hipErrorInvalidValue;
  if (ksa < 32 || ksa % 32 || ksb < 32 || ksb % 32) return hipErrorInvalidValue;
  const int tile = x3_tile_edge(M, N, sym);
  const int blocks = x3_blocks(M, N, sym);
  switch (pm) {
    case PM_X3:
      x3_dispatch<PM_X3>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, tile, blocks, ep, st, ksa,
                          ksb);
      break;
    case PM_HH:
      x3_dispatch<PM_HH>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, tile, blocks, ep, st, ksa,
                          ksb);
      break;
    case PM_X3F16:
      x3_dispatch<PM_X3F16>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, tile, blocks, ep, st, ksa,
                          ksb);
      break;
    default:
      x3_dispatch<PM_HHF16>(Ahi, Alo, lda, Bhi, Blo, ldb, M, N, K, sym, tile, blocks, ep, st, ksa,
                          ksb);
  }
  return hipGetLastError();
}

// FP32 tile edge: 64 or 256.  Its matrix-core instruction takes twice as long for the same fragments as
// a BF16 one, so a 64-wide tile is not held back by operand traffic and, four blocks a CU,
// leaves the least of the chip idle: 64 / 128 / 256 wide full N = 1024 40 / 89 / 275 us,
// N = 2048 167 / 175 / 543, N = 3072 527 / 614 / 833, N = 5120 2330 / 2804 / 2780; symmetric
// N = 3072 314 / 470 / 807, N = 4096 702 / 902 / 1067.  Only whole rounds of 256-wide tiles,
// one per CU, are faster: full N = 4096 1189 / 1499 / 1150 us.
int f32_tile_edge(int M, int N, bool sym) {
  const int want = forced_edge(M, N, sym);
  if (want == 64 || want == 256) return want;
  const bool whole = M % 256 == 0 && N % 256 == 0 && grid_blocks(M, N, 256, sym) % 256 == 0;
  return whole ? 256 : 64;
}
int f32_blocks(int M, int N, bool sym) {
  return grid_blocks(M, N, f32_tile_edge(M, N, sym), sym);
}

hipError_t launch_gemm_f32(const float* A, int lda, const float* B, int ldb, int M, int N, int K,
                           bool sym, const EpiParams& ep, hipStream_t st) {
  if (!dims_ok(M, N, K, sym)) return hipErrorInvalidValue;
  const int tile = f32_tile_edge(M, N, sym);
  const int blocks = f32_blocks(M, N, sym);
  if (tile == 256)
    f32_launch<256, 256, 2, 4>(A, lda, B, ldb, M, N, K, sym, blocks, ep, st);
  else
    f32_launch<64, 64, 2, 2>(A, lda, B, ldb, M, N, K, sym, blocks, ep, st);
  return hipGetLastError();
}

hipError_t launch_gemm_f64(const double* A, int lda, const double* B, int ldb, int M, int N, int K,
                           bool sym, const EpiParams& ep, hipStream_t st) {
  if (!dims_ok(M, N, K, sym)) return hipErrorInvalidValue;
  const int tiles = grid_blocks(M, N, 64, sym), whole = f64_whole_tiles(M, N, sym);
  const dim3 grid(tiles + 3 * (tiles - whole));
  if (sym)
    hipLaunchKernelGGL(gemm_f64_kernel<true>, grid, dim3(256), 0, st, A, lda, B, ldb, K, tiles,
                       whole, N / 64, sym_group(), ep);
  else
    hipLaunchKernelGGL(gemm_f64_kernel<false>, grid, dim3(256), 0, st, A, lda, B, ldb, K, tiles,
                       whole, N / 64, tile_group(M, 64), ep);
  return hipGetLastError();
}

}  // namespace zf
