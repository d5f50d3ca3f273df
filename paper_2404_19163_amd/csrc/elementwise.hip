// Bandwidth-bound helpers of the refinement path (gfx950): operand preparation
// (split, zero padding, layouts), the scaled-identity guess, the final copy-out
// and the deterministic reduction of the per-tile norm partials.
//
// Every matrix kernel here moves 4 consecutive elements of a row per thread, in 16-byte
// accesses: 8 rows of 128 columns a block where the layout is kept, one 32 x 32 tile a
// block, through LDS, where a transposed copy is written.  One such access per operand and
// thread, and thousands of blocks from N = 1000 on, so small orders wait for one memory
// latency only.  Bound by memory.  Against one element per access (64 x 64 tiles walked in
// 16 steps for the transposed copies): widen with FP16 pairs at N = 1024 13.9 -> 4.3 us; N =
// 4096 identity start 59 -> 29 us, widen 72 -> 63 us, S 59 -> 54 us.
#include "zf_internal.h"

namespace zf {

static inline int grid_for(size_t work, int block) {
  size_t g = (work + block - 1) / block;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

__device__ __forceinline__ void load4(const double* p, int j, int n, double v[4]) {
  if (j + 3 < n) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = p[j + k];
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = j + k < n ? p[j + k] : 0.0;
  }
}
template <typename T>
__device__ __forceinline__ void store4(double* p, const T v[4]) {
  reinterpret_cast<double2*>(p)[0] = double2{(double)v[0], (double)v[1]};
  reinterpret_cast<double2*>(p)[1] = double2{(double)v[2], (double)v[3]};
}
__device__ __forceinline__ void store4(float* p, const float f[4]) {
  *reinterpret_cast<float4*>(p) = float4{f[0], f[1], f[2], f[3]};
}
__device__ __forceinline__ void store_pair4(u16* hi, u16* lo, size_t k, const float f[4], int fmt) {
  u32x2_t h, l;
  split_pair4(f, h, l, fmt);
  *reinterpret_cast<u32x2_t*>(hi + k) = h;
  *reinterpret_cast<u32x2_t*>(lo + k) = l;
}

// ---------------------------------------------------------------------------
// S (n x n, ld_src) -> padded np x np: BF16 hi/lo pair (Sec. III.A: the FP64
// value is first rounded to FP32, then split) in the K-blocked layout of the
// matrix-core operands (kb_offset), optionally an FP64 / FP32 row-major copy.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
    split_pad_kernel(const double* __restrict__ src, int n, int ld_src, int np,
                     u16* __restrict__ hi, u16* __restrict__ lo, double* __restrict__ c64,
                     float* __restrict__ c32, int fmt, int* __restrict__ clear) {
  if (clear && blockIdx.x == 0 && threadIdx.x < 4) clear[threadIdx.x] = 0;
  const int across = (np + 127) / 128;
  const int i = (int)(blockIdx.x / across) * 8 + (threadIdx.x >> 5);
  const int j = (int)(blockIdx.x % across) * 128 + 4 * (threadIdx.x & 31);
  if (j >= np) return;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < n) load4(src + (size_t)i * ld_src, j, n, v);
  const float f[4] = {rounded_f32((float)v[0]), rounded_f32((float)v[1]),
                      rounded_f32((float)v[2]), rounded_f32((float)v[3])};
  const size_t e = (size_t)i * np + j;
  if (hi) store_pair4(hi, lo, kb_offset(i, j, np), f, fmt == 2 ? PAIR_F16 : PAIR_BF16);
  if (c64) store4(c64 + e, v);
  if (c32) store4(c32 + e, f);
}

hipError_t launch_split_pad(const double* src, int n, int ld_src, int np, u16* hi, u16* lo,
                            double* copy64, float* copy32, bool transpose_copy, int fmt,
                            hipStream_t st, int* clear) {
  (void)transpose_copy;
  if (np % 64 != 0 || n > np) return hipErrorInvalidValue;
  hipLaunchKernelGGL(split_pad_kernel, dim3((np + 127) / 128 * (np / 8)), dim3(256), 0, st, src, n,
                     ld_src, np, hi, lo, copy64, copy32, fmt, clear);
  return hipGetLastError();
}

__global__ void split_flat_kernel(const double* __restrict__ src, int64_t count, u16* __restrict__ hi,
                                  u16* __restrict__ lo, int fmt) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (int64_t)gridDim.x * blockDim.x) {
    const float x = (float)src[e];
    u16 h, l;
    if (fmt == 2) split_f16(x, h, l);
    else split_bf16(x, h, l);
    hi[e] = h;
    lo[e] = l;
  }
}

hipError_t launch_split_flat(const double* src, int64_t count, u16* hi, u16* lo, int fmt,
                             hipStream_t st) {
  hipLaunchKernelGGL(split_flat_kernel, dim3(grid_for((size_t)count, 256)), dim3(256), 0, st, src,
                     count, hi, lo, fmt);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gershgorin bound g = max_i sum_j |S_ij| (FP64).  One wave per row, then one
// block takes the maximum.
// ---------------------------------------------------------------------------
__global__ void row_abs_kernel(const double* __restrict__ S, int n, int ld, double* __restrict__ rs) {
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (wave >= n) return;
  const double* row = S + (size_t)wave * ld;
  double s = 0.0;
  for (int j = lane; j < n; j += 512) {  // 8 loads in flight; one running sum, in order
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = j + 64 * k < n ? row[j + 64 * k] : 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += fabs(v[k]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) rs[wave] = s;
}

__global__ void max_kernel(const double* __restrict__ v, int n, double* __restrict__ out) {
  __shared__ double red[256];
  double m = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) m = fmax(m, v[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0];
}

hipError_t launch_row_abs_max(const double* S, int n, int ld, double* row_sums, double* g_out,
                              hipStream_t st) {
  const int waves_per_block = 4;
  hipLaunchKernelGGL(row_abs_kernel, dim3((n + waves_per_block - 1) / waves_per_block),
                     dim3(64 * waves_per_block), 0, st, S, n, ld, row_sums);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(max_kernel, dim3(1), dim3(256), 0, st, row_sums, n, g_out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Z0 = I / sqrt(g) in every layout the sweep reads (g read on the device).  The
// pairs are K-blocked (kb_offset), where the row-major and the transposed pair of
// the (symmetric) Z0 coincide; the loop walks them in storage order.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
    init_identity_kernel(const double* __restrict__ g, int n, int np, float* __restrict__ z32,
                         double* __restrict__ z64r, double* __restrict__ z64c,
                         u16* __restrict__ zr_hi, u16* __restrict__ zr_lo,
                         u16* __restrict__ zc_hi, u16* __restrict__ zc_lo) {
  const double c = 1.0 / sqrt(g[0]);
  const unsigned total = (unsigned)((size_t)np * np / 4), across = (unsigned)np / 4;
  for (unsigned e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
    // storage elements 4 e .. 4 e + 3 of row-major matrices ...
    const int i = (int)(e / across), d = i < n ? i - 4 * (int)(e % across) : -1;
    const double v[4] = {d == 0 ? c : 0.0, d == 1 ? c : 0.0, d == 2 ? c : 0.0, d == 3 ? c : 0.0};
    const size_t at = (size_t)e * 4;
    if (z32) {
      const float f[4] = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
      store4(z32 + at, f);
    }
    if (z64r) store4(z64r + at, v);
    if (z64c) store4(z64c + at, v);
    if (zr_hi || zc_hi) {  // ... and of K-blocked pairs: k block, row, k % 32
      const unsigned row8 = e / 8, rr = row8 % (unsigned)np;
      const int k = (int)(row8 / (unsigned)np) * 32 + (int)(e % 8) * 4;
      const int dk = (int)rr < n ? (int)rr - k : -1;
      const float fc = rounded_f32((float)c);
      const float f[4] = {dk == 0 ? fc : 0.f, dk == 1 ? fc : 0.f, dk == 2 ? fc : 0.f,
                          dk == 3 ? fc : 0.f};
      u32x2_t h, l;
      split_pair4(f, h, l, PAIR_BF16);
      if (zr_hi) {
        *reinterpret_cast<u32x2_t*>(zr_hi + at) = h;
        *reinterpret_cast<u32x2_t*>(zr_lo + at) = l;
      }
      if (zc_hi) {
        *reinterpret_cast<u32x2_t*>(zc_hi + at) = h;
        *reinterpret_cast<u32x2_t*>(zc_lo + at) = l;
      }
    }
  }
}

hipError_t launch_init_identity(const double* g, int n, int np, float* z32, double* z64r,
                                double* z64c, u16* zr_hi, u16* zr_lo, u16* zc_hi, u16* zc_lo,
                                hipStream_t st) {
  const size_t total = (size_t)np * np / 4;
  if (np % 64 != 0 || np > 65536) return hipErrorInvalidValue;
  hipLaunchKernelGGL(init_identity_kernel, dim3(grid_for(total, 256)), dim3(256), 0, st, g, n, np,
                     z32, z64r, z64c, zr_hi, zr_lo, zc_hi, zc_lo);
  return hipGetLastError();
}

// Given Z0 (n x n, ld n): padded copies in row-major and transposed layouts (the
// pairs K-blocked, kb_offset).  The pairs are the split of Z0's FP32 value.
__device__ __forceinline__ void given_tile(const double* __restrict__ Z0, int n, int np, int i0,
                                           int j0, float* z32, double* z64r, double* z64c,
                                           u16* zr_hi, u16* zr_lo, u16* zc_hi, u16* zc_lo,
                                           double (*t)[33]) {
  const int r = threadIdx.x >> 3, c = 4 * (threadIdx.x & 7);
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  if (i0 + r < n) load4(Z0 + (size_t)(i0 + r) * n, j0 + c, n, v);
  const size_t idx = (size_t)(i0 + r) * np + j0 + c;
  float f[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) f[k] = rounded_f32((float)v[k]);
  if (z32) store4(z32 + idx, f);
  if (z64r) store4(z64r + idx, v);
  if (zr_hi) store_pair4(zr_hi, zr_lo, kb_offset(i0 + r, j0 + c, np), f, PAIR_BF16);
  if (!z64c && !zc_hi) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) t[r][c + k] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {  // transposed row j0 + r, columns i0 + c ..
    v[k] = t[c + k][r];
    f[k] = rounded_f32((float)v[k]);
  }
  if (z64c) store4(z64c + (size_t)(j0 + r) * np + i0 + c, v);
  if (zc_hi) store_pair4(zc_hi, zc_lo, kb_offset(j0 + r, i0 + c, np), f, PAIR_BF16);
}

__global__ void __launch_bounds__(256) init_given_kernel(const double* __restrict__ Z0, int n,
                                                         int np, float* __restrict__ z32,
                                                         double* __restrict__ z64r,
                                                         double* __restrict__ z64c,
                                                         u16* __restrict__ zr_hi,
                                                         u16* __restrict__ zr_lo,
                                                         u16* __restrict__ zc_hi,
                                                         u16* __restrict__ zc_lo) {
  __shared__ double t[32][33];
  const int T = np / 32;
  given_tile(Z0, n, np, (int)(blockIdx.x / T) * 32, (int)(blockIdx.x % T) * 32, z32, z64r, z64c,
             zr_hi, zr_lo, zc_hi, zc_lo, t);
}

// The residual's operands in one launch: S padded (first half of the grid), Z transposed and
// padded (second half), and 4 words set to 0.
__global__ void __launch_bounds__(256) stage_residual_kernel(const double* __restrict__ S,
                                                             const double* __restrict__ Z, int n,
                                                             int np, double* __restrict__ s64,
                                                             double* __restrict__ zc64,
                                                             int* __restrict__ clear) {
  __shared__ double t[32][33];
  if (blockIdx.x == 0 && threadIdx.x < 4) clear[threadIdx.x] = 0;
  const int T = np / 32;
  const bool z = blockIdx.x >= (unsigned)(T * T);
  const int b = (int)blockIdx.x - (z ? T * T : 0), i0 = b / T * 32, j0 = b % T * 32;
  given_tile(z ? Z : S, n, np, i0, j0, nullptr, z ? nullptr : s64, z ? zc64 : nullptr, nullptr,
             nullptr, nullptr, nullptr, t);
}

hipError_t launch_stage_residual(const double* S, const double* Z, int n, int np, double* s64,
                                 double* zc64, int* clear, hipStream_t st) {
  if (np % 64 != 0 || n > np) return hipErrorInvalidValue;
  const int T = np / 32;
  hipLaunchKernelGGL(stage_residual_kernel, dim3(2 * T * T), dim3(256), 0, st, S, Z, n, np, s64,
                     zc64, clear);
  return hipGetLastError();
}

hipError_t launch_init_given(const double* Z0, int n, int np, float* z32, double* z64r,
                             double* z64c, u16* zr_hi, u16* zr_lo, u16* zc_hi, u16* zc_lo,
                             hipStream_t st) {
  if (np % 64 != 0 || n > np) return hipErrorInvalidValue;
  const int T = np / 32;
  hipLaunchKernelGGL(init_given_kernel, dim3(T * T), dim3(256), 0, st, Z0, n, np, z32, z64r, z64c,
                     zr_hi, zr_lo, zc_hi, zc_lo);
  return hipGetLastError();
}

// FP32 matrix X (np x np, row-major) -> any of: FP64 row-major, FP64 transposed,
// FP32 transposed, and 16-bit pairs (format fmt) of scale * X in the K-blocked
// layout of the matrix-core operands (kb_offset), of X and/or of its transpose.
// scale is a power of two (exact).
__global__ void __launch_bounds__(256) widen_kernel(const float* __restrict__ z32, int np,
                                                    double* __restrict__ z64r,
                                                    double* __restrict__ z64c,
                                                    float* __restrict__ zc32, u16* __restrict__ prh,
                                                    u16* __restrict__ prl, u16* __restrict__ pch,
                                                    u16* __restrict__ pcl, float scale, int fmt) {
  __shared__ float t[32][33];
  const int T = np / 32;
  const int i0 = (int)(blockIdx.x / T) * 32, j0 = (int)(blockIdx.x % T) * 32;
  const int r = threadIdx.x >> 3, c = 4 * (threadIdx.x & 7);
  const size_t idx = (size_t)(i0 + r) * np + j0 + c;
  const float4 x = *reinterpret_cast<const float4*>(z32 + idx);
  float f[4] = {x.x, x.y, x.z, x.w}, p[4];
  if (z64r) store4(z64r + idx, f);
  if (prh) {
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = f[k] * scale;
    store_pair4(prh, prl, kb_offset(i0 + r, j0 + c, np), p, fmt);
  }
  if (!z64c && !zc32 && !pch) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) t[r][c + k] = f[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) f[k] = t[c + k][r];  // transposed row j0 + r, columns i0 + c ..
  const size_t tdx = (size_t)(j0 + r) * np + i0 + c;
  if (z64c) store4(z64c + tdx, f);
  if (zc32) store4(zc32 + tdx, f);
  if (pch) {
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = f[k] * scale;
    store_pair4(pch, pcl, kb_offset(j0 + r, i0 + c, np), p, fmt);
  }
}

hipError_t launch_widen(const float* z32, int np, double* z64r, double* z64c, hipStream_t st,
                        float* zc32, u16* prh, u16* prl, u16* pch, u16* pcl, float scale,
                        int fmt) {
  if (np % 64 != 0) return hipErrorInvalidValue;
  const int T = np / 32;
  hipLaunchKernelGGL(widen_kernel, dim3(T * T), dim3(256), 0, st, z32, np, z64r, z64c, zc32, prh,
                     prl, pch, pcl, scale, fmt);
  return hipGetLastError();
}

// The valid n x n block of a padded matrix.
template <typename T>
__global__ void __launch_bounds__(256)
    unpad_kernel(const T* __restrict__ src, int np, int n, double* __restrict__ dst) {
  const int across = (n + 127) / 128;
  const int i = (int)(blockIdx.x / across) * 4 + (threadIdx.x >> 6);
  const int j = (int)(blockIdx.x % across) * 128 + 2 * (threadIdx.x & 63);
  if (i >= n || j >= n) return;
  const T* s = src + (size_t)i * np + j;  // np is a multiple of 64: both are inside
  const double v0 = (double)s[0], v1 = (double)s[1];
  double* d = dst + (size_t)i * n + j;
  d[0] = v0;
  if (j + 1 < n) d[1] = v1;
}

template <typename T>
static hipError_t unpad(const T* src, int np, int n, double* dst, hipStream_t st) {
  if (np % 64 != 0 || n > np) return hipErrorInvalidValue;
  hipLaunchKernelGGL(unpad_kernel<T>, dim3((n + 127) / 128 * ((n + 3) / 4)), dim3(256), 0, st, src,
                     np, n, dst);
  return hipGetLastError();
}
hipError_t launch_unpad_f64(const double* src, int np, int n, double* dst, hipStream_t st) {
  return unpad(src, np, n, dst, st);
}
hipError_t launch_unpad_f32(const float* src, int np, int n, double* dst, hipStream_t st) {
  return unpad(src, np, n, dst, st);
}

// ---------------------------------------------------------------------------
// ||.||_F from per-tile partial sums: fixed summation order (bitwise repeatable).
// ---------------------------------------------------------------------------
__global__ void norm_finalize_kernel(const double* __restrict__ partials, int count, double* out,
                                     double div) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < count; i += 256) s += partials[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sqrt(red[0]) / div;
}

hipError_t launch_norm_finalize(const double* partials, int count, double* out, hipStream_t st,
                                double div) {
  hipLaunchKernelGGL(norm_finalize_kernel, dim3(1), dim3(256), 0, st, partials, count, out, div);
  return hipGetLastError();
}

// M's strict lower triangle from its upper (np x np).
__global__ void mirror_upper_kernel(double* M, int np) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y;
  if (j < i) M[(size_t)i * np + j] = M[(size_t)j * np + i];
}

hipError_t launch_mirror_upper(double* M, int np, hipStream_t st) {
  if (np % 64 != 0 || np > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mirror_upper_kernel, dim3((np + 255) / 256, np), dim3(256), 0, st, M, np);
  return hipGetLastError();
}

__global__ void fill_zero_kernel(uint32_t* p, size_t words) {
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < words;
       e += (size_t)gridDim.x * blockDim.x)
    p[e] = 0u;
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t st) {
  const size_t words = bytes / 4;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(words, 256)), dim3(256), 0, st, (uint32_t*)p, words);
  return hipGetLastError();
}

}  // namespace zf
