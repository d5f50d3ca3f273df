// A whole refinement in one kernel: for orders where a product takes less than the launch
// that carries it.
//
// A team of up to 64 workgroups (more than 32 only where every product is in FP64) runs
// set-up, both phases and the copy-out of one matrix, meeting between stages instead of
// ending a kernel.  Its members run on one XCD, whose L2 they share, so a meeting needs no
// cache maintenance: every wave waits for its stores to reach L2, one thread per workgroup counts itself in, and later loads of data that the
// kernel has written go past the CU's own cache (sc1).  Measured on gfx950: 1.0-1.2 us per
// meeting of 16-32 workgroups, against 1.9-3.0 us with agent-scope fences over all XCDs, and
// 4-5 us for the end of a kernel and the start of the next.  Workgroup b of a grid is
// dispatched to XCD b % 8; the members compare XCD numbers when they first meet, and if
// they differ the team uses agent-scope fences throughout, so only speed depends on it.
//
// The recursion, the stop test (above_power) and the arithmetic are those of separate
// launches; every member evaluates the stop test from the same partial sums in the same
// order, so the team agrees without another meeting.
//
// A wait is bounded (TeamCall::spin): a member that runs out of time poisons the counter,
// every member leaves, nothing has been written to Z, and the host runs the matrix by
// separate launches.  That happens only if members cannot all become resident, e.g. when
// other processes hold the XCD with waiting teams of their own.
#include <math.h>

#include "zf.h"
#include "zf_index.h"
#include "zf_team.h"
#include "gemm_tiles.inc"

namespace zf {

namespace {

// A matrix's record where nothing writes during the kernel (kernel arguments, or a table).
typedef const __attribute__((address_space(4))) TeamMat* MatArg;

constexpr int kNT = 256;  // threads of a workgroup
// 64-wide BF16x3 tiles on a four-stage ring (64 KB); FP64 tiles need half of it
constexpr int kTeamLds = x3_lds(64, 64, PM_X3, 4, 4);
static_assert(kTeamLds * 2 >= F64Cfg<32>::LDS * 8 && kTeamLds * 2 >= F64Cfg<64>::LDS * 8, "LDS");
static_assert(kTeamLds * 2 >= 64 * 65 * 8, "transposing copies");

struct Team {
  TeamCtl* ctl;
  int rank, size;
  unsigned want;  // arrivals that complete the next meeting
  bool multi;     // members on more than one XCD
  long long spin;
  int* ok;  // LDS
};

__device__ __forceinline__ unsigned ctl_load(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All members have done everything before this, and see what the others wrote.  False (in
// every member alike) if a member gave up waiting.
__device__ __forceinline__ bool team_meet(Team& t) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores are in L2
  __syncthreads();
  if (t.size == 1) return true;
  t.want += t.size;
  if (threadIdx.x == 0) {
    if (t.multi) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    unsigned v = __hip_atomic_fetch_add(&t.ctl->arrived, 1u, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT) + 1u;
    const long long t0 = wall_clock64();
    while (!(v & kTeamPoison) && v < t.want) {
      if (wall_clock64() - t0 > t.spin) {
        // the meeting is off unless it has completed meanwhile: poison only an
        // incomplete count, so that all members take the same way
        unsigned seen = v;
        if (__hip_atomic_compare_exchange_strong(&t.ctl->arrived, &seen, v | kTeamPoison,
                                                 __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
          seen = v | kTeamPoison;
        v = seen;
      } else {
        v = ctl_load(&t.ctl->arrived);
      }
    }
    if (t.multi) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *t.ok = !(v & kTeamPoison);
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*t.ok) != 0;
}

// First meeting: with fences, and every member's XCD number.
__device__ __forceinline__ bool team_join(Team& t) {
  t.multi = true;
  if (threadIdx.x == 0) {
    // HW_REG_XCC_ID (20), bits 3:0
    const unsigned xcc = __builtin_amdgcn_s_getreg((31 << 11) | (0 << 6) | 20) & 15u;
    __hip_atomic_fetch_or(&t.ctl->xcc_mask, 1u << xcc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!team_meet(t)) return false;
  if (t.size > 1) t.multi = __builtin_amdgcn_readfirstlane(__builtin_popcount(ctl_load(&t.ctl->xcc_mask))) != 1;
  return true;
}

// Every member leaves once, whatever happened; the last one resets the meeting point.
__device__ __forceinline__ void team_leave(Team& t) {
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (__hip_atomic_fetch_add(&t.ctl->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
      (unsigned)t.size) {
    __hip_atomic_store(&t.ctl->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&t.ctl->xcc_mask, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&t.ctl->left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---------------------------------------------------------------------------
// stages: a member takes tiles rank, rank + size, ...
// ---------------------------------------------------------------------------
__device__ __forceinline__ void stage_x3(const Team& t, int np, const u16* ah, const u16* al, const u16* bh,
                         const u16* bl, bool sym, const EpiCore& ep, u16* lds, double* red) {
  const int T = np / 64, count = sym ? T * (T + 1) / 2 : T * T;
  for (int k = t.rank; k < count; k += t.size) {
    int ti, tj;
    tile_coords(k, T, sym, ti, tj, 1);
    x3_tile<64, 64, 2, 2, PM_X3, 4, true>(ah, al, 32, bh, bl, 32, np, ti * 64, tj * 64,
                                          sym ? (ti == tj ? 2 : 1) : 0, ep, k, lds, red, 32 * np,
                                          32 * np);
    __syncthreads();
  }
}

// FP64 tiles are 32 wide: they are bound by the XCD's matrix cores, and small orders have few.
__device__ __forceinline__ void stage_f64(const Team& t, int np, const double* a, const double* b, bool sym,
                         const EpiCore& ep, u16* lds, double* red) {
  const int T = np / 32, count = sym ? T * (T + 1) / 2 : T * T;
  using C = F64Cfg<32>;
  for (int k = t.rank; k < count; k += t.size) {
    int ti, tj;
    tile_coords(k, T, sym, ti, tj, 1);
    f64_tile<32, 32, C::WM, C::WN, C::NS, true>(a, np, b, np, np, ti * 32, tj * 32,
                                                sym ? (ti == tj ? 2 : 1) : 0, ep, k,
                                                reinterpret_cast<double*>(lds), red);
    __syncthreads();
  }
}

// Frobenius norm from the partials, the same in every lane of the team.
__device__ __forceinline__ double team_norm(const double* partials, int count) {
  const int lane = threadIdx.x & 63;
  double s = 0.0;
  for (int i = lane; i < count; i += 64) s += load_f64<true>(partials + i);
  return sqrt(wave_sum(s));
}

// FP32 master -> FP64 row-major and transposed, 64 x 64 tiles through LDS.
__device__ __forceinline__ void team_widen(const Team& t, MatArg m, int cur, u16* lds) {
  float* tv = reinterpret_cast<float*>(lds);  // 64 x 65
  const int T = m->np / 64, np = m->np;
  for (int k = t.rank; k < T * T; k += t.size) {
    const int i0 = (k / T) * 64, j0 = (k % T) * 64;
#pragma unroll 4
    for (int e = threadIdx.x; e < 32 * 64; e += kNT) {
      const int r = e >> 5, c = 2 * (e & 31);
      const float2 f =
          __builtin_bit_cast(float2, load8<true>(m->z32[cur] + (size_t)(i0 + r) * np + j0 + c));
      *reinterpret_cast<double2*>(m->z64r[cur] + (size_t)(i0 + r) * np + j0 + c) =
          double2{(double)f.x, (double)f.y};
      tv[r * 65 + c] = f.x;
      tv[r * 65 + c + 1] = f.y;
    }
    __syncthreads();
#pragma unroll 4
    for (int e = threadIdx.x; e < 32 * 64; e += kNT) {
      const int r = e >> 5, c = 2 * (e & 31);
      *reinterpret_cast<double2*>(m->z64c[cur] + (size_t)(j0 + r) * np + i0 + c) =
          double2{(double)tv[c * 65 + r], (double)tv[(c + 1) * 65 + r]};
    }
    __syncthreads();
  }
}

// S -> BF16 pair and FP64 copy (zero-padded), its row sums, and Z0 (given, or I / sqrt(g) with
// g the largest row sum) in the layouts the first phase reads.
__device__ __forceinline__ bool team_setup(Team& t, MatArg m, const TeamCall& call, u16* lds) {
  const int n = m->n, np = m->np, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool w64 = call.fp64 || call.refine;
  for (int i = 4 * t.rank + wave; i < np; i += 4 * t.size) {
    double s = 0.0;
    for (int j = lane; j < np; j += 64) {
      const double a = (i < n && j < n) ? m->S[(size_t)i * n + j] : 0.0;
      s += fabs(a);
      if (w64) m->s64[(size_t)i * np + j] = a;
      if (!call.fp64) {
        u16 h, l;
        split_bf16((float)a, h, l);
        const size_t k = kb_offset(i, j, np);
        m->s_hi[k] = h;
        m->s_lo[k] = l;
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) m->rowsum[i] = s;
  }
  double c = 0.0;
  if (!m->Z0) {
    if (!team_meet(t)) return false;
    double g = 0.0;
    for (int i = lane; i < n; i += 64) g = fmax(g, load_f64<true>(m->rowsum + i));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) g = fmax(g, __shfl_xor(g, off, 64));
    c = 1.0 / sqrt(g);
  }
  double* tv = reinterpret_cast<double*>(lds);  // 64 x 65
  const int T = np / 64;
  for (int k = t.rank; k < T * T; k += t.size) {
    const int i0 = (k / T) * 64, j0 = (k % T) * 64;
    for (int e = threadIdx.x; e < 64 * 64; e += kNT) {
      const int r = e >> 6, q = e & 63, i = i0 + r, j = j0 + q;
      double v = 0.0;
      if (m->Z0) {
        if (i < n && j < n) v = m->Z0[(size_t)i * n + j];
      } else if (i == j && i < n) {
        v = c;
      }
      if (call.fp64) {
        m->z64r[0][(size_t)i * np + j] = v;
      } else {
        const float f = (float)v;
        m->z32[0][(size_t)i * np + j] = f;
        u16 h, l;
        split_bf16(f, h, l);
        const size_t o = kb_offset(i, j, np);
        m->zr_hi[0][o] = h;
        m->zr_lo[0][o] = l;
      }
      tv[r * 65 + q] = v;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 64; e += kNT) {
      const int r = e >> 6, q = e & 63;  // transposed row j0 + r, column i0 + q
      const double v = tv[q * 65 + r];
      if (call.fp64) {
        m->z64c[0][(size_t)(j0 + r) * np + i0 + q] = v;
      } else {
        u16 h, l;
        split_bf16((float)v, h, l);
        const size_t o = kb_offset(j0 + r, i0 + q, np);
        m->zc_hi[0][o] = h;
        m->zc_lo[0][o] = l;
      }
    }
    __syncthreads();
  }
  return team_meet(t);
}

// The refinement as a sequence of product stages with a meeting after each.  One place in
// the code runs the BF16x3 products and one the FP64 products, so the kernel's loop stays in
// the instruction cache; every decision is made wave-uniform, so operands stay in scalar
// registers.
enum { ST_EVAL1, ST_EVAL2, ST_HORNER, ST_UPDATE };

__device__ __forceinline__ void team_solve(Team& t, MatArg m, const TeamCall& call,
                                           u16* lds, double* red) {
  bool up = team_join(t);
  if (up && call.setup) up = team_setup(t, m, call, lds);
  const int np = m->np, order = call.order;
  const bool fp64 = call.fp64 != 0;
  bool high = fp64;  // FP64 residual and master Z
  int cur = 0, hist_len = 0, it = 0, hk = 0, op = ST_EVAL1;
  int status = 0, flags = 0, upd_l = 0, upd_h = 0, evals_l = 0, evals_h = 0;
  double prev = 0.0, err = 0.0, err_l = 0.0, err_h = 0.0;
  while (up) {
    // operands are read when a stage needs them: held across stages, their addresses would
    // take more scalar registers than there are
    asm volatile("" : "+s"(m));
    EpiCore e;
    memset(&e, 0, sizeof e);
    e.beta = 1.0;
    e.ld = np;
    e.n_valid = m->n;
    e.kb = 1;
    const bool use64 = (op == ST_EVAL1 || op == ST_EVAL2) ? high : fp64;
    const int nxt = cur ^ 1;
    const u16 *ah = nullptr, *al = nullptr, *bh = nullptr, *bl = nullptr;
    const double *a64 = nullptr, *b64 = nullptr;
    bool sym = false;
    if (op == ST_EVAL1) {  // A^T = Z^T S
      ah = m->zc_hi[cur];
      al = m->zc_lo[cur];
      bh = m->s_hi;
      bl = m->s_lo;
      a64 = m->z64c[cur];
      b64 = m->s64;
      if (high) {
        e.o64 = m->a64t;
      } else {
        e.ohi = m->at_hi;
        e.olo = m->at_lo;
      }
    } else if (op == ST_EVAL2) {  // delta = I - Z^T A
      ah = m->zc_hi[cur];
      al = m->zc_lo[cur];
      bh = m->at_hi;
      bl = m->at_lo;
      a64 = m->z64c[cur];
      b64 = m->a64t;
      sym = true;
      e.beta = -1.0;
      e.gamma = 1.0;
      e.partials = m->partials;
      if (high) e.o64 = e.ot64 = m->d64;
      if (!fp64) {
        e.ohi = e.othi = m->d_hi;
        e.olo = e.otlo = m->d_lo;
      }
    } else if (op == ST_HORNER) {  // U_k = c_k delta + delta U_{k+1}, U_order = c_order I
      const bool first = hk == order - 1, to_q = (hk & 1) != 0;
      sym = true;
      ah = m->d_hi;
      al = m->d_lo;
      bh = first ? m->d_hi : to_q ? m->u_hi : m->q_hi;
      bl = first ? m->d_lo : to_q ? m->u_lo : m->q_lo;
      a64 = m->d64;
      b64 = first ? m->d64 : to_q ? m->u64 : m->q64;
      e.alpha = call.c[hk];
      e.beta = first ? call.c[order] : 1.0;
      if (high) {
        e.d64 = m->d64;
      } else {
        e.dhi = m->d_hi;
        e.dlo = m->d_lo;
      }
      if (fp64) {
        e.o64 = e.ot64 = to_q ? m->q64 : m->u64;
      } else {
        e.ohi = e.othi = to_q ? m->q_hi : m->u_hi;
        e.olo = e.otlo = to_q ? m->q_lo : m->u_lo;
      }
    } else {  // Z' = Z + Z Q
      ah = m->zr_hi[cur];
      al = m->zr_lo[cur];
      bh = order == 1 ? m->d_hi : m->q_hi;
      bl = order == 1 ? m->d_lo : m->q_lo;
      a64 = m->z64r[cur];
      b64 = order == 1 ? m->d64 : m->q64;
      e.alpha = 1.0;
      e.beta = order == 1 ? call.c[1] : 1.0;
      if (high) {
        e.d64 = m->z64r[cur];
        e.o64 = m->z64r[nxt];
        e.ot64 = m->z64c[nxt];
      } else {
        e.d32 = m->z32[cur];
        e.o32 = m->z32[nxt];
        e.othi = m->zc_hi[nxt];
        e.otlo = m->zc_lo[nxt];
      }
      if (!fp64) {
        e.ohi = m->zr_hi[nxt];
        e.olo = m->zr_lo[nxt];
      }
    }
    if (use64) stage_f64(t, np, a64, b64, sym, e, lds, red);
    else stage_x3(t, np, ah, al, bh, bl, sym, e, lds, red);
    up = team_meet(t);
    if (!up) break;
    if (op == ST_EVAL1) {
      op = ST_EVAL2;
      continue;
    }
    if (op == ST_HORNER) {
      if (--hk == 0) op = ST_UPDATE;
      continue;
    }
    if (op == ST_UPDATE) {
      cur = nxt;
      prev = err;
      ++it;
      op = ST_EVAL1;
      continue;
    }
    // the stop test of Algorithm 2
    const int T = np / (high ? 32 : 64);
    err = team_norm(m->partials, T * (T + 1) / 2);
    if (t.rank == 0 && threadIdx.x == 0 && hist_len < call.hist_cap) m->hist[hist_len] = err;
    ++hist_len;
    if (high) ++evals_h;
    else ++evals_l;
    int code = 0;  // 1: stop with this iterate, 2: with the previous one, 3: not finite
    if (!isfinite(err)) code = 3;
    else if (it > 0 && (call.rule == ZF_STOP_MONOTONE ? err >= prev
                                                      : above_power(err, prev, order + 1)))
      code = err > prev ? 2 : 1;
    code = __builtin_amdgcn_readfirstlane(code);
    if (code == 3) {
      status = ZF_ERR_NONFINITE;
      break;
    }
    const bool capped = code == 0 && it >= (high && !fp64 ? call.max_h : call.max_l);
    if (code == 0 && !capped) {
      hk = order - 1;
      op = hk > 0 ? ST_HORNER : ST_UPDATE;
      continue;
    }
    if (capped) flags |= ZF_WARN_MAXSWEEPS;
    if (code == 2) cur ^= 1;  // still in the other buffer
    const int upd = code == 2 ? it - 1 : it;
    const double chosen = code == 2 ? prev : err;
    if (high) {
      upd_h = upd;
      err_h = chosen;
      break;
    }
    upd_l = upd;
    err_l = chosen;
    if (!call.refine) break;
    team_widen(t, m, cur, lds);
    up = team_meet(t);
    high = true;
    it = 0;
    op = ST_EVAL1;
  }
  if (up && m->Z && status == 0) {
    const int n = m->n;
    for (int i = t.rank; i < n; i += t.size)
      for (int j = threadIdx.x; j < n; j += kNT)
        m->Z[(size_t)i * n + j] =
            high ? load_f64<true>(m->z64r[cur] + (size_t)i * np + j)
                 : (double)__hip_atomic_load(m->z32[cur] + (size_t)i * np + j, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
  }
  if (t.rank == 0 && threadIdx.x == 0) {
    TeamOut o;
    o.done = up;
    o.status = status;
    o.flags = flags;
    o.cur = cur;
    o.upd_l = upd_l;
    o.upd_h = upd_h;
    o.evals_l = evals_l;
    o.evals_h = evals_h;
    o.hist_len = hist_len;
    o.err_l = err_l;
    o.err_h = err_h;
    *m->out = o;
  }
  team_leave(t);
}

// The team of one matrix: the grid's workgroups on XCD 0 (every eighth one).
__global__ void __launch_bounds__(kNT, 2) team_one_kernel(TeamMat mat, TeamCall call, int size) {
  __shared__ __attribute__((aligned(16))) u16 lds[kTeamLds];
  __shared__ double red[4];
  __shared__ int ok;
  if (blockIdx.x & 7) return;
  (void)mat;  // read as the first of the kernel's arguments
  const MatArg m = (MatArg)__builtin_amdgcn_kernarg_segment_ptr();
  Team t{m->ctl, (int)(blockIdx.x >> 3), size, 0u, true, call.spin, &ok};
  team_solve(t, m, call, lds, red);
}

__global__ void __launch_bounds__(kNT, 2) team_many_kernel(const TeamMat* __restrict__ mats,
                                                           const TeamSlot* __restrict__ slots,
                                                           TeamCall call) {
  __shared__ __attribute__((aligned(16))) u16 lds[kTeamLds];
  __shared__ double red[4];
  __shared__ int ok;
  const TeamSlot s = slots[blockIdx.x];
  if (s.mat < 0) return;
  const MatArg m = (MatArg)(uintptr_t)(mats + s.mat);
  Team t{m->ctl, s.rank, s.size, 0u, true, call.spin, &ok};
  team_solve(t, m, call, lds, red);
}

}  // namespace

hipError_t launch_team_one(const TeamMat& m, const TeamCall& call, int size, hipStream_t st) {
  if (m.np <= 0 || m.np % 64 != 0 || m.n > m.np || size < 1 || size > kTeamMaxSize)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(team_one_kernel, dim3(8 * (size - 1) + 1), dim3(kNT), 0, st, m, call, size);
  return hipGetLastError();
}

hipError_t launch_team_many(const TeamMat* mats, const TeamSlot* slots, int blocks,
                            const TeamCall& call, hipStream_t st) {
  if (blocks < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(team_many_kernel, dim3(blocks), dim3(kNT), 0, st, mats, slots, call);
  return hipGetLastError();
}

}  // namespace zf
