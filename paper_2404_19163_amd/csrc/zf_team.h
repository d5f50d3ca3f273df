// One refinement run by a team of workgroups of one XCD inside a single kernel (team.hip).
#pragma once

#include "zf_internal.h"

namespace zf {

constexpr int kTeamMaxSize = 64;  // workgroups of a team: two per CU of an XCD

// Meeting point of a team, zero between launches (the last workgroup to leave resets it).
struct TeamCtl {
  unsigned arrived;   // arrivals so far; kTeamPoison once a wait has run out
  unsigned left;      // workgroups that have ended
  unsigned xcc_mask;  // XCDs that members run on
  unsigned pad[29];   // a line of its own
};
constexpr unsigned kTeamPoison = 0x80000000u;

// What a team reports of its matrix.
struct TeamOut {
  int done;  // 0: the team gave up waiting; nothing was written to Z
  int status, flags;
  int cur;  // which of the ping-pong buffers holds the result
  int upd_l, upd_h, evals_l, evals_h, hist_len;
  double err_l, err_h;
};

// Buffers of one matrix.  Pairs are K-blocked (kb_offset), np a multiple of 64.
struct TeamMat {
  int n, np;
  u16 *s_hi, *s_lo, *zr_hi[2], *zr_lo[2], *zc_hi[2], *zc_lo[2];
  u16 *at_hi, *at_lo, *d_hi, *d_lo, *q_hi, *q_lo, *u_hi, *u_lo;
  float* z32[2];
  double *s64, *z64r[2], *z64c[2], *a64t, *d64, *q64, *u64;
  double* partials;  // (np / 32)(np / 32 + 1) / 2
  double* rowsum;    // np (set-up only)
  const double *S, *Z0;  // caller's matrices (set-up only); Z0 may be null
  double* Z;             // caller's result, or null: left in the buffers
  double* hist;
  TeamOut* out;
  TeamCtl* ctl;
};

// What the matrices of a launch share.
struct TeamCall {
  int order, rule, max_l, max_h, hist_cap;
  int fp64;    // every product in FP64 (no first phase)
  int refine;  // FP64-residual refinement phase after the BF16x3 phase
  int setup;   // split S and form Z0 in the kernel
  double c[8];
  long long spin;  // longest wait for a team, in ticks of the 100 MHz clock
};

// A late team says that its XCD is held, as a rule by other processes' teams that wait for
// members too.  The next calls then go by launches at once instead of waiting in vain.
struct TeamRest {
  int calls = 0;  // calls still to go by launches
  bool team() { return calls == 0 || calls-- == 0; }  // whether the next call is for a team
  void late(int rest) { calls = rest; }
};

// zf_api.hip: TeamCall::spin of a call (a batch's teams also wait for the teams ahead of them),
// and the calls that go by launches after a late team.
long long team_spin_ticks(bool batch);
int team_rest_calls();

// One matrix, its team on one XCD.
hipError_t launch_team_one(const TeamMat& m, const TeamCall& call, int size, hipStream_t st);
// first[b] of the grid's workgroups: b runs as rank[b] of matrix mat[b]'s team of size[b]
// (mat[b] < 0: none).  Members of a team are on one XCD when consecutive in b % 8 classes.
struct TeamSlot {
  int mat;
  short rank, size;
};
hipError_t launch_team_many(const TeamMat* mats, const TeamSlot* slots, int blocks,
                            const TeamCall& call, hipStream_t st);

}  // namespace zf
