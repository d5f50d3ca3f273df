// One refinement run by a team of workgroups of one XCD inside a single kernel (team.hip).
#pragma once

#include <algorithm>
#include <vector>

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
// Workgroup b of the grid runs as member slots[b].rank of the team, of slots[b].size, of matrix
// slots[b].mat (-1: none).  Workgroup b is dispatched to XCD b % 8, so the members of a team,
// all of one b % 8, share an XCD.
struct TeamSlot {
  int mat;
  short rank, size;
};

// The slots for matrices of padded orders np (multiples of 64): every matrix gets a team in
// proportion to its 32-wide tiles, such that a small batch fills the chip (two workgroups a
// CU) and a large one queues for it, and goes to the XCD with the least work so far, largest
// first.  A team's members are consecutive in their XCD's share of the grid, which is
// dispatched in order, so a team that waits for its last members waits only for teams that
// are complete.
inline void team_slots(const std::vector<int>& np, std::vector<TeamSlot>& slots) {
  const int count = (int)np.size();
  std::vector<int> order(count);
  double tiles = 0.0;
  for (int m = 0; m < count; ++m) {
    order[m] = m;
    tiles += (np[m] / 32) * (double)(np[m] / 32);
  }
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return np[a] > np[b]; });
  // 32-wide tiles a member: what fills 512 places, at most 8 (512 matrices of N = 64 to 256 take
  // 4.0 ms with 4, 3.7 with 8, 4.6 with 16)
  const double per = std::min(std::max(tiles / 512.0, 1.0), 8.0);
  double load[8] = {};
  std::vector<TeamSlot> run[8];
  for (int m : order) {
    const double T = np[m] / 32;
    const int size = std::min(std::max((int)(T * T / per + 0.5), 1), 32);
    int x = 0;
    for (int k = 1; k < 8; ++k)
      if (load[k] < load[x]) x = k;
    load[x] += T * T * (T + 4.0);
    for (int r = 0; r < size; ++r) run[x].push_back(TeamSlot{m, (short)r, (short)size});
  }
  size_t longest = 0;
  for (const auto& r : run) longest = std::max(longest, r.size());
  slots.assign(8 * longest, TeamSlot{-1, 0, 0});
  for (int x = 0; x < 8; ++x)
    for (size_t j = 0; j < run[x].size(); ++j) slots[8 * j + x] = run[x][j];
}

hipError_t launch_team_many(const TeamMat* mats, const TeamSlot* slots, int blocks,
                            const TeamCall& call, hipStream_t st);

}  // namespace zf
