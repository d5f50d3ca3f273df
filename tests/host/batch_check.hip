// Host-only check of the batched path's host arithmetic, the ratio stop rule and the blocks'
// XCDs (zf_index.h), and of the teams' slots and rests (zf_team.h), built and run by
// tests/test_host_batch.py under AddressSanitizer and UBSan.  Prints "ok <checks>" or the
// first failure and exits non-zero.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

#include "zf_index.h"
#include "zf_team.h"

using namespace zf;

static long g_checks = 0;
#define CHECK(cond, ...)                                 \
  do {                                                   \
    ++g_checks;                                          \
    if (!(cond)) {                                       \
      fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); \
      fprintf(stderr, __VA_ARGS__);                      \
      fprintf(stderr, "\n");                             \
      exit(1);                                           \
    }                                                    \
  } while (0)

// results_overlap_inputs against every pair of ranges; addresses are never dereferenced
static void overlaps(std::mt19937& rng) {
  auto at = [](int word) { return reinterpret_cast<double*>((uintptr_t)(4096 + 8 * word)); };
  int hits = 0;
  for (int t = 0; t < 20000; ++t) {
    const int count = 1 + (int)(rng() % 6), span = 20 + (int)(rng() % 400);
    std::vector<int> n(count), s(count), z0(count), z(count);
    std::vector<const double*> S(count), Z0(count);
    std::vector<double*> Z(count);
    for (int m = 0; m < count; ++m) {
      n[m] = 1 + (int)(rng() % 4);
      s[m] = (int)(rng() % span);
      z[m] = (int)(rng() % span);
      z0[m] = rng() % 3 ? (int)(rng() % span) : -1;
      if (rng() % 4 == 0) z0[m] = z[m];  // the factor replaced in place
      S[m] = at(s[m]);
      Z[m] = at(z[m]);
      Z0[m] = z0[m] < 0 ? nullptr : at(z0[m]);
    }
    const bool none = rng() % 5 == 0;  // no Z0 array at all
    auto meets = [&](int a, int na, int b, int nb) { return a < b + nb * nb && b < a + na * na; };
    bool want = false;
    for (int m = 0; m < count; ++m)
      for (int k = 0; k < count; ++k)
        if (k != m)
          want |= meets(z[m], n[m], s[k], n[k]) ||
                  (!none && z0[k] >= 0 && meets(z[m], n[m], z0[k], n[k]));
    const bool got = results_overlap_inputs(count, S.data(), none ? nullptr : Z0.data(), n.data(),
                                            Z.data());
    CHECK(got == want, "case %d: %d matrices, got %d", t, count, (int)got);
    hits += want;
  }
  CHECK(hits > 2000 && hits < 18000, "%d of 20000 cases overlap", hits);
}

// above_power is err > pow(prev, pw), also one rounding away from equality, where the power
// multiplied out gives other answers
static void powers(std::mt19937& rng) {
  std::uniform_real_distribution<double> lg(-18.0, 3.0);
  int differ = 0;
  for (int t = 0; t < 20000; ++t) {
    const int pw = 2 + (int)(rng() % 5);
    const double prev = pow(10.0, lg(rng)), p = pow(prev, (double)pw);
    double prod = prev;
    for (int k = 1; k < pw; ++k) prod *= prev;
    const double near[] = {p, nextafter(p, 0.0), nextafter(p, INFINITY), prod, p * (1.0 + 1e-13),
                           p * (1.0 - 1e-13), p * 2.0, p * 0.5, prev, 0.0};
    for (double err : near) {
      CHECK(above_power(err, prev, pw) == (err > p), "err %.17g prev %.17g pw %d", err, prev, pw);
      differ += (err > prod) != (err > p);
    }
  }
  CHECK(differ > 100, "%d answers differ from the multiplied power's", differ);
  for (double prev : {0.0, 1.0, 1e-70, 1e-110, 1e-160, 1e-200, 1e90, 1e160})
    for (double err : {0.0, 5e-324, 1e-310, 1e-300, 1e-9, 1.0, 1e300})
      for (int pw = 2; pw <= 6; ++pw)
        CHECK(above_power(err, prev, pw) == (err > pow(prev, (double)pw)), "err %g prev %g pw %d",
              err, prev, pw);
}

// Every matrix has one team, whole, on one XCD, its members consecutive in that XCD's share of
// the grid; what is no member's slot is marked so, and no XCD's share ends in a row of them.
static void slots_of(std::mt19937& rng, int count, int max_np) {
  std::vector<int> np(count);
  for (int& v : np) v = 64 * (1 + (int)(rng() % (max_np / 64)));
  std::vector<TeamSlot> s;
  team_slots(np, s);
  CHECK(s.size() % 8 == 0 && !s.empty(), "%zu slots", s.size());
  std::vector<int> next(count, 0), size(count, 0), at(count, -1);
  for (int x = 0; x < 8; ++x)
    for (size_t b = x; b < s.size(); b += 8) {
      const TeamSlot& t = s[b];
      if (t.mat < 0) {
        for (size_t q = b; q < s.size(); q += 8) CHECK(s[q].mat < 0, "a gap in XCD %d's share", x);
        break;
      }
      CHECK(t.mat < count && t.size >= 1 && t.size <= 32 && t.size <= (np[t.mat] / 32) * (np[t.mat] / 32),
            "matrix %d size %d", t.mat, t.size);
      CHECK(t.rank == next[t.mat]++ && (at[t.mat] < 0 || at[t.mat] == (int)b - 8),
            "member %d of matrix %d at %zu", t.rank, t.mat, b);
      CHECK(t.rank == 0 || size[t.mat] == t.size, "matrix %d changes its size", t.mat);
      size[t.mat] = t.size;
      at[t.mat] = (int)b;
    }
  for (int m = 0; m < count; ++m) CHECK(next[m] == size[m] && size[m] > 0, "matrix %d has no team", m);
  size_t last = 0;
  for (size_t b = s.size() - 8; b < s.size(); ++b) last += s[b].mat >= 0;
  CHECK(last > 0, "an empty last row");
}

// Each XCD takes one contiguous run of tiles, in order, also where 8 does not divide the grid:
// the first nb % 8 XCDs one tile more, the runs one after the other.
static void runs_of(int nb) {
  int expect = 0;
  for (int x = 0; x < 8; ++x)
    for (int b = x; b < nb; b += 8)
      CHECK(xcd_remap(b, nb) == expect++, "xcd_remap(%d, %d) = %d", b, nb, xcd_remap(b, nb));
  CHECK(expect == nb, "%d of %d blocks", expect, nb);
}

// after a late team the given number of calls go by launches, then a team is tried again
static void rests() {
  for (int rest : {0, 1, 3, 32}) {
    TeamRest r;
    for (int k = 0; k < 5; ++k) CHECK(r.team(), "a rest without a late team");
    for (int again = 0; again < 2; ++again) {
      r.late(rest);
      for (int k = 0; k < rest; ++k) CHECK(!r.team(), "rest %d ended after %d calls", rest, k);
      for (int k = 0; k < 5; ++k) CHECK(r.team(), "rest %d goes on", rest);
    }
  }
}

int main() {
  rests();
  for (int nb = 1; nb <= 3000; ++nb) runs_of(nb);
  std::mt19937 rng(7);
  for (int count : {1, 2, 7, 8, 9, 48, 100, 513, 5000})
    for (int max_np : {64, 128, 256, 512}) slots_of(rng, count, max_np);
  powers(rng);
  overlaps(rng);
  printf("ok %ld\n", g_checks);
  return 0;
}
