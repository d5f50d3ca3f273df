// Host-only check of the batched path's host arithmetic (zf_index.h), built and run by
// tests/test_host_batch.py under AddressSanitizer and UBSan.  Prints "ok <checks>" or the
// first failure and exits non-zero.
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

#include "zf_index.h"

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

int main() {
  std::mt19937 rng(7);
  overlaps(rng);
  printf("ok %ld\n", g_checks);
  return 0;
}
