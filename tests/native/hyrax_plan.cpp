// The plan of a commitment for every kind of split and workspace: a slice's
// columns go to enough lanes that none adds many more columns than a lane of
// the full plan, or to all 64 lanes of a wave, and its sums fit the workspace.
#include "hyrax.cpp"

#include <cstdio>

using namespace vl;

static int bad = 0;

static void check(uint32_t R, uint32_t m, uint32_t split, uint64_t room) {
  const Split full = plan_split(R, m, 0), s = plan_split(R, m, split, room);
  const uint32_t len = std::min(s.chunk, m);
  const uint64_t per = (len + s.lanes - 1) / s.lanes, most = std::max<uint64_t>(4ull * full.chunk, (len + 63) / 64);
  const bool lanes = s.lanes == 1 || (s.lanes >= 4 && s.lanes <= 64 && (s.lanes & (s.lanes - 1)) == 0);
  const bool cover = (uint64_t)s.n_split * s.chunk >= m && (uint64_t)(s.n_split - 1) * s.chunk < m;
  // a given split's runs may be left out of the workspace, its slices not
  const bool fits = R * (uint64_t)s.n_split * kPartialBytes <= room && (split || partial_bytes(R, s) <= room);
  if (per > most || !lanes || !cover || !fits || (!split && room >= partial_bytes(R, full) && s.lanes != 1)) {
    printf("R %u m %u split %u room %llu: %u slices of %u columns on %u lanes\n", R, m, split, (unsigned long long)room,
           s.n_split, s.chunk, s.lanes);
    ++bad;
  }
}

int main() {
  const uint32_t dims[] = {1, 2, 3, 5, 8, 16, 63, 64, 65, 100, 129, 257, 437, 1000, 1024, 1873, 3000, 4096, 4097, 11008, 131072, 200000};
  for (uint32_t R : dims)
    for (uint32_t m : dims) {
      const uint64_t all = vl_hyrax_commit_workspace_size(R, m, 0), least = least_bytes(R, m, 0);
      check(R, m, 0, UINT64_MAX);
      check(R, m, 0, all);
      for (int k = 0; k <= 8; ++k) check(R, m, 0, std::max(least, all / 8 * k));
      const uint32_t top = (m + 63) / 64;
      for (uint32_t split : {1u, 2u, 3u, 5u, 16u, 20u, 31u, top / 2, top - 1, top})
        if (split >= 1 && split <= top) {
          check(R, m, split, least_bytes(R, m, split));
          check(R, m, split, vl_hyrax_commit_workspace_size(R, m, split));
        }
    }
  return bad != 0;
}
