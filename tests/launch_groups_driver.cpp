// Test-only C wrapper around the host rule that cuts an ensemble's launches (csrc/launch_groups.h).
#include "../paper_1712_06121_amd/csrc/launch_groups.h"

extern "C" int count_threads() { return cube::kCountThreads; }

// the runs' first boxes into first (room for nbox + 1 entries); returns the number of runs
extern "C" int runs(const uint32_t* per_box, int nbox, int threads, int64_t* first) {
  const std::vector<size_t> r = cube::box_runs(std::vector<uint32_t>(per_box, per_box + nbox), (uint64_t)threads);
  for (size_t i = 0; i < r.size(); ++i) first[i] = (int64_t)r[i];
  return (int)r.size() - 1;
}
