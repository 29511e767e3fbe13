// Ensemble launches against the dispatch limit (host only).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace cube {

constexpr int kCountThreads = 1024;  // threads of a count-pass workgroup (one per tile)

// a dispatch holds fewer than 2^32 work-items
inline bool fits_dispatch(uint64_t blocks, uint64_t threads) { return blocks * threads < (1ull << 32); }

// Runs of consecutive boxes, per_box workgroups each, that one launch of workgroups of `threads` threads
// holds: entry i is the first box of run i, the last entry the number of boxes. A box that alone is too
// large is a run of its own (the launch then refuses it).
inline std::vector<size_t> box_runs(const std::vector<uint32_t>& per_box, uint64_t threads) {
  std::vector<size_t> first(1, 0);
  uint64_t blocks = 0;
  for (size_t b = 0; b < per_box.size(); ++b) {
    if (b > first.back() && !fits_dispatch(blocks + per_box[b], threads)) {
      first.push_back(b);
      blocks = 0;
    }
    blocks += per_box[b];
  }
  first.push_back(per_box.size());
  return first;
}

}  // namespace cube
