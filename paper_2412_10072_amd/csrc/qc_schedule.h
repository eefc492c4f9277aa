// Limits that the host keeps when it chooses how a call runs.  Plain C++ without
// HIP, so that the same code also builds on its own in a CPU test.
#pragma once

#include <algorithm>
#include <cstddef>

namespace qc {

// Memory of the context that a call can do without (tables, folded models): at most a
// sixteenth of the device's and, when it has to grow, an eighth of what is free (the
// arrays the caller may still want come first).
inline bool spare_fits(size_t bytes, size_t free_b, size_t total_b) {
  return bytes > 0 && bytes <= total_b / 16 && bytes <= free_b / 8;
}

// Parts per interval whose partial sums (`values` doubles each, of n_int intervals) stay
// within SPLIT_SUMS_BYTES and, beyond the `held` bytes that the context has for them, within
// half of what is free (the rest of the schedule's state is smaller): as many of
// `parts` as fit, 1 (not split: the fused schedule needs none of it) if not even two do.
constexpr double SPLIT_SUMS_BYTES = 2147483648.0;
inline int split_parts_within(int parts, int n_int, size_t values, size_t held, size_t free_b) {
  const double one = (double)n_int * (double)values * sizeof(double);
  const double most = std::min(SPLIT_SUMS_BYTES, std::max((double)held, 0.5 * (double)free_b));
  const int fit = (int)std::min(most / std::max(one, 1.0), (double)parts);
  return fit >= 2 ? fit : 1;
}

}  // namespace qc
