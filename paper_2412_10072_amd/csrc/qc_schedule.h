// Limits that the host keeps when it chooses how a call runs.  Plain C++ without
// HIP, so that the same code also builds on its own in a CPU test.
#pragma once

#include <cstddef>

namespace qc {

// Memory of the context that a call can do without (tables, folded models): at most a
// sixteenth of the device's and, when it has to grow, an eighth of what is free (the
// arrays the caller may still want come first).
inline bool spare_fits(size_t bytes, size_t free_b, size_t total_b) {
  return bytes > 0 && bytes <= total_b / 16 && bytes <= free_b / 8;
}

}  // namespace qc
