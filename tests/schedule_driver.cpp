// Driver of the host's scheduling limits (csrc/qc_schedule.h) for
// test_host_schedule.py.  Exit status 0 when every case agrees.
#include <cstdio>

#include "../paper_2412_10072_amd/csrc/qc_schedule.h"

static int failures = 0;

#define EXPECT(cond)                                       \
  do {                                                     \
    if (!(cond)) {                                         \
      std::printf("FAIL line %d: %s\n", __LINE__, #cond);  \
      ++failures;                                          \
    }                                                      \
  } while (0)

static void spare_cases() {
  const size_t GiB = (size_t)1 << 30;
  EXPECT(qc::spare_fits(GiB, 200 * GiB, 288 * GiB));
  EXPECT(qc::spare_fits(18 * GiB, 144 * GiB, 288 * GiB));
  EXPECT(!qc::spare_fits(18 * GiB + 1, 288 * GiB, 288 * GiB));     // a sixteenth of the device's
  EXPECT(!qc::spare_fits(GiB, 8 * GiB - 1, 288 * GiB));            // an eighth of what is free
  EXPECT(!qc::spare_fits(1, 0, 288 * GiB));
  EXPECT(!qc::spare_fits(0, 288 * GiB, 288 * GiB));                // nothing to hold
}

int main() {
  spare_cases();
  std::printf("%d failures\n", failures);
  return failures == 0 ? 0 : 1;
}
