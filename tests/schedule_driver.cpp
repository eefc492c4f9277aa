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

static void parts_cases() {
  const size_t GiB = (size_t)1 << 30, much = 200 * GiB;
  // 64 antennas, one gain direction, 6 values a block: nothing to cut
  EXPECT(qc::split_parts_within(512, 1, 64 * 6 + 1, 0, much) == 512);
  // 256 antennas, four gain directions, full blocks: fewer parts, not none
  const size_t wide = 256 * 4 * 24 + 1;
  const int p = qc::split_parts_within(16384, 1, wide, 0, much);
  EXPECT(p > 10000 && (double)p * wide * 8 <= qc::SPLIT_SUMS_BYTES && (double)(p + 1) * wide * 8 > qc::SPLIT_SUMS_BYTES);
  EXPECT(qc::split_parts_within(12, 1000, wide, 0, much) == 10);
  EXPECT(qc::split_parts_within(2, 100000, wide, 0, much) == 1);      // not even two parts fit
  EXPECT(qc::split_parts_within(1, 1, wide, 0, much) == 1);
  // half of what is free, unless the context holds more: fewer parts, then the
  // fused schedule instead of an allocation that fails
  EXPECT(qc::split_parts_within(1024, 4, 1000, 0, 64000000) == 1000);
  EXPECT(qc::split_parts_within(1024, 4, 1000, 0, 1000000) == 15);
  EXPECT(qc::split_parts_within(1024, 4, 1000, 0, 100000) == 1);
  EXPECT(qc::split_parts_within(1024, 4, 1000, 0, 0) == 1);
  EXPECT(qc::split_parts_within(1024, 4, 1000, 1024 * 32000, 0) == 1024);
}

int main() {
  spare_cases();
  parts_cases();
  std::printf("%d failures\n", failures);
  return failures == 0 ? 0 : 1;
}
