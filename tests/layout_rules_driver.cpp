// The rules that lay partitions out, at sizes no test loads. Built and run by
// tests/test_layout_rules.py; exits non-zero on a failed expectation.
#include <cstdio>

#include "gc_internal.h"

#define EXPECT(c) do { if (!(c)) { std::printf("FAIL line %d: %s\n", __LINE__, #c); ++fails; } } while (0)

using namespace gcx;

int main() {
  int fails = 0;
  const int64_t top = (int64_t(1) << 31) - 1;  // the most arcs are one fewer
  // the batched form reads ranges of 1024: a partition that it takes (no
  // stream layout, at most 1024 blocks) merges in those and no others
  for (int32_t W = 1 << 10; W <= 1 << 26; W *= 2)
    for (int64_t n = 1000; n < top; n = n * 3 / 2 + 1)
      for (int64_t m : {int64_t(0), n / 2, 16 * n, top - 2000, top - 1025, top - 1024, top - 1}) {
        const int64_t B = (n + W - 1) / W;
        if (m >= top || B > 1024 || pull_streams(static_cast<int32_t>(n), m, W, 1024)) continue;
        if (merge_width(static_cast<int32_t>(n), m, W, 1024) != 1024) {
          std::printf("FAIL n=%lld m=%lld W=%d\n", (long long)n, (long long)m, W);
          ++fails;
        }
      }
  // the stream layout ends at its width, at its range table and at its arcs
  EXPECT(pull_streams(1 << 20, 16 << 20, 1 << 15, 256) && !pull_streams(1 << 20, 16 << 20, 1 << 16, 256));
  EXPECT(pull_streams(100000, top - 1025, 1 << 15, 1024) && !pull_streams(100000, top - 1024, 1 << 15, 1024));
  EXPECT(!pull_streams(1 << 25, 1 << 26, 1 << 15, 1024) && pull_streams(1 << 24, 1 << 26, 1 << 15, 1024));
  // ranges are halved to a count, never below 256 or past the table's share of the arcs
  EXPECT(merge_width(300007, 3600000, 1 << 14, 4096) == 2048 && merge_width(300007, 3600000, 1 << 14, 256) == 256);
  EXPECT(merge_width(2500009, 37500000, 1 << 18, 4096) == 2048 && merge_width(1 << 24, 1 << 27, 1 << 18, 16384) == 2048);
  EXPECT(merge_width(1 << 28, 1000, 1 << 16, 16384) == 16384);
  std::printf("fails %d\n", fails);
  return fails != 0;
}
