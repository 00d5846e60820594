// Segments of PageRank's binned edges against 64-bit arithmetic: every part's
// segments cover it in order, none longer than `seg`, also where edge positions
// come close to 2^32.
#include <cinttypes>
#include <cstdio>

#include "pg_segments.hpp"

static int check(uint64_t b0, uint64_t b1, uint64_t seg) {
  using namespace cpma_dev;
  const uint64_t n = (b1 - b0 + seg - 1) / seg;
  uint64_t at = b0;
  if (pg_segment_count((uint32_t)b0, (uint32_t)b1, (uint32_t)seg) != n) return 1;
  for (uint64_t i = 0; i < n; i++) {
    const PgSegment s = pg_segment((uint32_t)b0, (uint32_t)b1, (uint32_t)seg, (uint32_t)i);
    const uint64_t want = at + seg < b1 ? at + seg : b1;
    if (s.e0 != at || s.e1 != want) return 1;
    at = want;
  }
  return at != b1;
}

int main() {
  const uint64_t top = (1ull << 32) - 1025;  // the most edges that are binned
  const uint64_t segs[] = {1u << 13, (1u << 13) + 4, 1u << 17};
  const uint64_t sizes[] = {0, 1, 3, 4, 5, (1u << 13) - 1, 1u << 13, (1u << 13) + 1, (1u << 17) - 1, 1u << 17,
                            (1u << 17) + 1, 3u << 17, (1u << 27) + 7, top / 2, top};
  const uint64_t ends[] = {top, top - 1, top - 1023, top - (1u << 17), top - (1u << 17) + 1, 1ull << 31, 12345678};
  int bad = 0;
  for (uint64_t seg : segs)
    for (uint64_t end : ends)
      for (uint64_t n : sizes)
        if (n <= end && check(end - n, end, seg)) {
          std::printf("part [%" PRIu64 ", %" PRIu64 ") in segments of %" PRIu64 "\n", end - n, end, seg);
          bad = 1;
        }
  return bad;
}
