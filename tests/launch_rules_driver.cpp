// Launch rules of the update and query paths, on the host.
#include <cstdio>

#include "launch_rules.hpp"

static int failures = 0;
#define EXPECT(x) \
  do { \
    if (!(x)) { \
      std::printf("line %d: %s\n", __LINE__, #x); \
      failures++; \
    } \
  } while (0)

using namespace cpma_dev;

static void wide_merge() {
  const uint32_t cus = 256, most = cus * 320;
  // a set of wide leaves: as many waves as the narrow merge has
  EXPECT(wide_waves(10'000'000, 1.0, cus, most) == most);
  EXPECT(wide_waves(50'000, 1.0, cus, 50'000) == 50'000);
  EXPECT(wide_waves(400'000, 0.5, cus, most) == most);
  // none, or the last leaf's slice only
  EXPECT(wide_waves(400'000, 0.0, cus, most) == 32 * cus);
  EXPECT(wide_waves(400'000, 1.0 / 400'000, cus, most) == 32 * cus);
  // never more than `most`, never none
  EXPECT(wide_waves(1, 1.0, cus, 1) == 1);
  EXPECT(wide_waves(100, 0.0, cus, 100) == 100);
}

// Batches of the given bit lengths, repeated: how many of the last 68 tried the split
// and how many were split.  Buckets counted for more bits than a batch has overflow.
static void run(const int* bits, int n, bool skewed, int* tried, int* split) {
  SplitGuess g;
  *tried = *split = 0;
  for (int i = 0; i < 200; i++) {
    const int b = bits[i % n];
    const bool t = g.tries(), ok = t && !skewed && b == g.bits;
    g.took(b, t, ok);
    if (i >= 132) {
      *tried += t;
      *split += ok;
    }
  }
}

static void small_split() {
  int t, s;
  const int same[] = {40}, alternating[] = {40, 34};
  run(same, 1, false, &t, &s);
  EXPECT(t == 68 && s == 68);
  run(same, 1, true, &t, &s);
  EXPECT(t == 4);  // a skewed stream: one try in 17
  run(alternating, 2, false, &t, &s);
  EXPECT(t <= 4);  // every count would be lost
  // a single change of length, shorter or longer, costs one count and no pause
  for (int b : {38, 42}) {
    SplitGuess g;
    g.took(40, false, false);
    EXPECT(g.tries());
    g.took(40, true, true);
    g.took(b, true, false);
    EXPECT(g.tries() && g.bits == b);
    g.took(b, true, true);
    EXPECT(g.tries());
  }
}

static void prefix_memory() {
  EXPECT(!takes_prefix(1, 1ull << 40));
  EXPECT(takes_prefix(32, 1) && !takes_prefix(31, 1000));
  EXPECT(takes_prefix(25, 1'000'000));  // few scans of a large set
  EXPECT(!takes_prefix(10, 400'000) && takes_prefix(2, 1ull << 22) && !takes_prefix(2, (1ull << 22) - 1));
}

static void lookups() {
  EXPECT(lane_lookups(64, 24576, true) && !lane_lookups(64, 24575, true) && !lane_lookups(512, 1 << 30, true));
  EXPECT(lane_lookups(256, 98304, true) && !lane_lookups(256, 1 << 30, false));
  EXPECT(lane_lookups(128, 98304, false) && !lane_lookups(128, 98303, false) && lane_lookups(64, 24576, false));
  EXPECT(ends_to_leaf_end(8192, false) && !ends_to_leaf_end(8193, false) && ends_to_leaf_end(1 << 20, true));
}

static void pagerank() {
  const uint64_t M = 1'000'000;
  EXPECT(!bins_pay(2 * M, 1u << 16, 10) && !bins_pay(8 * M, 1u << 18, 1) && bins_pay(8 * M, 1u << 18, 10));
  EXPECT(!bins_pay(2 * M, 1u << 20, 1) && bins_pay(2 * M, 1u << 20, 10) && bins_pay(33 * M, 1u << 20, 1));
  EXPECT(bins_pay(2 * M, 1u << 22, 1) && !bins_pay(1000 * M, 1u << 24, 0));
  EXPECT(pg_fits(2 * M, 1u << 20) && !pg_fits(2 * M, 1u << 24) && pg_fits(266 * M, 1u << 24));
  EXPECT(pg_fits((1ull << 32) - 1025, 1u << 25) && !pg_fits((1ull << 32) - 1024, 1u << 25));
  EXPECT(!pg_fits(1ull << 31, (1u << 25) + 1) && !pg_fits(10, 1));
}

int main() {
  wide_merge();
  pagerank();
  lookups();
  prefix_memory();
  small_split();
  return failures != 0;
}
