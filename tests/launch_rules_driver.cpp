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

int main() {
  wide_merge();
  return failures != 0;
}
