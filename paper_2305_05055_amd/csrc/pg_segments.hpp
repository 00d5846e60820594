// The gather segments of PageRank's binned edges: a part's edges [b0, b1) cut into
// runs of at most `seg`.  Edge positions fill 32 bits (a set of up to 2^32 - 1025
// edges is binned), so no sum here may pass b1.  Plain C++, also built without HIP.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define CPMA_HD __host__ __device__ inline
#else
#define CPMA_HD inline
#endif

namespace cpma_dev {

CPMA_HD uint32_t pg_segment_count(uint32_t b0, uint32_t b1, uint32_t seg) {
  const uint32_t n = b1 - b0;
  return n / seg + (n % seg ? 1u : 0u);
}

// Segment i, below pg_segment_count.
struct PgSegment {
  uint32_t e0, e1;
};
CPMA_HD PgSegment pg_segment(uint32_t b0, uint32_t b1, uint32_t seg, uint32_t i) {
  const uint32_t e0 = b0 + i * seg, left = b1 - e0;
  return PgSegment{e0, e0 + (left < seg ? left : seg)};
}

}  // namespace cpma_dev
