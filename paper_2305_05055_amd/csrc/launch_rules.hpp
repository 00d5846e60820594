// Host rules that size or choose launches from what a handle knows about its set
// and its earlier batches.  Plain C++, also built without HIP.
#pragma once
#include <algorithm>
#include <cstdint>

namespace cpma_dev {

// Waves of the merge over the list of wide segments, for a batch that touches at
// most `segs` leaves, with at most `most` waves.  `share`: wide segments among the
// last classified batch's (1 before there is one); which leaves are wide is a
// property of the set's keys, so it holds from batch to batch.  A wave per expected
// segment, as in the narrow merge: the dispatcher then evens out their unequal work
// (an edge set's batches of 2e6 keys, insert and delete: 2050 us with 320 waves a
// CU, 2344 with 32, 2909 with 15), while an empty list costs 12 us more with 320
// waves than with 32 (40-bit keys, batches of 1e5: 372 and 347 us).
inline uint32_t wide_waves(uint64_t segs, double share, uint32_t cus, uint32_t most) {
  const uint64_t expected = (uint64_t)(share * (double)segs) + 1;
  return (uint32_t)std::min<uint64_t>(most, std::max<uint64_t>(32ull * cus, expected));
}

}  // namespace cpma_dev
