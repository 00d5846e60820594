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

// Whether an unsorted batch of the small split's size tries it.  The split counts its
// buckets with the last such batch's bit length, while validating, and a count that
// does not hold is lost (about 15 us; split 34 us at 1e5 keys, radix passes 58).  A
// batch whose own bit length was the guess and whose buckets overflow is skewed, and
// the next 16 do not try.  One of another bit length says nothing about the next:
// that one tries with the new length, and only lost counts in a row (lengths that
// alternate) make the pauses between tries longer, up to the same 16.
struct SplitGuess {
  int bits = 0;  // of the last such batch (0: none yet)
  int skip = 0;  // batches that do not try
  int pause = 0;

  bool tries() const { return bits > 0 && skip == 0; }
  // A batch of `b` bits; tried: its buckets were counted; split: the counts held.
  void took(int b, bool tried, bool split) {
    if (!tried) {
      if (skip) skip--;
    } else if (split) {
      pause = 0;
    } else if (b == bits) {
      skip = 16;
    } else {
      skip = pause;
      pause = std::min(16, 2 * pause + 1);
    }
    bits = b;
  }
};

// Whether the lookup of a range's lower end goes on to the end of its leaf when the
// range ends in the next one, so that the leaf needs no visit of its own.  A batch of
// few queries waits for its longest chain, and a visit of one leaf is a chain of its
// own; many queries are bound by the lookups' instructions, and the visits of
// different queries share the chip better than longer walks.  Ranges of 3 keys in 5e6:
// 1000 queries 20 us to the end and 23 with the visits, 8000 21 and 34; of 300 keys:
// 30 000 56 and 52, 1e6 629 and 556.  Uncompressed leaves are read whole by the lookup
// anyway (1e6 ranges of 3 keys: 186 and 206).
inline bool ends_to_leaf_end(uint64_t q, bool raw) { return raw || q <= 8192; }

// Whether a batch of q ranges on a set of L leaves takes the memory of the leaf prefix
// sums (12 bytes a leaf) when the handle does not have it yet.  It needs them if it
// visits more leaves than there are, which the host cannot know; at most q L.  The
// memory costs 45 us, once per handle.  32 queries and more take it; fewer when the
// scans they may save, q - 1 of the whole set at about 0.24 ns a leaf, reach a
// millisecond (25 scans of 1e6 leaves: 6 ms leaf by leaf).
inline bool takes_prefix(uint64_t q, uint64_t L) { return q >= 32 || (q > 1 && L >= (1ull << 22) / (q - 1)); }

// Whether q lookups in leaves of S bytes take a lane each instead of a row of 16 lanes
// that walks 256 bytes a round.  Below that size a row's lanes lack bytes, and a lane
// per lookup does less work in all; its chain of bytes is longer, so there must be
// enough lookups to hide it.  Row and lane: ranges of 3 keys, 1e6 of them in 5e6 keys,
// at 64 bytes a leaf 271 and 155 us, at 256 231 and 173; 60 000 ranges of 100 keys in 1e6 at 64, 128
// and 256 bytes 51 and 44, 48 and 52, 48 and 72; 1e6 of them at 512 385 and 438.
// Membership of 1e6 keys among 5e6 at 64 bytes 118 and 78, of 16 000 and 30 000 in 1e6
// 10 and 10, 12 and 11, of 60 000 and 250 000 at 128 bytes 13 and 16, 37 and 30, of 1e6
// at 256 101 and 107.
inline bool lane_lookups(uint32_t S, uint64_t q, bool ranges) {
  return ranges ? S <= 256 && q >= 384ull * S : S <= 128 && q >= 6ull * S * S;
}

// PageRank's binned form (pagerank.hpp): parts of 2^kPgPartBits destinations, bins of at
// most 2^kPgBinBits sources, `cuts` of them at the leaves' limits.
constexpr uint32_t kPgPartBits = 15, kPgBinBits = 13;
inline uint32_t pg_parts(uint32_t nv) { return (uint32_t)(((uint64_t)nv + (1u << kPgPartBits) - 1) >> kPgPartBits); }
inline uint32_t pg_bins(uint32_t nv, uint32_t cuts) {
  return cuts + (uint32_t)(((uint64_t)nv + (1u << kPgBinBits) - 1) >> kPgBinBits);
}
// 2048 cuts with at least 16 edges to a (part, bin) run, 1024 with at least 8, else none.
inline uint32_t pg_cuts(uint64_t n, uint32_t nv) {
  if (n >= 16ull * pg_parts(nv) * pg_bins(nv, 2048)) return 2048;
  return n >= 8ull * pg_parts(nv) * pg_bins(nv, 1024) ? 1024 : 0;
}
// Whether the binned form applies: runs long enough, vertices and edge positions
// within what its tables hold.
inline bool pg_fits(uint64_t n, uint32_t nv) {
  return n < (1ull << 32) - 1024 && nv <= (1u << 25) && pg_cuts(n, nv) != 0;
}
// Whether it pays: binning costs about 50 us more than the pull's setup, and up to 1e6
// vertices, whose contributions the L2s hold, an iteration gains little.  Pull and
// bins, one iteration and ten: 2^16 vertices and 2e6 edges 60 and 134 us, 284 and 400;
// 2^18 and 8e6 155 and 222, 863 and 887; 2^20 and 2e6 100 and 143, 578 and 538; 2^20 and
// 3.3e7 603 and 529; 2^22 and 2e6 170 and 156.
inline bool bins_pay(uint64_t n, uint32_t nv, uint32_t iters) {
  return iters && (unsigned __int128)iters * (n + nv / 2) * nv >= (1ull << 43);
}

}  // namespace cpma_dev
