// Point lookups in leaves, four per wave at a time: how many keys of a leaf lie
// below x, their sum, and whether x is there (contains, get and the end leaves
// of range_map: Sections "Compressed Packed Memory Array", "Point queries", and
// "Packed Memory Array", "Design and operations").
//
// A row of 16 lanes decodes one leaf, 16 bytes per lane and 256 bytes per
// round, and stops after the round in which the keys reach x.  One lane per
// leaf, the obvious split, asks the L1 for 64 separate lines with every 16-byte
// load and walks its leaf in a chain of a dozen rounds, and a wave waits for the
// longest of its 64 walks.  1e6 membership tests on 1e8 keys: 389 -> 200 us; the
// partial end leaves of 1e6 ranges: 816 -> 423 us; get of 1e6 keys of a key-value
// set (byte loads before): 727 -> 151 us.  Walks that sum are bound by vector
// instructions (about 135 per round); membership in a large set by its random 256-byte
// reads (0.5 GB at 3.7 TB/s) and the head search (60 of the 200 us): a walk of a third
// fewer instructions changed nothing.  In leaves of fewer bytes than a round, large
// batches take a lane per lookup (lane_lookups).
#pragma once
#include "scan_lane.hpp"
#include "update.hpp"

namespace cpma_dev {

struct QueryArgs {
  const uint64_t* lo;
  const uint64_t* hi;
  uint64_t q;
  const uint64_t* head;
  const uint8_t* bytes;
  const uint32_t* used;
  uint64_t L;
  uint32_t S;
  uint32_t raw;  // uncompressed leaves (raw 8-byte keys)
  // key-value leaves: `used` above is each leaf's code bytes, `fill` its filled
  // bytes (codes and values); vals: sum values instead of keys
  const uint32_t* fill;
  uint32_t vals;
  uint32_t zero_fill;  // bytes past `used` are zero in place (every set without values)
};

// ---- DPP within rows of 16 lanes ---------------------------------------------------
template <typename T>
__device__ __forceinline__ T row_incl_scan(T v) {
  if constexpr (sizeof(T) == 4) {
    v += dpp32<0x111>(v);
    v += dpp32<0x112>(v);
    v += dpp32<0x114>(v);
    v += dpp32<0x118>(v);
  } else {
    v += dpp64<0x111>(v);
    v += dpp64<0x112>(v);
    v += dpp64<0x114>(v);
    v += dpp64<0x118>(v);
  }
  return v;
}
// Lane 15 of the row, to all its lanes.
__device__ __forceinline__ uint32_t row_last(uint32_t v) { return dpp32<0x15f>(v); }
__device__ __forceinline__ uint64_t row_last(uint64_t v) { return dpp64<0x15f>(v); }

// One lane's 16 bytes of a round, with what is not a code of the leaf turned
// into continuation bytes without payload: the first seven bytes of the head
// (its eighth becomes a terminator: one key at offset 0) and the bytes at or past
// `used` (zero fill, or values).
__device__ __forceinline__ uint4 lookup_bytes(uint4 q, uint32_t pos0, uint32_t used) {
  uint32_t w[4] = {q.x, q.y, q.z, q.w};
  if (pos0 == 0) {
    w[0] = 0x80808080u;
    w[1] = 0x00808080u;
  }
  const int32_t nv = (int32_t)used - (int32_t)pos0;
  if (nv < 16) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int32_t v = nv - 4 * k;
      const uint32_t keep = v >= 4 ? 0xffffffffu : (v <= 0 ? 0u : ((1u << (8 * v)) - 1u));
      w[k] = (w[k] & keep) | (0x80808080u & ~keep);
    }
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// The keys that end in 16 bytes, as offsets from what precedes them: f(offset,
// mask) per byte, mask all ones on a continuation byte, at which no key ends.
// sh: the shift the first byte's code has reached.  Returns the offset reached.
template <typename KT, class F>
__device__ __forceinline__ KT walk_bytes(const uint4 q, uint32_t sh, F&& f) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  KT run = 0;
#pragma unroll
  for (int j = 0; j < 16; j++) {
    const uint32_t x = w[j >> 2];
    uint32_t cm;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(cm) : "v"(x), "i"(8 * (j & 3) + 7));
    run += (KT)__builtin_amdgcn_ubfe(x, 8 * (j & 3), 7) << (sh & (8u * sizeof(KT) - 1u));
    sh = (sh + 7u) & cm;
    f(run, cm);
  }
  return run;
}

// Trailing continuation bytes of 16 bytes (KT 32 bits: at most 4 matter).
template <typename KT>
__device__ __forceinline__ uint32_t tail_run(const uint4 w) {
  const uint32_t e3 = ~w.w & 0x80808080u;
  uint32_t tc = e3 ? (uint32_t)__clz((int)e3) >> 3 : 4u;
  if constexpr (sizeof(KT) == 8) {
    const uint32_t e2 = ~w.z & 0x80808080u, e1 = ~w.y & 0x80808080u;
    if (!e3) tc += e2 ? (uint32_t)__clz((int)e2) >> 3 : 4u + (e1 ? (uint32_t)__clz((int)e1) >> 3 : 4u);
  }
  return tc;
}

// Where a lookup's walk reaches its key: the 16 bytes, the offset before them and
// the shift their first code has reached.
struct Reach {
  uint4 bytes;
  uint64_t at;
  uint32_t sh, pad;
};
constexpr uint32_t kReachBytes = sizeof(Reach) * kWave;  // LDS per wave

struct Lookup {
  uint64_t cnt;  // keys of the leaf below x
  uint64_t sum;  // their sum, or the sum of their values
  bool eq;       // x is a key of the leaf
  uint64_t cnt_from, sum_from;  // to the leaf's end: its other keys (then, with values, sum is not set)
};

// Four leaves' walks, one per row.  KT: the type of key offsets from the head, 32
// bits when every leaf's keys span less than 2^32 - 1 (so that X is below a
// continuation byte's all-ones mask).  The 16 bytes in which a row's offset
// reaches X go to `reach`; the lanes before them only need their totals (kSum: and
// the sum of their keys' offsets).  Returns the rows' lanes that reached X.
//
// kPair: a row may look for a second key X2 >= X in the same walk (dual), with its
// own slot, count, sum and lanes in `two`; or, with X2 above every offset, go on to
// the leaf's end, whose totals are then in `two`; X2 = X otherwise.
template <typename KT>
struct Second {
  KT X;
  bool dual;
  Reach* reach;
  uint32_t cnt;
  uint64_t sum, found;
};
template <typename KT, bool kSum, bool kPair>
__device__ __forceinline__ uint64_t row_walk(const uint8_t* __restrict__ leaf, uint4 w, uint32_t used, KT X,
                                             Reach* reach, uint32_t& cnt, uint64_t& sum, Second<KT>& two) {
  const uint32_t l16 = (uint32_t)lane_id() & 15u;
  KT base = 0;        // offset reached before the round (the row's lanes alike)
  uint32_t tail = 0;  // this lane's trailing continuation bytes in the round before
  uint64_t found = 0;
  for (uint32_t pos = 0;; pos += 256) {
    const uint32_t pos0 = pos + 16u * l16;
    w = lookup_bytes(w, pos0, used);
    // the run carried in: the lane before's; for the row's first lane the last
    // lane's of the round before (row rotation by one)
    const uint32_t tc = tail_run<KT>(w);
    const uint32_t wrap = dpp32<0x121>(tail), prev = dpp32<0x111>(tc);
    const uint32_t sh = 7u * (l16 ? prev : wrap);
    tail = tc;
    uint64_t s = 0;
    uint32_t s32 = 0;
    const KT run = walk_bytes<KT>(w, sh, [&](KT off, uint32_t cm) {
      if constexpr (kSum && sizeof(KT) == 8) {
        s += off & ~(KT)(int64_t)(int32_t)cm;
        // added as it comes: a tree over all sixteen offsets takes 60 registers, and the
        // narrow walk, in the same kernel, a wave of occupancy
        asm("" : "+v"(s));
      }
      if constexpr (kSum && sizeof(KT) == 4) s32 += (uint32_t)off & ~cm;
    });
    if constexpr (kSum && sizeof(KT) == 4) {
      // 16 offsets below 2^28 sum below 2^32; larger ones are added again in 64 bits
      s = s32;
      if (run >= (KT)(1u << 28)) {
        s = 0;
        walk_bytes<KT>(w, sh, [&](KT off, uint32_t cm) { s += (uint64_t)(off & ~(KT)(int64_t)(int32_t)cm); });
      }
    }
    const KT incl = row_incl_scan<KT>(run);
    const KT at = base + (incl - run), end = base + incl;
    base += row_last(incl);
    if constexpr (kSum) {
      if (end < (kPair ? two.X : X)) {
        const uint32_t c = 16u - (uint32_t)(__popc(w.x & 0x80808080u) + __popc(w.y & 0x80808080u) +
                                            __popc(w.z & 0x80808080u) + __popc(w.w & 0x80808080u));
        const uint64_t t = s + (uint64_t)c * (uint64_t)at;
        if (!kPair || end < X) {
          cnt += c;
          sum += t;
        }
        if constexpr (kPair) {
          two.cnt += c;
          two.sum += t;
        }
      }
    }
    const bool here = end >= X && (at < X || pos0 == 0);
    if (here) *reach = Reach{w, (uint64_t)at, sh, 0};
    found |= __ballot(here);
    if constexpr (kPair) {
      const bool here2 = two.dual && end >= two.X && (at < two.X || pos0 == 0);
      if (here2) *two.reach = Reach{w, (uint64_t)at, sh, 0};
      two.found |= __ballot(here2);
    }
    const bool more = pos + 256 < used && base < (kPair ? two.X : X);
    if (!__ballot(more)) return found;
    // a finished row goes on over bytes without keys
    w = make_uint4(0x80808080u, 0x80808080u, 0x80808080u, 0x80808080u);
    if (more && pos + 256 + 16u * l16 < used) w = load16(leaf + pos + 256 + 16u * l16);
  }
}

// Up to 64 lookups of one wave: lane l's lookup is key x in leaf `leaf` (valid:
// the lane has one; the lanes that do come first).  leaf must be the leaf x
// belongs to, or the one before when x is the next leaf's head.  kSum / kEq: what
// besides the count is wanted (kEq alone: not even the count, unless kCnt).
// Every lane then finishes its own lookup in the 16 bytes where it reached x: the
// per-key comparisons run once per 64 lookups instead of once per four.
//
// kPair: lanes 2i and 2i + 1 look up a range's two ends (x of the odd lane not below
// the even one's); pairs in one leaf share a walk, and `order` (64 entries of LDS per
// wave) lists the walks.  Many short ranges have both ends in one leaf: the end
// leaves of 1e6 Zipf(1.2) ranges take 423 us, 477 with a walk per end.  An even lane
// may also want what lies from x to the end of its leaf (to_end).
template <bool kCnt, bool kSum, bool kEq, bool kPair = false>
__device__ __forceinline__ Lookup wave_lookup(const QueryArgs& a, bool valid, uint64_t leaf, uint64_t x,
                                              Reach* reach, uint8_t* order = nullptr, bool to_end = false) {
  const uint32_t l = (uint32_t)lane_id(), l16 = l & 15u;
  const uint64_t head = valid ? a.head[leaf] : kNoKey;
  const uint64_t next = valid && leaf + 1 < a.L ? a.head[leaf + 1] : kNoKey;
  // x below the head (only below every key) and an empty leaf: nothing to read, but
  // to the leaf's end; nor for the reserved key, which no leaf holds (its offset can look like a
  // continuation byte's)
  const uint32_t used =
      valid && (x >= head || to_end) && head != kNoKey && !(kEq && x == kNoKey) ? a.used[leaf] : 0u;
  const uint64_t X = used && x >= head ? x - head : 0;
  const bool wide = used && next - head >= 0xffffffffull;
  const uint32_t nvalid = (uint32_t)__popcll(__ballot(valid));
  uint32_t nwalk = nvalid, slot = l;  // walks, and the one that answers this lane
  bool same = false, answered = true;
  if constexpr (kPair) {
    constexpr int kXor1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);
    const uint32_t other_used = dpp32<kXor1>(used);  // every lane takes part in the exchange
    const uint64_t other_leaf = dpp64<kXor1>(leaf);
    same = used && other_used && other_leaf == leaf;
    const bool own = used && !(same && (l & 1u));
    const uint64_t walks = __ballot(own);
    nwalk = (uint32_t)__popcll(walks);
    slot = __builtin_amdgcn_mbcnt_hi((uint32_t)(walks >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)walks, 0u));
    if (own) order[slot] = (uint8_t)l;
    const uint32_t other = dpp32<kXor1>(slot);
    if (same && (l & 1u)) slot = other;
    answered = used != 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }
  const uint32_t nit = (nwalk + 3u) / 4u;
  auto walk_lane = [&](uint32_t it) {
    const uint32_t w = 4u * it + (opaque_lane() >> 4);
    if constexpr (kPair)
      return w < nwalk ? (uint32_t)order[w] : 64u;
    else
      return w;
  };
  const bool any_wide = __ballot(wide) != 0;
  Lookup out{0, 0, false, 0, 0};
  bool reached = false;
  // the next lookups' first round is loaded before the current ones are decoded
  uint32_t n_used = 0, n_leaf = 0;
  bool n_wide = false;
  uint4 n_w = make_uint4(0, 0, 0, 0);
  auto fetch = [&](uint32_t it) {
    const uint32_t from = walk_lane(it);
    const uint32_t u = from_lane(used | (wide ? 1u << 31 : 0u), from);
    n_used = kPair && from == 64u ? 0u : u & ~(1u << 31);
    n_wide = (u >> 31) != 0;
    n_leaf = from_lane((uint32_t)leaf, from);
    if (16u * l16 < n_used) n_w = load16(a.bytes + (uint64_t)n_leaf * a.S + 16u * l16);
  };
  if (!a.raw) fetch(0);
#pragma unroll 1
  for (uint32_t it = 0; it < nit; it++) {
    const uint32_t from = walk_lane(it);
    const bool none = kPair && from == 64u;
    const uint64_t Xf = from_lane(X, from), Xr = none ? 1 : Xf;  // no key: a row without bytes never reaches 1
    bool dual = false;
    uint64_t X2 = Xr, sum2 = 0, found2 = 0;
    uint32_t cnt2 = 0;
    if constexpr (kPair) {
      const uint32_t want = from_lane(same ? 1u : (to_end ? 2u : 0u), from);  // every lane takes part
      const uint32_t d = none ? 0u : want;
      dual = d == 1u;
      const uint64_t o = from_lane(X, from | 1u);
      if (d) X2 = dual ? o : ~0ull;
    }
    uint64_t sum = 0, found = 0;
    uint32_t cnt = 0;
    bool eq = false;
    if (a.raw) {
      const uint32_t uf = from_lane(used, from), m = none ? 0u : uf / 8;
      const uint64_t hd = from_lane(head, from);
      const uint64_t* k = reinterpret_cast<const uint64_t*>(a.bytes + (uint64_t)from_lane((uint32_t)leaf, from) * a.S);
#pragma unroll 4
      for (uint32_t i = l16; i < m; i += 16) {
        const uint64_t d = k[i] - hd;
        cnt += d < Xr ? 1u : 0u;
        if constexpr (kSum) sum += d < Xr ? d : 0ull;
        if constexpr (kEq) eq |= d == Xr;
        if constexpr (kPair) {
          cnt2 += d < X2 ? 1u : 0u;
          sum2 += d < X2 ? d : 0ull;
        }
      }
    } else {
      const uint32_t ur = n_used;
      const uint8_t* lp = a.bytes + (uint64_t)n_leaf * a.S;
      const uint4 w = n_w;
      const bool walk_wide = __ballot(n_wide) != 0;  // one of these four
      if (it + 1 < nit) fetch(it + 1);
      auto walk = [&](auto zero) {
        using KT = decltype(zero);
        Second<KT> two{(KT)X2, dual, reach + (from | 1u), 0, 0, 0};
        found = row_walk<KT, kCnt || kSum, kPair>(lp, w, ur, (KT)Xr, reach + from, cnt, sum, two);
        cnt2 = two.cnt;
        sum2 = two.sum;
        found2 = two.found;
      };
      if (walk_wide)
        walk((uint64_t)0);
      else
        walk((uint32_t)0);
    }
    // to the lanes whose lookups these were
    const uint32_t ol = kPair ? slot : opaque_lane(), src = 16u * (ol & 3u);
    const bool mine = answered && (ol >> 2) == it, second = kPair && same && (l & 1u);
    if constexpr (kCnt || kSum) {
      uint32_t c = from_lane(row_last(row_incl_scan(cnt)), src);
      if constexpr (kPair) {
        const uint32_t c2 = from_lane(row_last(row_incl_scan(cnt2)), src);
        if (second) c = c2;
        if (mine && to_end) out.cnt_from = c2;
      }
      if (mine) out.cnt = c;
    }
    if constexpr (kSum) {
      uint64_t t = from_lane(row_last(row_incl_scan(sum)), src);
      if constexpr (kPair) {
        const uint64_t t2 = from_lane(row_last(row_incl_scan(sum2)), src);
        if (second) t = t2;
        if (mine && to_end) out.sum_from = t2;
      }
      if (mine) out.sum = t;
    }
    if (mine) reached = (((second ? found2 : found) >> src) & 0xffffu) != 0;
    if constexpr (kEq) {
      const uint64_t em = __ballot(eq);
      if (mine) out.eq = ((em >> src) & 0xffffu) != 0;
    }
  }
  if (!a.raw) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if (reached && used) {
      const Reach m = reach[l];
      auto finish = [&](auto zero) {
        using KT = decltype(zero);
        const KT lim = (KT)(X - m.at);
        uint64_t add = 0;
        uint32_t c = 0;
        bool hit = false;
        walk_bytes<KT>(m.bytes, m.sh, [&](KT off, uint32_t cm) {
          const KT k = off | (KT)(int64_t)(int32_t)cm;  // a continuation byte is no key: above every x
          if constexpr (kCnt || kSum) c += k < lim ? 1u : 0u;
          if constexpr (kSum) add += k < lim ? (uint64_t)k : 0ull;
          if constexpr (kEq) hit |= k == lim;
        });
        out.cnt += c;
        out.sum += add + (uint64_t)c * m.at;
        out.eq = hit;
      };
      if (any_wide)
        finish((uint64_t)0);
      else
        finish((uint32_t)0);
    }
    __builtin_amdgcn_wave_barrier();  // the slots may be written again
  }
  if constexpr (kPair) {  // from the leaf's totals
    if (to_end) {
      out.cnt_from -= out.cnt;
      out.sum_from = out.sum_from - out.sum + out.cnt_from * head;
    }
  }
  if constexpr (kSum) {
    if (!a.vals) {
      out.sum += out.cnt * head;
    } else {
      // the values of the keys below x: the first of the leaf's m values; to the
      // leaf's end: the others
      const uint32_t m = used ? (a.fill[leaf] - used) / 8 : 0u;
#pragma unroll 1
      for (uint32_t it = 0; it < (nvalid + 3u) / 4u; it++) {
        const uint32_t from = 4u * it + (opaque_lane() >> 4);
        const uint32_t v0 = from_lane(to_end ? (uint32_t)out.cnt : 0u, from);
        const uint32_t v1 = from_lane(to_end ? m : (uint32_t)out.cnt, from);
        const uint64_t* v = reinterpret_cast<const uint64_t*>(
            a.bytes + (uint64_t)from_lane((uint32_t)leaf, from) * a.S + a.S - 8u * from_lane(m, from));
        uint64_t s = 0;
        for (uint32_t i = v0 + l16; i < v1; i += 16) s += v[i];
        const uint32_t ol = opaque_lane();
        const uint64_t t = from_lane(row_last(row_incl_scan(s)), 16u * (ol & 3u));
        if ((ol >> 2) == it) (to_end ? out.sum_from : out.sum) = t;
      }
    }
  }
  return out;
}

// Leaf of x for each row of 16 lanes (x alike in a row): a 16-ary search of the
// heads, five dependent loads for a million leaves instead of twenty.
__device__ __forceinline__ uint64_t row_locate_leaf(const uint64_t* __restrict__ head, uint64_t L, uint64_t x,
                                                    bool active) {
  uint64_t lo = 0, hi = active ? L : 0;  // the first head above x lies in [lo, hi]
  const uint32_t l16 = (uint32_t)lane_id() & 15u, row = (uint32_t)lane_id() & 48u;
  while (__ballot(lo < hi)) {
    const uint64_t step = (hi - lo + 15) / 16;
    const uint64_t idx = lo + l16 * step;
    const bool le = lo < hi && idx < hi && head[idx] <= x;
    const uint32_t t = (uint32_t)__popc((uint32_t)(__ballot(le) >> row) & 0xffffu);  // a prefix of the pivots
    if (lo < hi) {
      if (t == 0) {
        hi = lo;
      } else {
        const uint64_t last = lo + (uint64_t)(t - 1) * step;
        lo = last + 1;
        hi = min(hi, last + step);
      }
    }
  }
  return lo ? lo - 1 : 0;
}

// The leaf of every lane's x (valid lanes first).  Up to four keys: a 16-ary
// search by a row each, whose chain of loads is a quarter as long; more: a
// binary search per lane, which asks for far fewer lines in all.
__device__ __forceinline__ uint64_t wave_locate(const QueryArgs& a, bool valid, uint64_t x) {
  if (__popcll(__ballot(valid)) <= 4) {
    const uint32_t row = opaque_lane() >> 4;
    const bool act = from_lane(valid ? 1u : 0u, row) != 0;
    const uint64_t f = row_locate_leaf(a.head, a.L, from_lane(x, row), act);
    return from_lane(f, 16u * (opaque_lane() & 3u));
  }
  return valid ? locate_leaf(a.head, a.L, x) : 0;
}

}  // namespace cpma_dev
