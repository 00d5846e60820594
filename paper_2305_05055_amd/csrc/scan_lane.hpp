// Per-lane pieces of the leaf decoders.
//
// A range query is a search followed by a scan (Section "Packed Memory Array",
// "Design and operations").  Leaves strictly inside a query's leaf span hold only
// keys of the range, so they need a sum and a count but no comparisons: zf_chunk
// decodes a lane's share of one, 16 bytes at a time.  leaf_sum_range walks a whole
// leaf in one lane and compares every key, for the ends of ranges and membership in
// small leaves; leaf_sum_fast sums one without comparisons and gives its last key,
// for the resize.
#pragma once
#include "common.hpp"

namespace cpma_dev {

struct LeafSum {
  uint64_t sum;    // wrapping sum of keys
  uint64_t count;  // number of keys
};

__device__ __forceinline__ uint4 load16(const uint8_t* p) { return *reinterpret_cast<const uint4*>(p); }

// Interior fast path: sum and count of every key of a leaf whose key span is
// below 2^28 (so every delta code is at most 4 bytes and fits 32-bit shifts).
//
// Per byte: p = payload bits, the running chunk-relative delta Dc grows by
// p << sh; at a terminator byte Dc equals (key - key at chunk start), so the
// chunk's keys sum to cnt * base + sum of Dc at terminators.  The byte loop has
// no validity tests: bytes at or past `used` are rewritten to 0x80, continuation
// bytes without payload (one masked merge per word, in the last chunk only); the head's eight
// bytes become seven such bytes and a zero terminator, so the head counts as a
// key at offset 0 from the chunk base (the head itself).  The terminator count
// is one popcount per word.  The leaf streams in 64-byte rounds with the next
// round's four loads in flight.
__device__ __forceinline__ void fast_chunk(const uint4 q, uint32_t c, uint32_t used, uint64_t& base, uint32_t& sh,
                                           LeafSum& r) {
  uint32_t w[4] = {q.x, q.y, q.z, q.w};
  if (c == 0) {
    w[0] = 0x80808080u;
    w[1] = 0x00808080u;
  }
  const int32_t nv = (int32_t)used - (int32_t)c;
  if (nv < 16) {
    // bytes at or past `used` (zero fill in place; arbitrary in an overflow
    // copy) become exactly 0x80
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int32_t v = nv - 4 * k;
      const uint32_t keep = v >= 4 ? 0xffffffffu : (v <= 0 ? 0u : ((1u << (8 * v)) - 1u));
      w[k] = (w[k] & keep) | (0x80808080u & ~keep);
    }
  }
  const uint32_t cnt = (uint32_t)(__popc(~w[0] & 0x80808080u) + __popc(~w[1] & 0x80808080u) +
                                  __popc(~w[2] & 0x80808080u) + __popc(~w[3] & 0x80808080u));
  uint32_t Dc = 0, Sc = 0;
#pragma unroll
  for (int i = 0; i < 16; i++) {
    const uint32_t x = w[i >> 2];
    const int o = 8 * (i & 3);
    const uint32_t p = (x >> o) & 0x7fu;
    const uint32_t cm = 0u - ((x >> (o + 7)) & 1u);  // all ones on a continuation byte
    Dc += p << (sh & 31u);
    Sc += Dc & ~cm;
    sh = (sh + 7u) & cm;
  }
  r.sum += (uint64_t)cnt * base + Sc;
  r.count += cnt;
  base += Dc;
}

// Also returns the leaf's last key through *last.
__device__ __forceinline__ LeafSum leaf_sum_fast(const uint8_t* __restrict__ leaf, uint32_t used,
                                                 uint64_t head, uint64_t* last = nullptr) {
  LeafSum r{0, 0};
  uint64_t base = head;  // key value reached by the running delta so far
  uint32_t sh = 0;
  const uint4 z = make_uint4(0, 0, 0, 0);
  uint4 a0 = load16(leaf);
  uint4 a1 = 16 < used ? load16(leaf + 16) : z;
  uint4 a2 = 32 < used ? load16(leaf + 32) : z;
  uint4 a3 = 48 < used ? load16(leaf + 48) : z;
  for (uint32_t c = 0; c < used; c += 64) {
    uint4 b0 = z, b1 = z, b2 = z, b3 = z;
    if (c + 64 < used) b0 = load16(leaf + c + 64);
    if (c + 80 < used) b1 = load16(leaf + c + 80);
    if (c + 96 < used) b2 = load16(leaf + c + 96);
    if (c + 112 < used) b3 = load16(leaf + c + 112);
    fast_chunk(a0, c, used, base, sh, r);
    fast_chunk(a1, c + 16, used, base, sh, r);
    fast_chunk(a2, c + 32, used, base, sh, r);
    fast_chunk(a3, c + 48, used, base, sh, r);
    a0 = b0;
    a1 = b1;
    a2 = b2;
    a3 = b3;
  }
  if (last) *last = base;
  return r;
}

// One byte (byte J of word x) of wave_leaf_sums: the running offset D grows by
// the byte's payload at its shift; a terminator's D is returned for the sum, a
// continuation byte returns 0.  The continuation mask is one sign-extending
// extract, written so that the compiler keeps it: left to itself it rebuilds
// the mask from a compare and two selects per byte.
template <int J>
__device__ __forceinline__ uint32_t zf_byte(uint32_t x, uint32_t& D, uint32_t& sh) {
  uint32_t cm;  // all ones on a continuation byte
  asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(cm) : "v"(x), "i"(8 * J + 7));
  D += __builtin_amdgcn_ubfe(x, 8 * J, 7) << (sh & 31u);
  sh = (sh + 7u) & cm;
  return D & ~cm;
}

// The same with 64-bit offsets.
template <int J>
__device__ __forceinline__ uint64_t zf_byte(uint32_t x, uint64_t& D, uint32_t& sh) {
  uint32_t cm;
  asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(cm) : "v"(x), "i"(8 * J + 7));
  D += (uint64_t)__builtin_amdgcn_ubfe(x, 8 * J, 7) << (sh & 63u);
  sh = (sh + 7u) & cm;
  return D & ~(uint64_t)(int64_t)(int32_t)cm;
}

// One 16-byte chunk of wave_leaf_sums.  `cont` counts continuation bytes.
// kSum64: every terminator's offset is added in 64 bits; otherwise offsets stay
// below 2^28, the chunk's 16 sum below 2^32 and are folded into the 64-bit total
// once.  KT: 32-bit offsets (up to 2^32) or 64-bit ones.
template <bool kSum64, typename KT>
__device__ __forceinline__ void zf_chunk(const uint4 q, KT& D, uint32_t& sh, uint64_t& Sc, uint32_t& cont) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < 4; j++) {
    const uint32_t x = w[j];
    const KT t0 = zf_byte<0>(x, D, sh);
    const KT t1 = zf_byte<1>(x, D, sh);
    const KT t2 = zf_byte<2>(x, D, sh);
    const KT t3 = zf_byte<3>(x, D, sh);
    if constexpr (kSum64) {
      Sc += ((uint64_t)t0 + t1) + ((uint64_t)t2 + t3);
      __builtin_amdgcn_sched_barrier(0);  // few registers: occupancy hides the loads
    } else {
      s += (uint32_t)((t0 + t1) + (t2 + t3));
    }
    cont += (uint32_t)__popc(x & 0x80808080u);
  }
  if constexpr (!kSum64) Sc += s;
}

// General path: 64-bit decode; counts and sums keys in [lo, hi).  Stops early
// once a key reaches hi.
__device__ __forceinline__ LeafSum leaf_sum_range(const uint8_t* __restrict__ leaf, uint32_t used,
                                                  uint64_t lo, uint64_t hi) {
  LeafSum r{0, 0};
  if (used < 8) return r;
  // 64-byte rounds with the next round's four loads in flight (a lane walks
  // its leaf alone, so every load would otherwise be a full round trip)
  const uint4 z = make_uint4(0, 0, 0, 0);
  uint4 a0 = load16(leaf);
  uint4 a1 = 16 < used ? load16(leaf + 16) : z;
  uint4 a2 = 32 < used ? load16(leaf + 32) : z;
  uint4 a3 = 48 < used ? load16(leaf + 48) : z;
  uint64_t key = ((uint64_t)a0.y << 32) | a0.x;
  if (key >= hi) return r;
  if (key >= lo) {
    r.sum += key;
    r.count++;
  }
  uint64_t acc = 0;
  uint32_t sh = 0;
  bool done = false;
  auto chunk = [&](const uint4 cur, uint32_t c) {
    const uint32_t words[4] = {cur.x, cur.y, cur.z, cur.w};
    const uint32_t nvalid = min(16u, used - c);
#pragma unroll
    for (int i = 0; i < 16; i++) {
      const uint32_t b = (words[i >> 2] >> (8 * (i & 3))) & 0xffu;
      const bool valid = (uint32_t)i < nvalid && !(c == 0 && i < 8) && !done;
      if (valid) {
        if (sh < 64) acc |= (uint64_t)(b & 0x7fu) << sh;
        sh += 7;
        if (!(b & 0x80u)) {
          key += acc;
          acc = 0;
          sh = 0;
          if (key >= hi) {
            done = true;
          } else if (key >= lo) {
            r.sum += key;
            r.count++;
          }
        }
      }
    }
  };
  for (uint32_t c = 0; c < used && !done; c += 64) {
    uint4 b0 = z, b1 = z, b2 = z, b3 = z;
    if (c + 64 < used) b0 = load16(leaf + c + 64);
    if (c + 80 < used) b1 = load16(leaf + c + 80);
    if (c + 96 < used) b2 = load16(leaf + c + 96);
    if (c + 112 < used) b3 = load16(leaf + c + 112);
    chunk(a0, c);
    if (c + 16 < used && !done) chunk(a1, c + 16);
    if (c + 32 < used && !done) chunk(a2, c + 32);
    if (c + 48 < used && !done) chunk(a3, c + 48);
    a0 = b0;
    a1 = b1;
    a2 = b2;
    a3 = b3;
  }
  return r;
}

}  // namespace cpma_dev
