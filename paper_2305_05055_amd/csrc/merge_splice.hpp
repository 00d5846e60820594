// Batch merge of the ordinary slices (the batch-merge phase of Section "Parallel
// Batch Updates in a PMA"): one wave per touched leaf whose keys and slice span
// less than 2^32, insert slices of at most 64 keys and delete slices of any
// length.
//
// A batch changes few codes of a leaf: new keys replace the code they split by
// their own codes and the rest of it, and a run of removed keys together with the
// next kept key becomes one code.  All other code bytes stay as they are and only
// move, so the wave neither compacts the old keys nor encodes them again.  It sums
// payloads over the bytes (every byte's key offset, K, goes to LDS; see
// splice_parse), searches the batch keys in K by byte, turns the changes into
// splices -- old bytes [a0, a1) become some new bytes -- and scans their sizes;
// then each lane collects 16 bytes of the new leaf from the unchanged stretches
// (unaligned LDS reads, one per stretch it meets) and the new codes are written
// over the gaps.
//
// Bound by vector instructions (190 of the 710 a leaf takes sum the payloads).
// 1e7 keys into 1e8 (37 into each of 267 000 leaves of 375 keys): 342 us, and their
// removal 389, against 481 each when the wave decoded the keys and encoded all of
// them again, and about 95 for reading and writing the leaves; 1e5 keys, about one a
// leaf: 70 and 77, against 110.
#pragma once
#include "merge_wave.hpp"

namespace cpma_dev {

constexpr uint32_t kSpliceRaw = kWaveMaxS;                    // old bytes
constexpr uint32_t kSpliceOut = kWaveMaxS + 13 * kWaveSlice;  // a new key adds a code and may lengthen one

template <bool kInsert>
struct SpliceLds {
  alignas(16) uint32_t K[kWaveMaxS];            // per byte: its key's offset so far; an insert's new bytes later
  alignas(16) uint8_t raw[16 + kSpliceRaw + 48];  // the old bytes, zeros around them; a delete's new bytes later
  // per splice, in order, and a closing entry: new end << 16 | a1, and in a delete
  // the new code's length << 11 (before that: a0 << 16 | a1)
  uint32_t so[kInsert ? kWaveSlice + 1 : kWaveMaxS / 2 + 2];
  uint64_t ends[kInsert ? kWaveSlice : 1];      // per lane: ends of codes in the lane before, here, in the next
  uint32_t term[kInsert ? 1 : kWaveMaxS / 32];  // ends of codes, by byte
  uint32_t gone[kInsert ? 1 : kWaveMaxS / 32];  // those of removed keys
};
static_assert(4 * kWaveMaxS >= kSpliceOut + 32, "an insert's new bytes fit over K");

// Key offsets by byte: K[p] is the offset from the segment's base of the key whose
// code ends at byte p, or for a byte before the end the part of it summed so far
// (less than the key, since a code's last group is not zero; at least the key
// before it).  K does not decrease, so the first p with K[p] >= x lies in the code
// of the first key >= x.  The head's eight bytes all hold its offset.  Returns the
// lane's 16 bits of code ends (the head's at byte 7).
__device__ __forceinline__ uint32_t splice_parse(uint4 w, uint32_t used, uint32_t head_rel, uint32_t* K) {
  const uint32_t lane = lane_id(), pos0 = 16u * lane;
  const int32_t nvalid = (int32_t)(used - pos0);  // bytes from `used` on are zero
  uint32_t vm = nvalid >= 16 ? 0xffffu : (nvalid > 0 ? (1u << nvalid) - 1u : 0u);
  uint32_t words[4] = {w.x, w.y, w.z, w.w};
  uint32_t lead = 0, head_end = 0;
  if (lane == 0 && used) {
    vm &= 0xff00u;  // the head is not a code
    lead = head_rel;
    head_end = 1u << 7;
    words[0] = 0;
    words[1] = 0;
  }
  const uint32_t msb = msb_byte(words[0], words[1]) | msb_byte(words[2], words[3]) << 8;
  uint32_t sh = 7u * dpp_prev32((uint32_t)__clz((int)~((vm & msb) << 16)));
  uint32_t run = lead, kk[16];
#pragma unroll
  for (int j = 0; j < 16; j++) {
    const uint32_t x = words[j >> 2];
    uint32_t c;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(c) : "v"(x), "i"(8 * (j & 3) + 7));
    run += __builtin_amdgcn_ubfe(x, 8 * (j & 3), 7) << (sh & 31u);
    kk[j] = run;
    sh = (sh + 7u) & c;
  }
  const uint32_t ex = dpp_incl_scan<uint32_t>(run) - run;
  uint4* dst = reinterpret_cast<uint4*>(K + pos0);
#pragma unroll
  for (int j = 0; j < 4; j++)
    dst[j] = make_uint4(kk[4 * j] + ex, kk[4 * j + 1] + ex, kk[4 * j + 2] + ex, kk[4 * j + 3] + ex);
  return (vm & ~msb) | head_end;
}

// First byte p with K[p] >= x, `used` if there is none, and K[p].  Bytes past
// `used` hold the last key's offset.
__device__ __forceinline__ uint32_t splice_find(const uint32_t* K, uint32_t used, uint32_t x, uint32_t* at) {
  uint32_t p = 0;
#pragma unroll
  for (uint32_t step = kWaveMaxS / 2; step; step /= 2) p += K[p + step - 1] < x ? step : 0u;
  *at = K[p];
  return *at < x ? used : min(p, used);
}

// 16 old bytes from offset o >= -16 (raw has zeros around them; a gap longer than
// a leaf's rest may ask for bytes further on, which are never used).
__device__ __forceinline__ uint4 splice_read(const uint8_t* raw, int o) {
  const uint32_t at = min((uint32_t)(o + 16), kSpliceRaw + 16);
  const uint32_t* q = reinterpret_cast<const uint32_t*>(raw) + at / 4;
  const uint32_t sh = 8 * (at & 3);
  const uint32_t a = q[0], b = q[1], c = q[2], d = q[3], e = q[4];
  return make_uint4(__builtin_amdgcn_alignbit(b, a, sh), __builtin_amdgcn_alignbit(c, b, sh),
                    __builtin_amdgcn_alignbit(d, c, sh), __builtin_amdgcn_alignbit(e, d, sh));
}

// Bytes [0, k) of a and [k, 16) of b, 0 < k < 16.
__device__ __forceinline__ uint4 splice_blend(uint4 a, uint4 b, uint32_t k) {
  const uint64_t m = ~0ull << (8 * (k & 7));
  const uint32_t m0 = (uint32_t)m, m1 = (uint32_t)(m >> 32);
  const bool low = k < 8;
  auto pick = [](uint32_t x, uint32_t y, uint32_t mask) { return (y & mask) | (x & ~mask); };
  return make_uint4(pick(a.x, b.x, low ? m0 : 0u), pick(a.y, b.y, low ? m1 : 0u), pick(a.z, b.z, low ? ~0u : m0),
                    pick(a.w, b.w, low ? ~0u : m1));
}

// Bytes [q, q + 16) of the new leaf (U bytes) from the old bytes the n splices
// leave; the splices' own bytes are undefined, those from U on zero.
__device__ __forceinline__ uint4 splice_gather(const uint8_t* raw, const uint32_t* so, uint32_t n, uint32_t q,
                                               uint32_t U) {
  uint32_t lo = 0, hi = n;  // the splices that end at or before q
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((so[mid] >> 16) <= q)
      lo = mid + 1;
    else
      hi = mid;
  }
  auto from = [&](uint32_t s) { return (int)q - ((int)(s >> 16) - (int)(s & 0x7ffu)); };
  uint4 v = splice_read(raw, lo ? from(so[lo - 1]) : (int)q);
  for (;;) {
    const uint32_t s = so[lo];  // so[n] closes the list
    if ((s >> 16) >= min(q + 16, U)) break;
    v = splice_blend(v, splice_read(raw, from(s)), (s >> 16) - q);
    lo++;
  }
  return q + 16 > U ? splice_blend(v, make_uint4(0, 0, 0, 0), U - q) : v;
}

template <bool kInsert>
__global__ void __launch_bounds__(kWave) k_merge_splice(MergeArgs a) {
  __shared__ SpliceLds<kInsert> L;
  uint32_t* const K = L.K;
  uint8_t* const raw = L.raw;
  const uint32_t lane = lane_id(), pos0 = 16u * lane;
  const uint32_t S = a.S;
  const uint64_t T = a.ctr->T, tstep = gridDim.x;
  uint32_t changed = 0;  // this lane's keys added or removed
  unsigned long long alg = 0;
  if (lane < 16) {
    reinterpret_cast<uint32_t*>(raw)[lane & 3] = 0;
    reinterpret_cast<uint32_t*>(raw + 16 + kSpliceRaw)[min(lane, 11u)] = 0;
  }
  // Software pipeline: the next segment's descriptor, leaf bytes and batch keys
  // are loaded while the current one is merged.
  uint4 d_cur = make_uint4(0, 0, 0, 0), d_nxt = d_cur, w_cur = d_cur, w_nxt = d_cur;
  uint32_t e_cur = 0, e_nxt = 0;
  uint64_t b_cur = 0, b_nxt = 0;
  uint64_t t = blockIdx.x;
  if (t < T) {
    d_cur = a.seg_desc[t];
    e_cur = a.seg_begin[t + 1];
    if (!d_cur.w) {
      if (pos0 < d_cur.z) w_cur = *reinterpret_cast<const uint4*>(a.bytes + (uint64_t)d_cur.x * S + pos0);
      if (lane < e_cur - d_cur.y) b_cur = a.B[d_cur.y + lane];
    }
  }
  for (; t < T; t += tstep) {
    const uint64_t tn = t + tstep;
    if (tn < T) {
      d_nxt = a.seg_desc[tn];
      e_nxt = a.seg_begin[tn + 1];
    }
    // every lane loaded the same descriptor: scalar from here on
    const uint64_t leaf = readlane_t(d_cur.x, 0);
    const uint32_t b = readlane_t(d_cur.y, 0), nb = readlane_t(e_cur, 0) - b;
    const uint32_t used0 = readlane_t(d_cur.z, 0);
    const bool routed = readlane_t(d_cur.w, 0) != 0;  // on the wide or the spill list
    uint4 w = w_cur;
    const uint64_t bj0 = b_cur;
    if (tn < T) {
      w_nxt = make_uint4(0, 0, 0, 0);
      b_nxt = 0;
      if (!readlane_t(d_nxt.w, 0)) {
        const uint8_t* np = a.bytes + (uint64_t)readlane_t(d_nxt.x, 0) * S;
        const uint32_t nb0 = readlane_t(d_nxt.y, 0);
        if (pos0 < readlane_t(d_nxt.z, 0)) w_nxt = *reinterpret_cast<const uint4*>(np + pos0);
        if (lane < readlane_t(e_nxt, 0) - nb0) b_nxt = a.B[nb0 + lane];
      }
    }
    d_cur = d_nxt;
    e_cur = e_nxt;
    w_cur = w_nxt;
    b_cur = b_nxt;
    if (routed) continue;
    // offsets count from the segment's smallest possible key: the old head or
    // the first slice key
    const uint64_t hd = readlane_t(((uint64_t)w.y << 32) | w.x, 0), b0 = readlane_t(bj0, 0);
    const uint64_t base = used0 && hd < b0 ? hd : b0;
    uint8_t* lp = a.bytes + leaf * (uint64_t)S;
    __syncthreads();  // the segment before is done with the LDS
    const uint32_t tm = splice_parse(w, used0, (uint32_t)(hd - base), K);
    *reinterpret_cast<uint4*>(raw + 16 + pos0) = w;
    uint32_t U, nsplice;
    if constexpr (kInsert) {
      const uint32_t tp = dpp_prev32(tm), tn1 = dpp_next32(tm);
      L.ends[lane] = (uint64_t)(tp | (tm << 16)) | (uint64_t)(lane < kWave - 1 ? tn1 : 0u) << 32;
      __syncthreads();
      const bool has_b = lane < nb;
      const uint32_t x = has_b ? (uint32_t)(bj0 - base) : 0u;
      uint32_t cs = used0, ce = used0;  // the old code that x is in or before
      bool isnew = has_b;
      if (has_b) {
        uint32_t v;
        const uint32_t p = splice_find(K, used0, x, &v);
        if (p < used0) {
          const uint64_t e3 = L.ends[p / 16];
          const uint32_t bit = 16 + (p & 15);
          const uint32_t after = (uint32_t)(e3 >> bit), before = (uint32_t)e3 & ((1u << bit) - 1u);
          ce = p + (uint32_t)__builtin_ctz(after | 0x80000000u) + 1;
          cs = before ? p - (p & 15) - 16 + (32u - (uint32_t)__clz((int)before)) : 0u;
          isnew = !(v == x && (p < 8 || (after & 1u)));
        }
      }
      const uint32_t mine = isnew ? cs : 0xffffffffu;
      const uint32_t x_prev = dpp_prev32(x);
      const uint32_t cs_prev = dpp_prev32(mine), cs_next = dpp_next32(mine);
      const bool same_prev = isnew && lane > 0 && cs_prev == cs;
      const bool last = isnew && !(lane < kWave - 1 && cs_next == cs);
      const bool has_pred = same_prev || cs > 0;
      uint32_t d1 = 0, d2 = 0, c1 = 0, c2 = 0;  // the key's own code and the rest of the old one
      if (isnew) {
        if (has_pred) {
          d1 = x - (same_prev ? x_prev : K[cs - 1]);
          c1 = vlen_t(d1);
        } else {
          c1 = 8;
        }
        if (last && ce > cs) {
          d2 = K[ce - 1] - x;
          c2 = vlen_t(d2);
        }
      }
      const uint32_t size = (c1 + c2) | (last ? (ce - cs) << 16 : 0u);
      const uint32_t incl = dpp_incl_scan<uint32_t>(size), ex = incl - size;
      const uint32_t at = cs + (ex & 0xffffu) - (ex >> 16);  // where the key's code goes
      const uint32_t all = lane63_u32(incl);
      U = used0 + (all & 0xffffu) - (all >> 16);
      const uint64_t newmask = __ballot(isnew), lastmask = __ballot(last);
      nsplice = (uint32_t)__popcll(lastmask);
      if (last)
        L.so[__builtin_amdgcn_mbcnt_hi((uint32_t)(lastmask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lastmask, 0u))] =
            (at + c1 + c2) << 16 | ce;
      if (lane == 0) L.so[nsplice] = 0xffff0000u;
      changed += isnew ? 1u : 0u;
      alg += used0 + (U > S ? U : (U + 15u) & ~15u) + 8ull * nb + 20;
      if (!newmask) continue;
      uint8_t* dst = lp;
      uint32_t same = readlane_t(cs, __ffsll((unsigned long long)newmask) - 1);  // bytes before it stay
      if (U > S) {
        const uint64_t off = arena_region(a, t);
        if (off + (((uint64_t)U + 15) & ~15ull) > a.arena_cap) {
          if (lane == 0) atomicOr(&a.ctr->error, 1u);
          continue;
        }
        dst = a.arena + off;
        same = 0;
        if (lane == 0) a.ovf[leaf] = off;
      }
      __syncthreads();  // K has been read: the new bytes take its place
      uint8_t* out = reinterpret_cast<uint8_t*>(K);
      for (uint32_t q = pos0; q < U; q += 16 * kWave)
        *reinterpret_cast<uint4*>(out + q) = splice_gather(raw, L.so, nsplice, q, U);
      __syncthreads();
      if (isnew) {
        put_key_bytes<uint32_t>(out + at, !has_pred, has_pred ? d1 : x, 0, base);
        if (c2) vput_t<uint32_t>(out + at + c1, d2);
      }
      __syncthreads();
      for (uint32_t q = pos0; q < U; q += 16 * kWave)
        if (q + 16 > same) *reinterpret_cast<uint4*>(dst + q) = *reinterpret_cast<const uint4*>(out + q);
      if (isnew && !has_pred) a.head[leaf] = base + (uint64_t)x;
      if (lane == 0) a.used[leaf] = U;
    } else {
      // ends of codes as a bitmap, two lanes a word
      const uint32_t tm2 = dpp_next32(tm);
      if (!(lane & 1)) {
        L.term[lane / 2] = tm | tm2 << 16;
        L.gone[lane / 2] = 0;
      }
      __syncthreads();
      for (uint32_t c0 = 0; c0 < nb; c0 += kWave) {
        const uint32_t j = c0 + lane;
        if (j < nb) {
          const uint32_t x = (uint32_t)((c0 ? a.B[b + j] : bj0) - base);
          uint32_t v;
          uint32_t p = splice_find(K, used0, x, &v);
          if (p < used0 && v == x) {
            if (p < 8) p = 7;
            if ((L.term[p / 32] >> (p & 31)) & 1u) atomicOr(&L.gone[p / 32], 1u << (p & 31));
          }
        }
      }
      __syncthreads();
      const uint32_t gone = (L.gone[lane / 2] >> (16 * (lane & 1))) & 0xffffu;
      alg += used0 + ((used0 + 15u) & ~15u) + 8ull * nb + 20;
      const uint64_t gonemask = __ballot(gone != 0);
      if (!gonemask) continue;
      changed += (uint32_t)__popc(gone);
      const uint32_t kept = tm & ~gone;
      // from the lanes before: whether their last key goes, where their last kept one ends
      const uint32_t st = tm ? 2 * lane + 2 + ((gone >> (31 - __clz((int)tm))) & 1u) : 0u;
      const uint32_t ke = kept ? pos0 + 32 - (uint32_t)__clz((int)kept) : 0u;
      const uint32_t st_all = dpp_incl_max(st), ke_all = dpp_incl_max(ke);
      const uint32_t st_in = dpp_prev32(st_all), ke_in = dpp_prev32(ke_all);
      // Kept keys with a removed one before them.  A removed key sends a carry up
      // through the bytes that end no code, which stops at the next key's end.
      uint32_t entries = ((gone << 1 | (st_in & 1u)) + (~tm & 0xffffu)) & kept;
      const uint32_t ne = (uint32_t)__popc(entries), ne_all = dpp_incl_scan<uint32_t>(ne);
      nsplice = lane63_u32(ne_all);
      // one splice per entry: from the end of the last kept key before it to its own
      for (uint32_t i = ne_all - ne; entries; entries &= entries - 1, i++) {
        const uint32_t e = (uint32_t)__builtin_ctz(entries), below = kept & ((1u << e) - 1u);
        L.so[i] = (below ? pos0 + 32 - (uint32_t)__clz((int)below) : ke_in) << 16 | (pos0 + e + 1);
      }
      if (lane == 0) L.so[nsplice] = 0xffff0000u;
      const uint32_t low = gone ? (gone & (0u - gone)) - 1u : 0u, kb = kept & low;
      const uint32_t same = readlane_t(kb ? pos0 + 32 - (uint32_t)__clz((int)kb) : ke_in,
                                       __ffsll((unsigned long long)gonemask) - 1);  // bytes before it stay
      const uint32_t end = lane63_u32(ke_all);  // what follows the last kept key goes
      __syncthreads();
      // a lane per splice: its key's new code and where it goes
      int shift = 0;  // of the old bytes behind the splices so far
      uint32_t a0 = 0, d1 = 0, at = 0;
      for (uint32_t c0 = 0; c0 < nsplice; c0 += kWave) {
        const uint32_t i = c0 + lane;
        uint32_t a1 = 0, c = 0;
        int grow = 0;
        if (i < nsplice) {
          a1 = L.so[i] & 0xffffu;
          a0 = L.so[i] >> 16;
          d1 = K[a1 - 1] - (a0 ? K[a0 - 1] : 0u);
          c = a0 ? vlen_t(d1) : 8u;
          grow = (int)(c - (a1 - a0));
        }
        const int incl = (int)dpp_incl_scan<uint32_t>((uint32_t)grow);
        if (i < nsplice) {
          at = (uint32_t)((int)a0 + shift + incl - grow);
          L.so[i] = (at + c) << 16 | c << 11 | a1;
        }
        shift += (int)lane63_u32((uint32_t)incl);
      }
      U = (uint32_t)((int)end + shift);
      __syncthreads();
      const uint4 v = pos0 < U ? splice_gather(raw, L.so, nsplice, pos0, U) : make_uint4(0, 0, 0, 0);
      __syncthreads();  // the old bytes have been read: the new ones take their place
      uint8_t* out = raw + 16;
      *reinterpret_cast<uint4*>(out + pos0) = v;
      __syncthreads();
      for (uint32_t c0 = 0; c0 < nsplice; c0 += kWave) {
        const uint32_t i = c0 + lane;
        if (i < nsplice) {
          if (nsplice > kWave) {  // else this lane's splice is at hand
            const uint32_t so = L.so[i], before = i ? L.so[i - 1] : 0u;
            at = (so >> 16) - ((so >> 11) & 15u);
            a0 = at - ((before >> 16) - (before & 0x7ffu));
            d1 = K[(so & 0x7ffu) - 1] - (a0 ? K[a0 - 1] : 0u);
          }
          put_key_bytes<uint32_t>(out + at, !a0, d1, 0, base);
          if (!a0) a.head[leaf] = base + (uint64_t)d1;
        }
      }
      __syncthreads();
      if (pos0 < used0 && pos0 + 16 > same)
        *reinterpret_cast<uint4*>(lp + pos0) = *reinterpret_cast<const uint4*>(out + pos0);
      if (lane == 0) {
        a.used[leaf] = U;
        if (!U) a.head[leaf] = kNoKey;
      }
    }
  }
  changed = wave_sum(changed);
  if (lane == 0) {
    a.part[2 * blockIdx.x] = changed;
    a.part[2 * blockIdx.x + 1] = alg;
  }
}

}  // namespace cpma_dev
