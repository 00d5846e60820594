// Query kernels: batched range_map (sum, count over [lo, hi)) and contains.
//
// range_map(start, end, f) is a search for the first element followed by a scan
// (Section "Packed Memory Array", "Design and operations"); in the CPMA the search
// runs on the uncompressed leaf heads and the scan decodes every leaf it passes
// (Section "Compressed Packed Memory Array", "Point queries").  A batch of
// queries becomes a flat list of leaf visits (query q visits leaves
// leaf(lo_q) .. leaf(hi_q - 1)).  The partial leaves at each query's ends are
// looked up; the leaves taken whole are flattened over
// all queries and split into fixed-size chunks, so long and short ranges balance
// across the GPU in one launch.
#pragma once
#include "lookup.hpp"
#include "scan_lane.hpp"
#include "update.hpp"

namespace cpma_dev {

// End leaves of every query.  With f and l the leaves of lo and of hi - 1, the
// keys of [lo, hi) are those of leaves f .. l - 1 and the ones of leaf l below hi,
// without the ones of leaf f below lo; the result initialises sum / count with
// the two partial leaves (in wrapping 64-bit arithmetic), and leaves f .. l - 1
// are the query's interior visits.  With kToEnd, lo's lookup goes on to the end of
// its leaf when l is the next one, and the query has no visits: a short range that
// runs into the next leaf then waits for no scan.  Two lookups
// per query, each stopping where it reaches its key.  A wave takes `per` lookups (4 .. 64) at a time: as many as
// it has lanes for when there are plenty, four when that leaves waves idle.
template <bool kToEnd>
__global__ void __launch_bounds__(256) k_rm_ends(QueryArgs a, uint64_t* __restrict__ first_int,
                                                 uint64_t* __restrict__ nint,
                                                 unsigned long long* __restrict__ sum,
                                                 unsigned long long* __restrict__ count,
                                                 unsigned long long* __restrict__ alg, unsigned int* ticket,
                                                 uint32_t per) {
  __shared__ Reach reach[256 / kWave][kWave];
  __shared__ uint8_t order[256 / kWave][kWave];
  Reach* const mine = reach[threadIdx.x / kWave];
  if (ticket && blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0;  // for k_rm_interior's prefix pass
  const uint32_t wave = blockIdx.x * (256 / kWave) + threadIdx.x / kWave, nwaves = gridDim.x * (256 / kWave);
  const uint32_t lane = (uint32_t)lane_id();
  uint64_t visited = 0;
  for (uint64_t base = (uint64_t)wave * per; base < 2 * a.q; base += (uint64_t)nwaves * per) {
    const uint64_t i = (base + lane) >> 1;
    const bool valid = lane < per && i < a.q;
    const uint64_t lo = valid ? a.lo[i] : 0, hi = valid ? a.hi[i] : 0;
    const bool some = lo < hi;
    // the even lane looks lo up, the odd one hi in the leaf of hi - 1
    const uint64_t leaf = wave_locate(a, valid, lane & 1 ? (some ? hi - 1 : 0) : lo);
    constexpr int kXor1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);
    const uint64_t leaf_l = dpp64<kXor1>(leaf);
    const bool whole = kToEnd && some && !(lane & 1) && leaf_l == leaf + 1;
    const Lookup r = wave_lookup<true, true, false, true>(a, valid, leaf, lane & 1 ? hi : lo, mine,
                                                          order[threadIdx.x / kWave], whole);
    const uint64_t sum_l = dpp64<kXor1>(r.sum), cnt_l = dpp64<kXor1>(r.cnt);
    if (valid && !(lane & 1)) {
      first_int[i] = whole ? leaf + 1 : leaf;
      nint[i] = some ? leaf_l - leaf - (whole ? 1 : 0) : 0;
      sum[i] = some ? sum_l + (whole ? r.sum_from : 0 - r.sum) : 0;
      count[i] = some ? cnt_l + (whole ? r.cnt_from : 0 - r.cnt) : 0;
      if (alg && some) visited += a.used[leaf_l] + (whole ? a.used[leaf] : 0u);
    }
  }
  if (alg) {  // statistics: one slot per wave (no shared counter), summed by k_fold_sum
    const uint64_t t = wave_sum(visited);
    if (lane == 0) alg[wave] = t;
  }
}

// The same for small leaves and many queries (lane_lookups): a lane per query scans its
// one or two end leaves with comparisons, and the interior visits are f + 1 .. l - 1.
// A row of 16 lanes has bytes for as many only in leaves of 256.
__global__ void __launch_bounds__(256) k_rm_ends_lane(QueryArgs a, uint64_t* __restrict__ first_int,
                                                      uint64_t* __restrict__ nint,
                                                      unsigned long long* __restrict__ sum,
                                                      unsigned long long* __restrict__ count,
                                                      unsigned long long* __restrict__ alg, unsigned int* ticket,
                                                      uint32_t) {
  if (ticket && blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0;  // for k_rm_interior's prefix pass
  uint64_t visited = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.q;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t lo = a.lo[i], hi = a.hi[i];
    uint64_t f = 0, l = 0;
    LeafSum r{0, 0};
    if (lo < hi) {
      f = locate_leaf(a.head, a.L, lo);
      l = locate_leaf(a.head, a.L, hi - 1);
      const uint32_t uf = a.used[f];
      r = leaf_sum_range(a.bytes + f * a.S, uf, lo, hi);
      visited += uf;
      if (l != f) {
        const uint32_t ul = a.used[l];
        const LeafSum r2 = leaf_sum_range(a.bytes + l * a.S, ul, lo, hi);
        r.sum += r2.sum;
        r.count += r2.count;
        visited += ul;
      }
    }
    first_int[i] = f + 1;
    nint[i] = l > f ? l - f - 1 : 0;
    sum[i] = r.sum;
    count[i] = r.count;
  }
  if (alg) {
    const uint64_t t = wave_sum(visited);
    if (lane_id() == 0) alg[((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave] = t;
  }
}

// ---- whole leaves, 32 or 64 per wave ------------------------------------------------
// Sums and counts of whole leaves, kPer lanes per leaf: one, or two (the wave's 32
// leaves need not be neighbours; lanes 2i and 2i + 1 pass the same leaf and `valid`).
// A leaf must have a successor, whose head bounds its key span.  The result is in
// the even lane; the odd lane returns zeros.
//
// With two lanes (lane_visits says when), the leaf's 64-byte rounds are split between its two lanes.  A key's offset
// from the head is the sum of the payloads of every code byte before it, each
// shifted by 7 times its place in its code, so a lane sums its own terminators'
// offsets from zero, and the second lane adds the first one's total to each of
// its keys.  The shift a code carries into the second half is 7 times the run
// of continuation bytes just before it (at most 4 within a span of 2^32, where a
// code has at most 5 bytes, and 9 otherwise).  Two lanes halve the chain of dependent rounds, which
// bounds a scan of few leaves, and give a set of 4e5 leaves twice as many waves.
//
// A round is loaded for the whole wave, four lanes to one lane's 64 bytes, and
// handed over through LDS (`stage`, 4 KiB per wave): each 64-byte line is
// requested once.  Lanes that load their own bytes, 16 at a time, ask the L1
// for each line four times, and a wave's 64 lines have often left it in
// between (3.4 times the set's bytes came over from L2 that way).  The slots
// are permuted so that the 16 lanes of an LDS access cycle cover all banks.
// The next round's loads are in flight while one is decoded.  Bound: VALU
// issue, 7.3 instructions per byte of the decode.
constexpr uint32_t kStageBytes = 64u * kWave;
constexpr uint32_t kStepLeaves = kWave / 2;

template <uint32_t kPer, bool kZero, bool kSum64, typename KT>
__device__ __forceinline__ LeafSum wave_code_sums(const QueryArgs& a, uint32_t leaf, uint64_t head, uint32_t used,
                                                  uint8_t* stage) {
  const uint32_t lane = (uint32_t)lane_id(), r = lane & (kPer - 1u);
  const uint32_t half = (used + 64u * kPer - 1u) / (64u * kPer);  // rounds of the first lane
  const uint32_t own = r ? ((used + 63u) >> 6) - half : half;
  const uint32_t start = r ? 64u * half : 0u;
  const uint32_t R = lane63_u32(dpp_incl_max(half));
  // this lane loads, for run 16 j + lane / 4, the chunk that goes to slot lane % 4
  const uint8_t* src[4];
  uint32_t cnt[4];
  const uint32_t ol = opaque_lane();
#pragma unroll
  for (uint32_t j = 0; j < 4; j++) {
    const uint32_t o = 16u * j + (ol >> 2);
    const uint32_t lf = from_lane(leaf, o);
    const uint32_t w = from_lane(start | (own << 16), o);
    cnt[j] = w >> 16;
    src[j] = a.bytes + (uint64_t)lf * a.S + (w & 0xffffu) + 16u * ((ol & 3u) ^ ((o >> 2) & 3u));
  }
  // the run of continuation bytes just before this lane's part
  uint32_t tail = 0;
  if (r && own) {
    const uint8_t* part = a.bytes + leaf * (uint64_t)a.S + start;
    if constexpr (sizeof(KT) == 8) {
      tail = tail_run<KT>(load16(part - 16));
    } else {
      const uint32_t ends = ~*reinterpret_cast<const uint32_t*>(part - 4) & 0x80808080u;
      tail = ends ? (uint32_t)__clz((int)ends) >> 3 : 4u;
    }
  }
  uint4 nx[4];
#pragma unroll
  for (uint32_t j = 0; j < 4; j++) {
    nx[j] = make_uint4(0, 0, 0, 0);
    if (cnt[j]) nx[j] = load16(src[j]);
  }
  KT D = 0;
  uint32_t cont = 0, sh = 7u * tail;
  uint64_t Sc = 0;
  uint4* const put = reinterpret_cast<uint4*>(stage) + lane;
  const uint4* const get = reinterpret_cast<const uint4*>(stage) + 4u * lane;
  const uint32_t perm = (lane >> 2) & 3u;
#pragma unroll 1
  for (uint32_t t = 0; t < R; t++) {
#pragma unroll
    for (uint32_t j = 0; j < 4; j++) put[kWave * j] = nx[j];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    uint4 w = get[perm];
#pragma unroll
    for (uint32_t j = 0; j < 4; j++)
      if (t + 1 < cnt[j]) nx[j] = load16(src[j] + 64u * (t + 1));
    if (t < own) {
      if (t == 0 && r == 0) {
        // the head's eight bytes: seven continuation bytes without payload
        // and a terminator, so one key at offset 0
        w.x = 0x80808080u;
        w.y = 0x00808080u;
      }
#pragma unroll
      for (uint32_t c = 0; c < 4; c++) {
        // one chunk's bytes at a time: the scheduler would otherwise spread all
        // four over the registers and cost a wave of occupancy
        const uint4 ahead = get[(c < 3 ? c + 1 : c) ^ perm];
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!kZero) {
          // bytes at or past `used` (values may lie there) become 0x80
          const int32_t nv = (int32_t)used - (int32_t)(start + 64u * t + 16u * c);
          if (nv < 16) {
            uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int k = 0; k < 4; k++) {
              const int32_t v = nv - 4 * k;
              const uint32_t keep = v >= 4 ? 0xffffffffu : (v <= 0 ? 0u : ((1u << (8 * v)) - 1u));
              x[k] = (x[k] & keep) | (0x80808080u & ~keep);
            }
            w = make_uint4(x[0], x[1], x[2], x[3]);
          }
        }
        zf_chunk<kSum64, KT>(w, D, sh, Sc, cont);
        w = ahead;
      }
    }
    __builtin_amdgcn_wave_barrier();  // the next round's writes follow every lane's reads
  }
  uint32_t keys = 64u * own - cont;
  if constexpr (kZero) {
    // bytes past `used` are zero; each decoded as a zero delta, one more copy of the last key
    const uint32_t from = max(used, start), end = start + 64u * own;
    const uint32_t zeros = own && end > from ? end - from : 0u;
    keys -= zeros;
    Sc -= (uint64_t)zeros * D;
  }
  if constexpr (kPer == 1) return LeafSum{Sc + (uint64_t)keys * head, keys};
  constexpr int kXor1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);  // DPP quad permutation: the pair's other lane
  KT D0;
  if constexpr (sizeof(KT) == 8)
    D0 = dpp64<kXor1>(D);
  else
    D0 = dpp32<kXor1>(D);
  uint64_t s = Sc + (uint64_t)keys * (head + (r ? D0 : (KT)0));
  s += dpp64<kXor1>(s);
  keys += dpp32<kXor1>(keys);
  return r ? LeafSum{0, 0} : LeafSum{s, keys};
}

struct __attribute__((packed, aligned(8))) WordPair {  // values begin at any multiple of 8
  uint64_t a, b;
};

// Sums of 8-byte words of 32 leaves (lane 2i, and 2i + 1 alike: m words at byte
// `at` of `leaf`), eight lanes per leaf and eight leaves at a time.
__device__ __forceinline__ LeafSum wave_word_sums(const QueryArgs& a, uint32_t leaf, uint32_t at, uint32_t m) {
  const uint32_t l = opaque_lane();
  LeafSum out{0, 0};
#pragma unroll 1
  for (uint32_t it = 0; it < 4; it++) {
    const uint32_t from = 16u * it + 2u * (l >> 3);
    const uint64_t lf = from_lane(leaf, from);
    const uint32_t n = from_lane(m, from);
    const WordPair* w = reinterpret_cast<const WordPair*>(a.bytes + lf * a.S + from_lane(at, from));
    uint64_t s = 0;
    // 512 bytes of every leaf in flight; the last pair's second word may be past the end
    for (uint32_t i = l & 7u; 2 * i < n; i += 32) {
      WordPair p[4];
#pragma unroll
      for (uint32_t k = 0; k < 4; k++) {
        p[k] = WordPair{0, 0};
        if (2 * (i + 8 * k) + 1 < n)
          p[k] = w[i + 8 * k];
        else if (2 * (i + 8 * k) < n)
          p[k].a = w[i + 8 * k].a;
      }
      s += ((p[0].a + p[0].b) + (p[1].a + p[1].b)) + ((p[2].a + p[2].b) + (p[3].a + p[3].b));
    }
    constexpr int kXor1 = 1 | (0 << 2) | (3 << 4) | (2 << 6), kXor2 = 2 | (3 << 2) | (0 << 4) | (1 << 6);
    s += dpp64<kXor1>(s);
    s += dpp64<kXor2>(s);
    s += dpp64<0x141>(s);  // the row's other quad of the eight
    const uint64_t mine = from_lane(s, 4u * (l & 14u));
    if ((l >> 4) == it && !(l & 1u)) out = LeafSum{mine, m};
  }
  return out;
}

// What an interior visit sums: the keys of leaves that are zero past `used` (every
// compressed set without values), the keys of key-value leaves, or 8-byte words (an
// uncompressed leaf's keys, a key-value leaf's values).  One kernel instance each:
// together the decoders need more registers than four waves per SIMD leave.
enum class Visit { kPlain, kCodes, kWords };

template <Visit kVisit, uint32_t kPer>
__device__ __forceinline__ LeafSum wave_leaf_sums(const QueryArgs& a, uint32_t leaf, bool valid, uint8_t* stage,
                                                  uint32_t& visited) {
  const uint32_t r = (uint32_t)lane_id() & (kPer - 1u);
  const uint32_t u = valid ? a.used[leaf] : 0u;
  if (!r) visited += u;
  if constexpr (kVisit == Visit::kWords) {
    // the values at the leaf's end, or the keys from its start
    const uint32_t m = !valid ? 0u : (a.vals ? (a.fill[leaf] - u) / 8 : u / 8);
    return wave_word_sums(a, leaf, a.vals ? a.S - 8u * m : 0u, m);
  }
  constexpr bool kPlain = kVisit == Visit::kPlain;
  const uint64_t h = u ? a.head[leaf] : 0;
  const uint64_t span = u ? a.head[leaf + 1] - h : 0;
  // three classes of leaves, each decoded at once: offsets and a chunk's sum in 32
  // bits, 32-bit offsets summed in 64, and 64-bit offsets (one lane walking such a
  // leaf alone took 80 us at 1 KiB and 300 at 4; thirty scans of a whole set of 63-bit
  // keys 665 us, 191 now)
  const bool mid = span >= (1ull << 28) && span < (1ull << 32), wide = span >= (1ull << 32);
  LeafSum x = wave_code_sums<kPer, kPlain, false, uint32_t>(a, leaf, h, mid || wide ? 0u : u, stage);
  if (__ballot(mid || wide)) {
    if (__ballot(mid)) {
      const LeafSum y = wave_code_sums<kPer, kPlain, true, uint32_t>(a, leaf, h, mid ? u : 0u, stage);
      if (mid) x = y;
    }
    if (__ballot(wide)) {
      const LeafSum y = wave_code_sums<kPer, kPlain, true, uint64_t>(a, leaf, h, wide ? u : 0u, stage);
      if (wide) x = y;
    }
  }
  return x;
}

// Per-leaf prefix sums, for a batch of queries that visits more interior leaves
// than the set has: every leaf is then summed once and a query's interior is
// the difference of two prefixes, exact in wrapping 64-bit arithmetic.  A block
// takes one run of `range` leaves, its waves 32 leaves at a time.
//   ps / pc: exclusive prefix of the leaf sums / counts inside groups of 32 leaves;
//   ss / sc: the 32 leaves' totals, then their exclusive prefix in the run;
//   ts / tc: the runs' totals, then their exclusive prefix.
// ps NULL: no memory for it, visit leaf by leaf.  10^6 Zipf(1.2) queries on
// 10^8 keys visit 1.4e10 / 270 leaves: 7.28 ms leaf by leaf.
struct LeafPrefix {
  uint64_t *ps, *ss, *ts, *sc, *tc;
  uint32_t* pc;
  unsigned int* ticket;  // blocks done; zeroed by the end-leaf kernel
  uint32_t range;        // a multiple of 32
};
// Up to this many queries the last block of the prefix pass applies the
// prefixes itself, which saves the launch of k_rm_prefix_apply (2.5 us, also
// when the visits were few) but costs every block an agent-scope release, a
// write-back of its XCD's L2 (25 us in all on a full grid, 110 us when every
// wave did one).
constexpr uint64_t kPrefixInline = 64;
constexpr uint32_t kPrefixRuns = 2048;  // blocks of the prefix pass, at most

__device__ __forceinline__ LeafSum prefix_at(const LeafPrefix& lp, const uint64_t* ts, const uint64_t* tc,
                                              uint64_t f) {
  const uint32_t run = (uint32_t)f / lp.range;
  return LeafSum{lp.ps[f] + lp.ss[f / kStepLeaves] + ts[run], lp.pc[f] + lp.sc[f / kStepLeaves] + tc[run]};
}

__device__ __forceinline__ void prefix_apply(const LeafPrefix& lp, const uint64_t* ts, const uint64_t* tc,
                                             uint64_t first, uint64_t n, uint64_t i, unsigned long long* sum,
                                             unsigned long long* count) {
  const LeafSum e = prefix_at(lp, ts, tc, first + n), b = prefix_at(lp, ts, tc, first);
  sum[i] += e.sum - b.sum;
  count[i] += e.count - b.count;
}

// Exclusive scan of v[0, n) and w[0, n) in place by a block of 256 threads;
// returns the totals.
__device__ __forceinline__ LeafSum block_scan_pairs(uint64_t* v, uint64_t* w, uint64_t n, uint64_t (*red)[4]) {
  const uint32_t tid = threadIdx.x, wid = tid / kWave;
  LeafSum run{0, 0};
  for (uint64_t base = 0; base < n; base += 1024) {
    const uint64_t i0 = base + 4 * tid;
    uint64_t x[4], y[4], s = 0, c = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      x[j] = i0 + j < n ? v[i0 + j] : 0;
      y[j] = i0 + j < n ? w[i0 + j] : 0;
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
      s += x[j];
      c += y[j];
    }
    const uint64_t is = wave_incl_scan(s), ic = wave_incl_scan(c);
    __syncthreads();
    if (lane_id() == kWave - 1) {
      red[0][wid] = is;
      red[1][wid] = ic;
    }
    __syncthreads();
    uint64_t ps = run.sum + is - s, pc = run.count + ic - c;
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) {
      if (k < wid) {
        ps += red[0][k];
        pc += red[1][k];
      }
      run.sum += red[0][k];
      run.count += red[1][k];
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
      if (i0 + j < n) {
        v[i0 + j] = ps;
        w[i0 + j] = pc;
      }
      ps += x[j];
      pc += y[j];
    }
  }
  return run;
}

// The end of the prefix pass, after a block's waves have written their leaves:
// the run's prefix, and for few queries, in the last block to finish, the rest.
__device__ __forceinline__ void leaf_prefix_finish(const QueryArgs& a, const LeafPrefix& lp,
                                                   const uint64_t* __restrict__ ioff,
                                                   const uint64_t* __restrict__ first_int,
                                                   unsigned long long* __restrict__ sum,
                                                   unsigned long long* __restrict__ count, uint64_t f0, uint64_t f1) {
  __shared__ uint64_t red[2][4];
  __shared__ bool last;
  const uint32_t tid = threadIdx.x;
  __threadfence_block();
  __syncthreads();
  const uint64_t g0 = f0 / kStepLeaves, g1 = (f1 + kStepLeaves - 1) / kStepLeaves;
  const LeafSum t = f0 < f1 ? block_scan_pairs(lp.ss + g0, lp.sc + g0, g1 - g0, red) : LeafSum{0, 0};
  if (tid == 0) {
    lp.ts[blockIdx.x] = t.sum;
    lp.tc[blockIdx.x] = t.count;
  }
  if (a.q > kPrefixInline) return;
  __syncthreads();
  if (tid == 0) {
    __threadfence();  // after the barrier: the whole block's writes
    last = atomicAdd(lp.ticket, 1u) + 1u == gridDim.x;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  block_scan_pairs(lp.ts, lp.tc, gridDim.x, red);
  __threadfence_block();
  __syncthreads();
  for (uint64_t i = tid; i < a.q; i += 256) {
    const uint64_t n = ioff[i + 1] - ioff[i];
    if (n) prefix_apply(lp, lp.ts, lp.tc, first_int[i], n, i, sum, count);
  }
}

// Interior visits, flattened over all queries.  When they outnumber the leaves,
// every leaf is summed once into the prefixes above, a block taking one run of
// leaves.  Otherwise waves take groups of consecutive visits, group g by wave
// g mod (number of waves): `chunk` steps of 64 leaves, fewer when that would leave
// waves idle.  Part of a group: 64 visits with a lane each or 32 with two, so the
// wave's loads fall on neighbouring leaves, and the waves running at the same time
// sweep one region of the leaf array together.  The
// query of a group's first visit is found by one binary search over the visit
// offsets, with wave-uniform (scalar) loads; each lane then walks forward to its
// own visit's query, and the next part continues from there.  Partial sums are
// exact integers, so they may be combined in any order:
//  * while every visit of a part belongs to the same query, each lane adds its
//    leaf to a running share; the shares are summed across the wave and
//    flushed with one pair of 64-bit atomics when the query changes;
//  * a part whose lanes span several queries is reduced at once by query
//    (visits ascend with the lane, so equal queries sit in runs of lanes), one
//    pair of atomics per run -- a query spanning millions of leaves would
//    otherwise serialise on one address.
template <Visit kVisit, uint32_t kPer>
__device__ __forceinline__ void interior_visits(const QueryArgs& a, const uint64_t* __restrict__ ioff,
                                                const uint64_t* __restrict__ first_int, uint32_t chunk,
                                                unsigned long long* __restrict__ sum,
                                                unsigned long long* __restrict__ count,
                                                unsigned long long* __restrict__ alg, const LeafPrefix& lp,
                                                uint8_t* stage) {
  constexpr uint32_t kStep = kWave / kPer;  // leaves at a time
  const int lane = lane_id();
  const uint64_t V = uniform64(ioff[a.q]);
  const bool by_prefix = lp.ps && V > a.L;
  uint32_t visited = 0;  // used bytes this lane's leaves hold
  // this wave's items (leaves or visits): groups of G from g * G on, every `step`-th group
  uint64_t G, g, step, end;
  uint64_t f0 = 0, f1 = 0;
  if (by_prefix) {
    f0 = min(a.L, (uint64_t)blockIdx.x * lp.range);
    f1 = min(a.L, f0 + lp.range);
    G = kStep;
    g = f0 / kStep + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    step = 256 / kWave;
    end = f0 < f1 ? f1 : 0;
  } else {
    step = (uint64_t)gridDim.x * (256 / kWave);
    g = (uint64_t)blockIdx.x * (256 / kWave) + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint64_t share = (V + step - 1) / step;
    G = max<uint64_t>(1, min<uint64_t>((uint64_t)kWave * chunk, (share + kStep - 1) / kStep * kStep));
    end = V;
  }
  uint64_t cq = ~0ull, cs = 0;  // carried query (wave-uniform) and this lane's share of its sum
  uint32_t cn = 0;              // and count
  auto flush_carry = [&]() {
    if (cq != ~0ull) {
      const uint64_t ts = wave_sum<uint64_t>(cs), tn = wave_sum<uint64_t>((uint64_t)cn);
      if (lane == 0 && tn) {
        atomicAdd(&sum[cq], (unsigned long long)ts);
        atomicAdd(&count[cq], (unsigned long long)tn);
      }
    }
    cq = ~0ull;
    cs = 0;
    cn = 0;
  };
  for (; g * G < end; g += step) {
    const uint64_t Wend = min((g + 1) * G, end);
    // the query of the group's first visit; then of the part before
    uint64_t q0 = by_prefix ? 0 : uniform64(upper_bound_u64(ioff, a.q + 1, g * G) - 1);
    for (uint64_t base = g * G; base < Wend; base += kStep) {
      const uint64_t v = base + (uint32_t)lane / kPer;
      uint64_t vq = ~0ull;
      uint32_t leaf = (uint32_t)v;
      if (!by_prefix && v < Wend) {
        uint64_t qi = q0;
        // a few steps forward, then (many queries without interior leaves in
        // between) a search
        for (int steps = 0; ioff[qi + 1] <= v; qi++)
          if (++steps > 8) {
            qi += upper_bound_u64(ioff + qi, a.q + 1 - qi, v) - 1;
            break;
          }
        vq = qi;
        leaf = (uint32_t)(first_int[qi] + (v - ioff[qi]));
      }
      // nothing lies after the last leaf: no prefix needs its sum
      const LeafSum x = wave_leaf_sums<kVisit, kPer>(a, leaf, v < Wend && leaf + 1ull < a.L, stage, visited);
      uint64_t s = x.sum;
      uint32_t n = (uint32_t)x.count;
      if (by_prefix) {
        uint64_t is = wave_incl_scan(s);
        uint32_t ic = wave_incl_scan(n);
        if (kPer == 1) {  // two groups of kStepLeaves
          const uint64_t s31 = from_lane(is, kStepLeaves - 1);
          const uint32_t c31 = from_lane(ic, kStepLeaves - 1);
          if (lane >= (int)kStepLeaves) {
            is -= s31;
            ic -= c31;
          }
        }
        if (!(lane & (kPer - 1u)) && v < Wend) {
          lp.ps[v] = is - s;
          lp.pc[v] = ic - n;
        }
        const uint64_t group = base / kStepLeaves + (kPer == 1 ? (uint32_t)lane / kStepLeaves : 0u);
        if ((kPer == 1 ? (lane & (kStepLeaves - 1u)) == kStepLeaves - 1u : lane == kWave - 1) &&
            group * kStepLeaves < Wend) {
          lp.ss[group] = is;
          lp.sc[group] = ic;
        }
        continue;
      }
      q0 = uniform64(vq);
      const bool uni = __ballot(vq != q0) == 0;
      if (uni && q0 == cq) {
        cs += s;
        cn += n;
        continue;
      }
      flush_carry();
      if (uni) {
        cq = q0;
        cs = s;
        cn = n;
        continue;
      }
      // several queries in this part: segmented inclusive scan over runs of equal vq
      const uint32_t ol = opaque_lane();
#pragma unroll
      for (uint32_t d = 1; d < kWave; d <<= 1) {
        const uint64_t qu = from_lane(vq, ol - d);
        const uint64_t su = from_lane(s, ol - d);
        const uint32_t nu = from_lane(n, ol - d);
        if (ol >= d && qu == vq) {
          s += su;
          n += nu;
        }
      }
      const uint64_t qn = from_lane(vq, ol + 1);  // every lane takes part
      const bool run_end = ol == kWave - 1 || qn != vq;
      if (run_end && vq != ~0ull && n) {
        atomicAdd(&sum[vq], (unsigned long long)s);
        atomicAdd(&count[vq], (unsigned long long)n);
      }
    }
  }
  if (by_prefix) {
    leaf_prefix_finish(a, lp, ioff, first_int, sum, count, f0, f1);
  } else {
    // what the block's waves carry at the end: one pair of atomics per query, since a
    // scan of one query ends with all of them on one address, about 7 ns each
    __shared__ uint64_t end_q[256 / kWave], end_s[256 / kWave], end_n[256 / kWave];
    const uint64_t ts = wave_sum<uint64_t>(cs), tn = wave_sum<uint64_t>((uint64_t)cn);
    if (lane == 0) {
      end_q[threadIdx.x / kWave] = cq;
      end_s[threadIdx.x / kWave] = ts;
      end_n[threadIdx.x / kWave] = tn;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      uint64_t s = 0, n = 0;
      for (uint32_t w = 0; w < 256 / kWave; w++) {
        s += end_s[w];
        n += end_n[w];
        if (w + 1 < 256 / kWave && end_q[w + 1] == end_q[w]) continue;
        if (end_q[w] != ~0ull && n) {
          atomicAdd(&sum[end_q[w]], (unsigned long long)s);
          atomicAdd(&count[end_q[w]], (unsigned long long)n);
        }
        s = n = 0;
      }
    }
  }
  if (alg) {
    const uint64_t t = wave_sum((uint64_t)visited);
    if (lane_id() == 0) alg[((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave] = t;
  }
}

// Leaves a scan sums from which on each gets one lane, not two.  Two lanes halve a
// leaf's chain of 64-byte rounds, which bounds a scan of few leaves; one lane wastes
// no half round and takes 64 leaves per wait for memory.  The fewer rounds a leaf has,
// the sooner that counts; about a third of a key-value leaf is codes.  One lane and
// two: whole scans of 5e6 40-bit keys at 256 bytes a leaf (80 000 leaves) 20 and 23 us, of
// 5e7 and 2e8 at 1 KiB 53 and 56, 128 and 134, of 2e8 at 2 KiB 125 and 136; but four
// scans of 3e5 key-value keys at 1 KiB (22 000 visits) 26 and 18, ranges of 3000 keys
// among 5e6 at 1 and 2 KiB 32 and 27, 43 and 33, 1000 ranges of 1e5 keys at 4 KiB (72 000
// visits) 96 and 77.
__host__ __device__ inline uint64_t lane_visits(const QueryArgs& a) {
  const uint32_t codes = a.zero_fill ? a.S : a.S / 2;
  return codes <= 512 ? 32768 : (codes <= 2048 ? 65536 : 262144);
}

// Batches of up to kOwnScanQueries queries: every block scans the visit counts itself,
// into LDS (block 0 also to memory, for k_rm_prefix_apply), which takes it a
// microsecond; a launch for it costs 2.8.
constexpr uint32_t kOwnScanQueries = 1024;
__device__ __forceinline__ void visit_offsets(const uint64_t* __restrict__ nint, uint32_t q, uint64_t* offs,
                                              uint64_t* __restrict__ ioff) {
  __shared__ uint64_t red[4];
  const uint32_t i0 = 4 * threadIdx.x, wid = threadIdx.x / kWave;
  uint64_t x[4], t = 0;
#pragma unroll
  for (uint32_t j = 0; j < 4; j++) {
    x[j] = i0 + j < q ? nint[i0 + j] : 0;
    t += x[j];
  }
  const uint64_t incl = wave_incl_scan(t);
  if (lane_id() == kWave - 1) red[wid] = incl;
  __syncthreads();
  uint64_t at = incl - t;
#pragma unroll
  for (uint32_t w = 0; w < 4; w++) at += w < wid ? red[w] : 0;
#pragma unroll
  for (uint32_t j = 0; j < 4; j++) {
    if (i0 + j <= q) {
      offs[i0 + j] = at;
      if (blockIdx.x == 0) ioff[i0 + j] = at;
    }
    at += x[j];
  }
  if (q == kOwnScanQueries && threadIdx.x == 255) {
    offs[q] = at;
    if (blockIdx.x == 0) ioff[q] = at;
  }
  __syncthreads();
}

// Compressed leaves (kPlain: zero past `used`; the other instance takes three waves
// per SIMD, at four it spills 46 registers: a scan of 5e7 key-value keys 117 and 87 us).
// nint: with few queries, the visit counts to scan.
template <bool kPlain>
__global__ void __launch_bounds__(256, kPlain ? 4 : 3) k_rm_interior(QueryArgs a, uint64_t* __restrict__ ioff,
                                                     const uint64_t* __restrict__ nint,
                                                     const uint64_t* __restrict__ first_int, uint32_t chunk,
                                                     unsigned long long* __restrict__ sum,
                                                     unsigned long long* __restrict__ count,
                                                     unsigned long long* __restrict__ alg, LeafPrefix lp) {
  __shared__ __align__(16) uint8_t stages[256 / kWave][kStageBytes];
  __shared__ uint64_t offs[kOwnScanQueries + 1];
  constexpr Visit kVisit = kPlain ? Visit::kPlain : Visit::kCodes;
  uint8_t* const stage = stages[threadIdx.x / kWave];
  auto visits = [&](const uint64_t* off) {
    const uint64_t V = uniform64(off[a.q]);
    if ((lp.ps && V > a.L ? a.L : V) >= lane_visits(a))
      interior_visits<kVisit, 1>(a, off, first_int, chunk, sum, count, alg, lp, stage);
    else
      interior_visits<kVisit, 2>(a, off, first_int, chunk, sum, count, alg, lp, stage);
  };
  if (a.q <= kOwnScanQueries) {
    visit_offsets(nint, (uint32_t)a.q, offs, ioff);
    visits(offs);
  } else {
    visits(ioff);
  }
}

// 8-byte words.
__global__ void __launch_bounds__(256, 4) k_rm_words(QueryArgs a, uint64_t* __restrict__ ioff,
                                                  const uint64_t* __restrict__ nint,
                                                  const uint64_t* __restrict__ first_int, uint32_t chunk,
                                                  unsigned long long* __restrict__ sum,
                                                  unsigned long long* __restrict__ count,
                                                  unsigned long long* __restrict__ alg, LeafPrefix lp) {
  __shared__ uint64_t offs[kOwnScanQueries + 1];
  if (a.q <= kOwnScanQueries) {
    visit_offsets(nint, (uint32_t)a.q, offs, ioff);
    interior_visits<Visit::kWords, 2>(a, offs, first_int, chunk, sum, count, alg, lp, nullptr);
  } else {
    interior_visits<Visit::kWords, 2>(a, ioff, first_int, chunk, sum, count, alg, lp, nullptr);
  }
}

// After a prefix pass of more than kPrefixInline queries (the same test as in
// k_rm_interior): every query's interior from the prefixes.  Each block scans
// the runs' totals for itself.
__global__ void __launch_bounds__(256) k_rm_prefix_apply(QueryArgs a, const uint64_t* __restrict__ ioff,
                                                         const uint64_t* __restrict__ first_int, LeafPrefix lp,
                                                         uint32_t runs, unsigned long long* __restrict__ sum,
                                                         unsigned long long* __restrict__ count) {
  if (ioff[a.q] <= a.L) return;
  __shared__ uint64_t ts[kPrefixRuns], tc[kPrefixRuns], red[2][4];
  for (uint32_t i = threadIdx.x; i < runs; i += 256) {
    ts[i] = lp.ts[i];
    tc[i] = lp.tc[i];
  }
  __syncthreads();
  block_scan_pairs(ts, tc, runs, red);
  __syncthreads();
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.q;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t n = ioff[i + 1] - ioff[i];
    if (n) prefix_apply(lp, ts, tc, first_int[i], n, i, sum, count);
  }
}

// Sum of n per-wave statistics slots, added to *out (one block).
__global__ void __launch_bounds__(1024) k_fold_sum(const unsigned long long* __restrict__ part, uint64_t n,
                                                   unsigned long long* out) {
  __shared__ uint64_t red[1024 / kWave];
  uint64_t t = 0;
  for (uint64_t i = threadIdx.x; i < n; i += blockDim.x) t += part[i];
  t = wave_sum(t);
  if (lane_id() == 0) red[threadIdx.x / kWave] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < (int)(blockDim.x / kWave); i++) t += red[i];
    atomicAdd(out, (unsigned long long)t);
  }
}

// Values of key-value leaves: found[i] = whether keys[i] is present, val[i] its
// value (0 if not).  per: as in k_rm_ends.
__global__ void __launch_bounds__(256) k_kv_get(QueryArgs a, const uint64_t* __restrict__ keys,
                                                uint64_t* __restrict__ val, uint8_t* __restrict__ found,
                                                uint32_t per) {
  __shared__ Reach reach[256 / kWave][kWave];
  Reach* const mine = reach[threadIdx.x / kWave];
  const uint32_t wave = blockIdx.x * (256 / kWave) + threadIdx.x / kWave, nwaves = gridDim.x * (256 / kWave);
  for (uint64_t base = (uint64_t)wave * per; base < a.q; base += (uint64_t)nwaves * per) {
    const uint64_t i = base + lane_id();
    const bool valid = (uint32_t)lane_id() < per && i < a.q;
    const uint64_t x = valid ? keys[i] : 0;
    const uint64_t leaf = wave_locate(a, valid, x);
    const Lookup r = wave_lookup<true, false, true>(a, valid, leaf, x, mine);
    if (valid) {
      uint64_t v = 0;
      if (r.eq) {
        const uint32_t m = (a.fill[leaf] - a.used[leaf]) / 8;
        v = reinterpret_cast<const uint64_t*>(a.bytes + leaf * (uint64_t)a.S + a.S - 8u * m)[r.cnt];
      }
      val[i] = v;
      found[i] = r.eq ? 1 : 0;
    }
  }
}

// Membership.  n: the number of keys on the device (NULL: a.q).
__global__ void __launch_bounds__(256) k_contains(QueryArgs a, const uint64_t* __restrict__ keys,
                                                  uint8_t* __restrict__ out, uint32_t per,
                                                  const unsigned long long* __restrict__ n) {
  __shared__ Reach reach[256 / kWave][kWave];
  Reach* const mine = reach[threadIdx.x / kWave];
  const uint32_t wave = blockIdx.x * (256 / kWave) + threadIdx.x / kWave, nwaves = gridDim.x * (256 / kWave);
  const uint64_t q = n ? (uint64_t)*n : a.q;
  for (uint64_t base = (uint64_t)wave * per; base < q; base += (uint64_t)nwaves * per) {
    const uint64_t i = base + lane_id();
    const bool valid = (uint32_t)lane_id() < per && i < q;
    const uint64_t x = valid ? keys[i] : 0;
    const Lookup r = wave_lookup<false, false, true>(a, valid, wave_locate(a, valid, x), x, mine);
    if (valid) out[i] = r.eq ? 1 : 0;
  }
}

// The same for small leaves and many keys (lane_lookups): a lane per key.
__global__ void __launch_bounds__(256) k_contains_lane(QueryArgs a, const uint64_t* __restrict__ keys,
                                                       uint8_t* __restrict__ out, uint32_t,
                                                       const unsigned long long* __restrict__ n) {
  const uint64_t q = n ? (uint64_t)*n : a.q;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < q; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t x = keys[i], leaf = locate_leaf(a.head, a.L, x);
    out[i] = leaf_sum_range(a.bytes + leaf * a.S, a.used[leaf], x, x + 1).count ? 1 : 0;
  }
}

}  // namespace cpma_dev
