// Merges of long insert slices into their leaves (the batch-merge phase of Section
// "Parallel Batch Updates in a PMA" for slices too long for the one-key-per-lane
// wave merge or for one lane): one block per slice, and for the longest slices
// one block per piece of a slice.
#pragma once
#include "merge_wave.hpp"
#include "update.hpp"

namespace cpma_dev {

constexpr uint32_t kHeavyThreads = 256;
constexpr uint32_t kHeavyLds = 1024;   // merged keys held in LDS beyond a full leaf's
constexpr uint32_t kGiantSlice = 4096; // longer slices are merged piece by piece
constexpr uint32_t kGiantPiece = 1024; // batch keys per piece

// Exclusive scan of one value per thread over a block of kHeavyThreads; *total: the sum.
__device__ __forceinline__ uint32_t heavy_scan(uint32_t v, uint32_t* wsum, uint32_t* total) {
  const uint32_t wid = threadIdx.x / kWave;
  const uint32_t incl = wave_incl_scan(v);
  __syncthreads();
  if (lane_id() == kWave - 1) wsum[wid] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (uint32_t w = 0; w < kHeavyThreads / kWave; w++) {
    before += w < wid ? wsum[w] : 0u;
    all += wsum[w];
  }
  *total = all;
  return before + incl - v;
}

// Exclusive prefix sum of F[0, n) in place; returns the total.
__device__ __forceinline__ uint32_t heavy_scan_inplace(uint32_t* F, uint32_t n, uint32_t* wsum) {
  const uint32_t per = (n + kHeavyThreads - 1) / kHeavyThreads;
  const uint32_t i0 = min(n, per * threadIdx.x), i1 = min(n, i0 + per);
  uint32_t s = 0, total;
  for (uint32_t i = i0; i < i1; i++) s += F[i];
  uint32_t run = heavy_scan(s, wsum, &total);
  for (uint32_t i = i0; i < i1; i++) {
    const uint32_t v = F[i];
    F[i] = run;
    run += v;
  }
  __syncthreads();
  return total;
}

// Encoding of keys C[0, m) as one run of codes: every thread takes consecutive
// keys, whose byte counts a block scan turns into output offsets.  has_pred: the
// run starts with the code of C[0] - pred, else with a leaf's head (8 bytes).
struct HeavyRun {
  uint32_t i0, i1, off;  // this thread's keys and its byte offset
  uint32_t total;
};
template <typename KT>
__device__ __forceinline__ uint32_t heavy_cost(const KT* C, uint32_t i, bool has_pred, KT pred) {
  return i ? vlen_t((KT)(C[i] - C[i - 1])) : (has_pred ? vlen_t((KT)(C[0] - pred)) : 8u);
}
template <typename KT>
__device__ __forceinline__ HeavyRun heavy_plan(const KT* C, uint32_t m, bool has_pred, KT pred, uint32_t* wsum) {
  HeavyRun r;
  const uint32_t per = (m + kHeavyThreads - 1) / kHeavyThreads;
  r.i0 = min(m, per * threadIdx.x);
  r.i1 = min(m, r.i0 + per);
  uint32_t s = 0;
  for (uint32_t i = r.i0; i < r.i1; i++) s += heavy_cost(C, i, has_pred, pred);
  r.off = heavy_scan(s, wsum, &r.total);
  return r;
}
template <typename KT, typename P>
__device__ __forceinline__ void heavy_encode(const KT* C, const HeavyRun& r, bool has_pred, KT pred, uint64_t base,
                                             P dst) {
  auto p = dst + r.off;
  for (uint32_t i = r.i0; i < r.i1; i++) {
    if (i == 0 && !has_pred) {
      put_le64(p, base + (uint64_t)C[0]);
      p += 8;
    } else {
      KT d = C[i] - (i ? C[i - 1] : pred);
      while (d >= 0x80) {
        *p++ = (uint8_t)(d | 0x80);
        d >>= 7;
      }
      *p++ = (uint8_t)d;
    }
  }
}

// LDS of k_merge_heavy for leaf size S and merged-key room cap beyond a full
// leaf (byte offsets, each 16-byte aligned for even S): old keys A (a leaf
// holds at most S - 7 keys: an 8-byte head and one byte per further key), the
// counts P by rank, and, with cap > 0, room for ccap = S - 7 + cap merged keys of 8
// bytes or twice as many offsets of 4.  The new codes take the place of A and P.
struct HeavyLayout {
  uint32_t p, c, ccap, total;
  __host__ __device__ HeavyLayout(uint32_t S, uint32_t cap) {
    const uint32_t maxA = S - 7;
    p = 8u * (maxA + 1);
    c = (p + 4u * (maxA + 1) + 15u) & ~15u;
    ccap = cap ? maxA + cap : 0u;
    total = c + 8u * ccap;
  }
};

// Old keys of a leaf of at most 1024 bytes as offsets from base, four bytes a thread:
// a code of at most five bytes carries its place in from the word before.
__device__ __forceinline__ uint32_t heavy_decode_narrow(const uint8_t* __restrict__ lp, uint32_t used,
                                                        uint32_t head_rel, uint32_t* A, uint32_t* wsum) {
  const uint32_t pos = 4u * threadIdx.x;
  uint32_t w = pos < used ? *reinterpret_cast<const uint32_t*>(lp + pos) : 0u;
  const uint32_t before = pos > 8 && pos < used ? *reinterpret_cast<const uint32_t*>(lp + pos - 4) : 0u;
  const uint32_t nvalid = pos < used ? min(4u, used - pos) : 0u;
  uint32_t valid = nvalid == 4 ? 0x80808080u : (1u << (8 * nvalid)) - 1u;
  uint32_t run = 0;
  if (pos < 8) {  // the head: one key, counted at byte 7
    w = 0x80808080u;
    valid = 0;
    if (pos == 0) run = head_rel;
  }
  const uint32_t stop = ~before & 0x80808080u;
  uint32_t sh = stop ? 7u * ((uint32_t)__clz((int)stop) >> 3) : 28u, k[4];
#pragma unroll
  for (int j = 0; j < 4; j++) {
    uint32_t c;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(c) : "v"(w), "i"(8 * j + 7));
    if (8 * j < 32 && (valid >> (8 * j)) & 0xffu) run += __builtin_amdgcn_ubfe(w, 8 * j, 7) << (sh & 31u);
    k[j] = run;
    sh = (sh + 7u) & c;
  }
  const uint32_t ends = (~w & valid & 0x80808080u) | (pos == 4 && used ? 0x80000000u : 0u);
  const uint32_t n = (uint32_t)__popc(ends);
  // both scans in one exchange
  const uint32_t wid = threadIdx.x / kWave, is = wave_incl_scan(run), in = wave_incl_scan(n);
  if (lane_id() == kWave - 1) {
    wsum[2 * wid] = is;
    wsum[2 * wid + 1] = in;
  }
  __syncthreads();
  uint32_t at = in - n, base = is - run, all = 0;
#pragma unroll
  for (uint32_t v = 0; v < kHeavyThreads / kWave; v++) {
    base += v < wid ? wsum[2 * v] : 0u;
    at += v < wid ? wsum[2 * v + 1] : 0u;
    all += wsum[2 * v + 1];
  }
#pragma unroll
  for (int j = 0; j < 4; j++)
    if (ends & (0x80u << (8 * j))) A[at++] = base + k[j];
  return all;
}

// One block merges one long insert slice into its leaf.  Each batch key is ranked
// among the old keys by binary search in LDS; an old key's output position is its
// index plus the number of new batch keys ranked at or below it (counted by rank in
// LDS, scanned together with the batch keys already present, 16 bits each), so the
// slice is only streamed.  The merged keys are built in LDS when they fit, else in
// the HBM staging buffer, then encoded in LDS where A and P were and copied to the
// leaf or the arena.  KT: 32-bit offsets from the segment's smallest possible key
// for segments that span less than 2^32, else the keys.  Four waves share a slice's
// LDS (29 KB at S = 1024).  36 000 slices of 540 keys: 2.23 ms with one wave per
// slice, 0.70 with four waves, 64-bit keys, one wave decoding and two searches per
// batch key, 0.50 now (half of that vector instructions; the rest waits at barriers).
template <typename KT>
__device__ __forceinline__ void heavy_slice(const MergeArgs& a, uint32_t s, uint64_t base, uint8_t* smem,
                                            const HeavyLayout& lay, uint32_t* wsum, uint64_t* shared,
                                            unsigned long long& delta, unsigned long long& alg) {
  constexpr bool kNarrow = sizeof(KT) == 4;
  const uint32_t S = a.S, tid = threadIdx.x;
  KT* A = reinterpret_cast<KT*>(smem);
  uint32_t* P = reinterpret_cast<uint32_t*>(smem + lay.p);
  const uint64_t leaf = a.seg_leaf[s];
  const uint32_t b = a.seg_begin[s];
  const uint32_t nb = a.seg_begin[s + 1] - b;
  uint8_t* lp = a.bytes + leaf * (uint64_t)S;
  const uint32_t used0 = a.used[leaf];
  const uint64_t* Bs = a.B + b;
  __syncthreads();  // the slice before is done with the LDS
  uint32_t nA;
  for (uint32_t i = tid; i <= S - 7; i += kHeavyThreads) P[i] = 0;
  if constexpr (kNarrow) {
    nA = heavy_decode_narrow(lp, used0, (uint32_t)(a.head[leaf] - base), A, wsum);
    __syncthreads();
  } else {
    if (tid < kWave) {
      const uint32_t n = wave_decode_leaf(lp, used0, [&](uint32_t i, uint64_t x, uint64_t) { A[i] = x; });
      if (tid == 0) shared[0] = n;
    }
    __syncthreads();
    nA = (uint32_t)shared[0];
  }
  // the first batch keys of a thread keep their ranks in registers
  constexpr uint32_t kKeep = 4;
  KT kept[kKeep];
  uint32_t rk[kKeep];  // rank, or ~0 when present or past the slice
  auto rank = [&](KT x, uint32_t& r) {
    r = lds_lower_bound<KT>(A, nA, x);
    return r < nA && A[r] == x;
  };
#pragma unroll
  for (uint32_t q = 0; q < kKeep; q++) {
    const uint32_t j = tid + q * kHeavyThreads;
    kept[q] = 0;
    rk[q] = ~0u;
    if (j < nb) {
      kept[q] = (KT)(Bs[j] - base);
      uint32_t r;
      const bool present = rank(kept[q], r);
      atomicAdd(&P[r], present ? 1u << 16 : 1u);
      if (!present) rk[q] = r;
    }
  }
  for (uint32_t j = tid + kKeep * kHeavyThreads; j < nb; j += kHeavyThreads) {
    uint32_t r;
    const bool present = rank((KT)(Bs[j] - base), r);
    atomicAdd(&P[r], present ? 1u << 16 : 1u);
  }
  __syncthreads();
  // P[i], scanned: new batch keys whose rank is below i, and (high half) batch keys
  // present among A[0, i)
  heavy_scan_inplace(P, nA + 1, wsum);
  // all batch keys are ranked at most nA: the last entry lacks those ranked nA, which
  // are new
  const uint32_t present = P[nA] >> 16;
  const uint32_t m = nA + nb - present;
  KT* stage = nullptr;
  if (m > lay.ccap * (kNarrow ? 2u : 1u)) {
    if (tid == 0) shared[1] = atomicAdd(&a.ctr->stage_cursor, (unsigned long long)m);
    __syncthreads();
    if (shared[1] + m > a.stage_cap) {
      if (tid == 0) atomicOr(&a.ctr->error, 2u);
      return;
    }
    stage = reinterpret_cast<KT*>(a.stage + shared[1]);
  }
  // C in LDS or in the staging buffer: two instances, so that each copy's
  // accesses have a known address space
  auto place_and_store = [&](auto C) {
#pragma unroll
    for (uint32_t q = 0; q < kKeep; q++)
      if (rk[q] != ~0u) C[rk[q] + (tid + q * kHeavyThreads) - (P[rk[q]] >> 16)] = kept[q];
    for (uint32_t j = tid + kKeep * kHeavyThreads; j < nb; j += kHeavyThreads) {
      const KT x = (KT)(Bs[j] - base);
      uint32_t r;
      if (!rank(x, r)) C[r + j - (P[r] >> 16)] = x;
    }
    // new batch keys before A[i]: those ranked at most i
    for (uint32_t i = tid; i < nA; i += kHeavyThreads) C[i + (P[i + 1] & 0xffffu)] = A[i];
    __threadfence_block();
    __syncthreads();  // A and P have been read
    const HeavyRun run = heavy_plan<KT>(C, m, false, (KT)0, wsum);
    const uint32_t T = run.total;
    uint64_t written = T;
    uint8_t* dst = lp;
    if (T > S) {
      const uint64_t off = arena_region(a, s);
      if (off + (((uint64_t)T + 15) & ~15ull) > a.arena_cap) {
        if (tid == 0) atomicOr(&a.ctr->error, 1u);
        return;
      }
      dst = a.arena + off;
      if (tid == 0) a.ovf[leaf] = off;
    }
    const uint32_t len = ((T > S ? T : max(used0, T)) + 15u) & ~15u;
    if (T <= S) written = len;
    if (len <= lay.c) {
      for (uint32_t o = 16u * tid; o < len; o += 16u * kHeavyThreads)
        *reinterpret_cast<uint4*>(smem + o) = make_uint4(0, 0, 0, 0);
      __syncthreads();
      heavy_encode<KT>(C, run, false, (KT)0, base, smem);
      __syncthreads();
      for (uint32_t o = 16u * tid; o < len; o += 16u * kHeavyThreads)
        *reinterpret_cast<uint4*>(dst + o) = *reinterpret_cast<const uint4*>(smem + o);
    } else {
      heavy_encode<KT>(C, run, false, (KT)0, base, dst);
    }
    if (tid == 0) {
      a.used[leaf] = T;
      a.head[leaf] = base + (uint64_t)C[0];
    }
    alg += used0 + written + 8ull * nb + 20;
    delta += nb - present;
  };
  if (stage)
    place_and_store(stage);
  else
    place_and_store(reinterpret_cast<KT*>(smem + lay.c));
}

// Merges the slices of the heavy list (the lane merge's longest), or with
// from_spill those of the spill list (the wave merge's long inserts); slices of
// more than kGiantSlice keys go to giant_list instead (giant_list NULL: there are
// none).  Up to S - 7 + cap merged keys stay in LDS; the launch's dynamic LDS is
// HeavyLayout(S, cap).total.  Every block writes its {keys added, algorithmic
// bytes} slot of a.part.
__global__ void __launch_bounds__(kHeavyThreads) k_merge_heavy(MergeArgs a, uint32_t cap, int from_spill,
                                                               uint32_t* __restrict__ giant_list) {
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ uint32_t wsum[2 * kHeavyThreads / kWave];
  __shared__ uint64_t shared[2];
  const HeavyLayout lay(a.S, cap);
  const uint32_t n = from_spill ? a.ctr->nspill : a.ctr->heavy;
  const uint32_t* list = from_spill ? a.spill_list : a.heavy_list;
  unsigned long long delta = 0, alg = 0;
  for (uint32_t h = blockIdx.x; h < n; h += gridDim.x) {
    const uint32_t s = list[h];
    if (giant_list && a.seg_begin[s + 1] - a.seg_begin[s] > kGiantSlice) {
      if (threadIdx.x == 0) giant_list[atomicAdd(&a.ctr->ngiant, 1u)] = s;
      continue;
    }
    const uint64_t leaf = a.seg_leaf[s], head = a.head[leaf], first = a.B[a.seg_begin[s]];
    const uint64_t base = a.used[leaf] && head < first ? head : first;
    const uint64_t above = leaf + 1 < a.L ? a.head[leaf + 1] : ~0ull;
    if (a.S <= kWaveMaxS && above - base <= 1ull << 32)
      heavy_slice<uint32_t>(a, s, base, smem, lay, wsum, shared, delta, alg);
    else
      heavy_slice<uint64_t>(a, s, 0, smem, lay, wsum, shared, delta, alg);
  }
  if (threadIdx.x == 0) {
    a.part[2 * blockIdx.x] = delta;
    a.part[2 * blockIdx.x + 1] = alg;
  }
}

// ---- giant slices: one block per piece of kGiantPiece batch keys -------------------
// A skewed batch can put most of its keys into one leaf (a Zipf batch of 1e6 keys
// into 1e8: 5.9 ms of its 7.6 ms insert and delete went to one wave merging one
// leaf).  Piece p of a slice owns the batch keys [c0, c1) and the old keys in
// between (from the first batch key of the piece up to that of the next; the
// first piece also those below, the last those above), so pieces merge
// independently: the only thing a piece needs of the one before is its last key,
// the larger of the old key and of the batch key just before it.  One pass counts
// the pieces' bytes, a scan places them, a second pass writes them to the leaf's
// arena region.  (More than kGiantSlice distinct keys never fit a leaf.)
struct GiantArgs {
  const uint32_t* list;       // n giant segments
  uint32_t n;
  uint32_t* first;            // n + 1: each slice's first piece
  uint64_t* bytes;            // per piece
  const uint64_t* scan;       // their exclusive scan
  uint64_t* prev;             // per piece: the key before it (0: none)
  uint32_t* keys;             // per piece: its keys
};

__global__ void __launch_bounds__(kHeavyThreads) k_giant_plan(MergeArgs a, GiantArgs g) {
  __shared__ uint32_t wsum[kHeavyThreads / kWave];
  uint32_t run = 0;
  for (uint32_t base = 0; base < g.n; base += kHeavyThreads) {
    const uint32_t i = base + threadIdx.x;
    uint32_t v = 0, total;
    if (i < g.n) {
      const uint32_t s = g.list[i];
      v = (a.seg_begin[s + 1] - a.seg_begin[s] + kGiantPiece - 1) / kGiantPiece;
    }
    const uint32_t ex = heavy_scan(v, wsum, &total);
    if (i < g.n) g.first[i] = run + ex;
    run += total;
  }
  if (threadIdx.x == 0) g.first[g.n] = run;
}

__host__ __device__ inline uint32_t giant_smem(uint32_t S) {  // old keys, rank histogram, merged keys
  return 8u * (S - 6) + 4u * ((S + 3u) & ~3u) + 8u * (S - 7 + kGiantPiece);
}

template <bool kWrite>
__global__ void __launch_bounds__(kHeavyThreads) k_giant_merge(MergeArgs a, GiantArgs g, uint64_t npieces_bound) {
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ uint32_t wsum[kHeavyThreads / kWave];
  __shared__ uint32_t sh_n;
  const uint32_t S = a.S, tid = threadIdx.x;
  uint64_t* A = reinterpret_cast<uint64_t*>(smem);
  uint32_t* N = reinterpret_cast<uint32_t*>(smem + 8u * (S - 6));
  uint64_t* M = reinterpret_cast<uint64_t*>(smem + 8u * (S - 6) + 4u * ((S + 3u) & ~3u));
  const uint32_t np = g.first[g.n];
  for (uint32_t p = blockIdx.x; p < npieces_bound; p += gridDim.x) {
    if (p >= np) {
      if (!kWrite && tid == 0) {  // the scans cover the bound
        g.bytes[p] = 0;
        g.keys[p] = 0;
      }
      continue;
    }
    uint32_t lo = 0, hi = g.n;  // the slice: the last with first[] <= p
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (g.first[mid] <= p)
        lo = mid;
      else
        hi = mid;
    }
    const uint32_t s = g.list[lo];
    const uint64_t leaf = a.seg_leaf[s];
    const uint32_t b = a.seg_begin[s], nb = a.seg_begin[s + 1] - b;
    const uint32_t c0 = (p - g.first[lo]) * kGiantPiece, c1 = min(nb, c0 + kGiantPiece);
    const uint64_t* Bs = a.B + b;
    const uint32_t used0 = a.seg_desc[s].z;  // the size before the batch (the first piece overwrites used[])
    __syncthreads();
    if (tid < kWave) {
      const uint32_t n = wave_decode_leaf(a.bytes + leaf * (uint64_t)S, used0,
                                          [&](uint32_t i, uint64_t x, uint64_t) { A[i] = x; });
      if (tid == 0) sh_n = n;
    }
    for (uint32_t i = tid; i <= S - 7; i += kHeavyThreads) N[i] = 0;
    __syncthreads();
    const uint32_t nA = sh_n;
    const uint32_t r0 = c0 ? lds_lower_bound(A, nA, Bs[c0]) : 0u;
    const uint32_t r1 = c1 < nb ? lds_lower_bound(A, nA, Bs[c1]) : nA;
    constexpr uint32_t kPer = kGiantPiece / kHeavyThreads;
    uint64_t x[kPer];
    uint32_t rk[kPer], fresh = 0;
#pragma unroll
    for (uint32_t q = 0; q < kPer; q++) {
      const uint32_t j = c0 + tid * kPer + q;
      rk[q] = ~0u;
      x[q] = 0;
      if (j < c1) {
        x[q] = Bs[j];
        const uint32_t r = lds_lower_bound(A, nA, x[q]);
        if (!(r < nA && A[r] == x[q])) {
          rk[q] = r - r0;
          fresh++;
          atomicAdd(&N[r - r0], 1u);
        }
      }
    }
    uint32_t nnew;
    uint32_t pos = heavy_scan(fresh, wsum, &nnew);
    heavy_scan_inplace(N, r1 - r0 + 1, wsum);
#pragma unroll
    for (uint32_t q = 0; q < kPer; q++)
      if (rk[q] != ~0u) M[rk[q] + pos++] = x[q];
    for (uint32_t i = r0 + tid; i < r1; i += kHeavyThreads)
      M[i - r0 + N[i - r0 + 1]] = A[i];  // new keys before it: those ranked at most i
    __syncthreads();
    const uint32_t m = r1 - r0 + nnew;
    const bool has_pred = c0 > 0;
    uint64_t pred = has_pred ? Bs[c0 - 1] : 0;
    if (has_pred && r0 && A[r0 - 1] > pred) pred = A[r0 - 1];
    const HeavyRun run = heavy_plan<uint64_t>(M, m, has_pred, pred, wsum);
    if (!kWrite) {
      if (tid == 0) {
        g.bytes[p] = run.total;
        g.prev[p] = pred;
        g.keys[p] = m;
      }
    } else {
      const uint64_t start = g.scan[g.first[lo]], off = g.scan[p] - start;
      const uint64_t U = g.scan[g.first[lo + 1]] - start, region = arena_region(a, s);
      const bool fits = region + ((U + 15) & ~15ull) <= a.arena_cap;
      if (fits)
        heavy_encode<uint64_t>(M, run, has_pred, pred, 0, a.arena + region + off);
      else if (tid == 0)
        atomicOr(&a.ctr->error, 1u);
      if (tid == 0) {
        atomicAdd(&a.ctr->delta, (unsigned long long)nnew);
        atomicAdd(&a.ctr->alg_bytes_h, (unsigned long long)run.total + 8ull * (c1 - c0) + (c0 ? 0u : used0 + 20u));
        if (c0 == 0) {
          a.used[leaf] = (uint32_t)U;
          a.head[leaf] = M[0];
          a.ovf[leaf] = region;
        }
      }
    }
  }
}

// Staging of the giant leaves of a redistribution, a wave per piece (k_win_pack
// leaves them out: one wave decoding a megabyte of codes takes 400 us).  key_scan:
// exclusive scan of the pieces' keys.
__global__ void __launch_bounds__(kWave) k_giant_pack(WinArgs wa, SrcLeaves src, MergeArgs a, GiantArgs g,
                                                      const uint32_t* __restrict__ key_scan,
                                                      const uint64_t* __restrict__ koff,
                                                      uint64_t* __restrict__ stage, uint32_t* __restrict__ win_id,
                                                      uint8_t* __restrict__ ccost) {
  const uint32_t np = g.first[g.n];
  for (uint32_t p = blockIdx.x; p < np; p += gridDim.x) {
    const uint32_t gi = (uint32_t)(upper_bound_u32(g.first, g.n + 1, p) - 1);
    const uint64_t leaf = a.seg_leaf[g.list[gi]];
    const uint32_t w = (uint32_t)upper_bound_u64(wa.src_begin, wa.W, leaf) - 1u;  // windows are in leaf order
    if (w == ~0u || leaf - wa.src_begin[w] >= wa.src_flat[w + 1] - wa.src_flat[w]) continue;
    const uint64_t at = koff[wa.src_flat[w] + (leaf - wa.src_begin[w])] + (key_scan[p] - key_scan[g.first[gi]]);
    const bool head = p == g.first[gi];
    const uint64_t start = g.scan[p] - g.scan[g.first[gi]];
    const uint64_t bytes = g.scan[p + 1] - g.scan[p];
    const uint8_t* base = src.ptr(leaf, src.used[leaf]);
    // 16-byte chunks of the leaf from the one the piece starts in: what lies
    // before it decodes as nothing
    wave_decode_piece(base, start, start + bytes, head, g.prev[p], [&](uint32_t i, uint64_t x, uint64_t d) {
      stage[at + i] = x;
      win_id[at + i] = w;
      ccost[at + i] = head && i == 0 ? (uint8_t)8 : (uint8_t)vlen(d);
    });
  }
}

}  // namespace cpma_dev
