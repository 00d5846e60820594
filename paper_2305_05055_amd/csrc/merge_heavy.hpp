// Merges of long insert slices into their leaves (the batch-merge phase of Section
// "Parallel Batch Updates in a PMA" for slices too long for the one-key-per-lane
// wave merge or for one lane): one block per slice, and for the longest slices
// one block per piece of a slice.
#pragma once
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
__device__ __forceinline__ uint32_t heavy_cost(const uint64_t* C, uint32_t i, bool has_pred, uint64_t pred) {
  return i ? vlen(C[i] - C[i - 1]) : (has_pred ? vlen(C[0] - pred) : 8u);
}
__device__ __forceinline__ HeavyRun heavy_plan(const uint64_t* C, uint32_t m, bool has_pred, uint64_t pred,
                                               uint32_t* wsum) {
  HeavyRun r;
  const uint32_t per = (m + kHeavyThreads - 1) / kHeavyThreads;
  r.i0 = min(m, per * threadIdx.x);
  r.i1 = min(m, r.i0 + per);
  uint32_t s = 0;
  for (uint32_t i = r.i0; i < r.i1; i++) s += heavy_cost(C, i, has_pred, pred);
  r.off = heavy_scan(s, wsum, &r.total);
  return r;
}
template <typename P>
__device__ __forceinline__ void heavy_encode(const uint64_t* C, const HeavyRun& r, bool has_pred, uint64_t pred,
                                             P dst) {
  auto p = dst + r.off;
  for (uint32_t i = r.i0; i < r.i1; i++) {
    if (i == 0 && !has_pred) {
      put_le64(p, C[0]);
      p += 8;
    } else {
      p += vput(p, C[i] - (i ? C[i - 1] : pred));
    }
  }
}

// LDS of k_merge_heavy for leaf size S and merged-key room cap beyond a full
// leaf (byte offsets, each 16-byte aligned for even S): old keys A (a leaf
// holds at most S - 7 keys: an 8-byte head and one byte per further key),
// their presence flags F, the histogram N of the new batch keys' ranks, the
// encode buffer and, with cap > 0, ccap = S - 7 + cap merged keys.
struct HeavyLayout {
  uint32_t f, n, buf, c, ccap, total;
  __host__ __device__ HeavyLayout(uint32_t S, uint32_t cap) {
    const uint32_t maxA = S - 7;
    f = 8u * (maxA + 1);
    n = f + 4u * ((maxA + 4) & ~3u);
    buf = n + 4u * ((maxA + 4) & ~3u);
    c = buf + ((S + 15u) & ~15u);
    ccap = cap ? maxA + cap : 0u;
    total = c + 8u * ccap;
  }
};

// One block merges one long insert slice into its leaf.  Each batch key is ranked
// among the old keys by binary search in LDS; an old key's output position is its
// index plus the number of new batch keys ranked at or below it (an LDS histogram
// of those ranks, scanned), so the slice is only streamed, twice.  The merged keys
// are built in LDS when at most ccap of them result, else in the HBM staging
// buffer, then encoded in place or into the arena.  Four waves share a slice's
// LDS (33 KB at S = 1024): with one wave per slice and 41 KB three waves fitted a
// CU, and 36 000 slices of 540 keys took 2.23 ms.
__device__ __forceinline__ void heavy_slice(const MergeArgs& a, uint32_t s, uint8_t* smem, const HeavyLayout& lay,
                                            uint32_t* wsum, uint64_t* shared, unsigned long long& delta,
                                            unsigned long long& alg) {
  const uint32_t S = a.S, tid = threadIdx.x;
  uint64_t* A = reinterpret_cast<uint64_t*>(smem);
  uint32_t* F = reinterpret_cast<uint32_t*>(smem + lay.f);
  uint32_t* N = reinterpret_cast<uint32_t*>(smem + lay.n);
  uint8_t* buf = smem + lay.buf;
  const uint64_t leaf = a.seg_leaf[s];
  const uint32_t b = a.seg_begin[s];
  const uint32_t nb = a.seg_begin[s + 1] - b;
  uint8_t* lp = a.bytes + leaf * (uint64_t)S;
  const uint32_t used0 = a.used[leaf];
  const uint64_t* Bs = a.B + b;
  __syncthreads();  // the slice before is done with the LDS
  if (tid < kWave) {
    const uint32_t n = wave_decode_leaf(lp, used0, [&](uint32_t i, uint64_t x, uint64_t) { A[i] = x; });
    if (tid == 0) shared[0] = n;
  }
  for (uint32_t i = tid; i <= S - 7; i += kHeavyThreads) {
    F[i] = 0;
    N[i] = 0;
  }
  __syncthreads();
  const uint32_t nA = (uint32_t)shared[0];
  for (uint32_t j = tid; j < nb; j += kHeavyThreads) {
    const uint64_t x = Bs[j];
    const uint32_t r = lds_lower_bound(A, nA, x);
    if (r < nA && A[r] == x)
      F[r] = 1;
    else
      atomicAdd(&N[r], 1u);
  }
  __syncthreads();
  // exclusive scans: F[i] = batch keys already present among A[0, i),
  // N[i] = new batch keys whose rank among the old keys is below i
  heavy_scan_inplace(F, nA + 1, wsum);
  heavy_scan_inplace(N, nA + 1, wsum);
  const uint32_t present = F[nA];
  const uint32_t m = nA + nb - present;
  uint64_t* stage = nullptr;
  if (m > lay.ccap) {
    if (tid == 0) shared[1] = atomicAdd(&a.ctr->stage_cursor, (unsigned long long)m);
    __syncthreads();
    if (shared[1] + m > a.stage_cap) {
      if (tid == 0) atomicOr(&a.ctr->error, 2u);
      return;
    }
    stage = a.stage + shared[1];
  }
  // C in LDS or in the staging buffer: two instances, so that each copy's
  // accesses have a known address space
  auto place_and_store = [&](auto C) {
    for (uint32_t j = tid; j < nb; j += kHeavyThreads) {
      const uint64_t x = Bs[j];
      const uint32_t r = lds_lower_bound(A, nA, x);
      if (!(r < nA && A[r] == x)) C[r + j - F[r]] = x;
    }
    // new batch keys before A[i]: those ranked at most i
    for (uint32_t i = tid; i < nA; i += kHeavyThreads) C[i + N[i + 1]] = A[i];
    __threadfence_block();
    __syncthreads();
    const HeavyRun run = heavy_plan(C, m, false, 0, wsum);
    const uint32_t T = run.total;
    uint64_t written;
    if (T <= S) {
      const uint32_t len = (max(used0, T) + 15u) & ~15u;
      for (uint32_t o = 16u * tid; o < len; o += 16u * kHeavyThreads)
        *reinterpret_cast<uint4*>(buf + o) = make_uint4(0, 0, 0, 0);
      __syncthreads();
      heavy_encode(C, run, false, 0, buf);
      __syncthreads();
      for (uint32_t o = 16u * tid; o < len; o += 16u * kHeavyThreads)
        *reinterpret_cast<uint4*>(lp + o) = *reinterpret_cast<const uint4*>(buf + o);
      written = len;
    } else {
      const uint64_t off = arena_region(a, s);
      if (off + (((uint64_t)T + 15) & ~15ull) > a.arena_cap) {
        if (tid == 0) atomicOr(&a.ctr->error, 1u);
        return;
      }
      heavy_encode(C, run, false, 0, a.arena + off);
      if (tid == 0) a.ovf[leaf] = off;
      written = T;
    }
    if (tid == 0) {
      a.used[leaf] = T;
      a.head[leaf] = C[0];
    }
    alg += used0 + written + 8ull * nb + 20;
    delta += nb - present;
  };
  if (stage)
    place_and_store(stage);
  else
    place_and_store(reinterpret_cast<uint64_t*>(smem + lay.c));
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
  __shared__ uint32_t wsum[kHeavyThreads / kWave];
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
    heavy_slice(a, s, smem, lay, wsum, shared, delta, alg);
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
    const HeavyRun run = heavy_plan(M, m, has_pred, pred, wsum);
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
        heavy_encode(M, run, has_pred, pred, a.arena + region + off);
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
