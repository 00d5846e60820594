// PageRank on the CPMA's edge keys (Section "Evaluation on graph workloads"), the
// edges laid out once per call so that an iteration's gathers and sums run in LDS.
//
// An iteration adds contrib[v] over every edge (u, v) into u.  Read in key order
// (by source), every edge gathers 4 bytes of the contribution vector and moves a
// 128-byte line to do so: 2.5e8 requests past L1 for 2.7e8 edges, 4.3 ms at 2^24
// vertices.  That is what the L2s deliver for such requests: binning the edges so
// that nearly all of them hit L2 (one 4 MB share of the vector per XCD) still took
// 3.1 ms.  So the edges are binned two ways at once, by (part, bin): a part is a
// range of destinations whose contributions fit LDS, a bin a range of sources whose
// sums do.  The edges of a part lie together, in it those of a bin, each as its
// source within the bin and its destination within the part (4 bytes).  An
// iteration is two streams over them:
//   gather: a block loads a part's contributions to LDS and writes every edge's;
//   add: a block adds its bin's values, one run per part, to sums in LDS (64
//        bits), and finishes the bin's vertices.
// 16 bytes of HBM per edge and iteration, all in order.
#pragma once
#include "fgraph.hpp"
#include "pg_segments.hpp"
#include "update.hpp"

namespace cpma_dev {

constexpr uint32_t kPgThreads = 1024;
constexpr uint32_t kPgWaves = kPgThreads / kWave;

struct PgArgs {
  uint32_t nv;
  uint32_t pbits;   // destinations of a part: 2^pbits, at most 2^15
  uint32_t bbits;   // sources of a bin: at most 2^bbits
  uint32_t P, B;    // parts, bins
  uint32_t cuts;    // bin limits taken from the leaves (the other B - cuts: every 2^bbits)
  uint32_t* limit;  // first source of every bin, then nv
  uint32_t* leaf;   // the leaf that may hold its first key
  uint32_t seg;     // edges of a gather segment, at most
  uint32_t* cnt;         // [bin][part] edges
  uint32_t* pos;         // [part][bin] edges, then (P B + 1) the first edge
  uint2* run;            // [bin][part] first edge and end (read by bin: [part][bin] would take a line for each)
  uint32_t* nseg;        // segments of every part
  const uint32_t* segoff;  // their exclusive scan (P + 1)
  uint32_t* segpart;     // the part of every segment
  uint32_t* E;           // edges: source within the bin << 16 | destination within the part
  float* val;            // their contributions
  uint32_t* deg;
  float* contrib;
};

// The bins' first sources: the sources of every L / cuts-th leaf's head merged with
// the multiples of 2^bbits (equal ones leave empty bins).
__global__ void __launch_bounds__(256) k_pg_limits(FgArgs g, PgArgs a) {
  auto cut = [&](uint32_t i) { return min(src_of(g.head[(uint64_t)i * g.L / a.cuts]), g.nv); };
  for (uint32_t t = blockIdx.x * 256 + threadIdx.x; t <= a.B; t += gridDim.x * 256) {
    uint32_t u = g.nv, at = a.B;
    if (t < a.cuts) {
      u = cut(t);
      at = t + min(a.B - a.cuts, (uint32_t)(((uint64_t)u + (1u << a.bbits) - 1) >> a.bbits));  // multiples below u
    } else if (t < a.B) {
      u = (t - a.cuts) << a.bbits;
      uint32_t lo = 0, hi = a.cuts;  // cuts at or below u
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (cut(mid) <= u)
          lo = mid + 1;
        else
          hi = mid;
      }
      at = t - a.cuts + lo;
    }
    a.limit[at] = u;
    a.leaf[at] = (uint32_t)locate_leaf(g.head, g.L, (uint64_t)u << 32);
  }
}

// A block per bin: its edges by part, its vertices' degrees (edges to vertices that
// exist) and the first contributions, of uniform ranks.  LDS: P + 2^bbits counters.
__global__ void __launch_bounds__(kPgThreads) k_pg_count(FgArgs g, PgArgs a, float rank0) {
  extern __shared__ uint32_t pg_lds[];
  uint32_t* hist = pg_lds;
  uint32_t* deg = pg_lds + a.P;
  const uint32_t bin = 1u << a.bbits, wid = threadIdx.x / kWave;
  for (uint32_t b = blockIdx.x; b < a.B; b += gridDim.x) {
    const uint32_t u0 = a.limit[b], u1 = a.limit[b + 1];
    for (uint32_t i = threadIdx.x; i < a.P + bin; i += kPgThreads) pg_lds[i] = 0;
    __syncthreads();
    for (uint64_t leaf = a.leaf[b] + wid; u0 < u1 && leaf <= a.leaf[b + 1]; leaf += kPgWaves) {
      uint64_t kk[16];
      const uint32_t tm = wave_leaf_keys(g.bytes + leaf * (uint64_t)g.S, g.used[leaf], kk);
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const uint32_t s = src_of(kk[i]), d = dst_of(kk[i]);
        if (((tm >> i) & 1u) && s >= u0 && s < u1 && d < g.nv) {
          atomicAdd(&hist[d >> a.pbits], 1u);
          atomicAdd(&deg[s - u0], 1u);
        }
      }
    }
    __syncthreads();
    for (uint32_t p = threadIdx.x; p < a.P; p += kPgThreads) a.cnt[(uint64_t)b * a.P + p] = hist[p];
    for (uint32_t i = threadIdx.x; i < u1 - u0; i += kPgThreads) {
      const uint32_t d = deg[i];
      a.deg[u0 + i] = d;
      a.contrib[u0 + i] = d ? rank0 / (float)d : 0.f;
    }
    __syncthreads();
  }
}

// The counts to [part][bin] order (kBack: the scanned ones back, as runs), 64 x 64 at
// a time through LDS.
template <bool kBack>
__global__ void __launch_bounds__(256) k_pg_transpose(PgArgs a, uint32_t* __restrict__ out) {
  __shared__ uint32_t t[64][65];
  const uint32_t b0 = blockIdx.x * 64, p0 = blockIdx.y * 64;
  __shared__ uint32_t edge[64];  // kBack: the bin after the tile
  for (uint32_t i = threadIdx.x; i < 64 * 64; i += 256) {
    const uint32_t y = i >> 6, x = i & 63u;
    if (kBack) {
      if (p0 + y < a.P && b0 + x <= a.B) t[y][x] = a.pos[(uint64_t)(p0 + y) * a.B + b0 + x];
      if (x == 63 && p0 + y < a.P && b0 + 64 <= a.B) edge[y] = a.pos[(uint64_t)(p0 + y) * a.B + b0 + 64];
    } else {
      if (b0 + y < a.B && p0 + x < a.P) t[y][x] = a.cnt[(uint64_t)(b0 + y) * a.P + p0 + x];
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < 64 * 64; i += 256) {
    const uint32_t y = i >> 6, x = i & 63u;
    if (kBack) {
      if (b0 + y < a.B && p0 + x < a.P)
        a.run[(uint64_t)(b0 + y) * a.P + p0 + x] = make_uint2(t[x][y], y < 63 ? t[x][y + 1] : edge[x]);
    } else {
      if (p0 + y < a.P && b0 + x < a.B) out[(uint64_t)(p0 + y) * a.B + b0 + x] = t[x][y];
    }
  }
}

// A block per bin: its edges to their runs (any order within a run).  base: the
// scanned counts.  LDS: a cursor per part.
__global__ void __launch_bounds__(kPgThreads) k_pg_scatter(FgArgs g, PgArgs a) {
  extern __shared__ uint32_t pg_lds[];
  const uint32_t part = 1u << a.pbits, wid = threadIdx.x / kWave;
  for (uint32_t b = blockIdx.x; b < a.B; b += gridDim.x) {
    const uint32_t u0 = a.limit[b], u1 = a.limit[b + 1];
    for (uint32_t p = threadIdx.x; p < a.P; p += kPgThreads) pg_lds[p] = a.run[(uint64_t)b * a.P + p].x;
    __syncthreads();
    for (uint64_t leaf = a.leaf[b] + wid; u0 < u1 && leaf <= a.leaf[b + 1]; leaf += kPgWaves) {
      uint64_t kk[16];
      const uint32_t tm = wave_leaf_keys(g.bytes + leaf * (uint64_t)g.S, g.used[leaf], kk);
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const uint32_t s = src_of(kk[i]), d = dst_of(kk[i]);
        if (((tm >> i) & 1u) && s >= u0 && s < u1 && d < g.nv) {
          const uint32_t at = atomicAdd(&pg_lds[d >> a.pbits], 1u);
          a.E[at] = ((s - u0) << 16) | (d & (part - 1u));
        }
      }
    }
    __syncthreads();
  }
}

// Gather segments of every part, and each segment's part.
__global__ void k_pg_segments(PgArgs a) {
  for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < a.P; p += gridDim.x * blockDim.x)
    a.nseg[p] = pg_segment_count(a.pos[(uint64_t)p * a.B], a.pos[(uint64_t)(p + 1) * a.B], a.seg);
}
__global__ void k_pg_segparts(PgArgs a) {
  for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < a.P; p += gridDim.x * blockDim.x)
    for (uint32_t s = a.segoff[p]; s < a.segoff[p + 1]; s++) a.segpart[s] = p;
}

// val[e] = contrib[destination of e], a segment per block.  LDS: the part's contributions.
__global__ void __launch_bounds__(kPgThreads) k_pg_gather(PgArgs a) {
  extern __shared__ uint32_t pg_lds[];
  float* c = reinterpret_cast<float*>(pg_lds);
  const uint32_t part = 1u << a.pbits, nseg = a.segoff[a.P];
  for (uint32_t s = blockIdx.x; s < nseg; s += gridDim.x) {
    const uint32_t p = a.segpart[s];
    const uint32_t b0 = a.pos[(uint64_t)p * a.B], b1 = a.pos[(uint64_t)(p + 1) * a.B];
    const PgSegment sg = pg_segment(b0, b1, a.seg, s - a.segoff[p]);
    const uint32_t e0 = sg.e0, e1 = sg.e1;
    const uint32_t v0 = p << a.pbits;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < part && v0 + i < a.nv; i += kPgThreads) c[i] = a.contrib[v0 + i];
    __syncthreads();
    // whole groups of four edges, and the ragged ends
    const uint32_t q0 = min(e1, (e0 + 3u) & ~3u), q1 = max(q0, e1 & ~3u);
    if (threadIdx.x < q0 - e0) a.val[e0 + threadIdx.x] = c[a.E[e0 + threadIdx.x] & 0xffffu];
    if (threadIdx.x < e1 - q1) a.val[q1 + threadIdx.x] = c[a.E[q1 + threadIdx.x] & 0xffffu];
    const uint4* E4 = reinterpret_cast<const uint4*>(a.E);
    float4* V4 = reinterpret_cast<float4*>(a.val);
#pragma unroll 4
    for (uint32_t i = q0 / 4 + threadIdx.x; i < q1 / 4; i += kPgThreads) {
      const uint4 e = E4[i];
      V4[i] = make_float4(c[e.x & 0xffffu], c[e.y & 0xffffu], c[e.z & 0xffffu], c[e.w & 0xffffu]);
    }
  }
}

// A block per bin: its vertices' sums over the bin's runs, then the
// ranks p = base + damping * sum and (more) the contributions of the next iteration.
// LDS: 2^bbits sums.
__global__ void __launch_bounds__(kPgThreads) k_pg_add(PgArgs a, float base, float damping, float* __restrict__ p,
                                                       int more) {
  extern __shared__ uint32_t pg_lds[];
  double* acc = reinterpret_cast<double*>(pg_lds);
  const uint32_t wid = threadIdx.x / kWave, lane = (uint32_t)lane_id();
  for (uint32_t b = blockIdx.x; b < a.B; b += gridDim.x) {
    const uint32_t u0 = a.limit[b], u1 = a.limit[b + 1];
    if (u0 == u1) continue;
    for (uint32_t i = threadIdx.x; i < u1 - u0; i += kPgThreads) acc[i] = 0.0;
    __syncthreads();
    auto add = [&](uint32_t e, float v) {
      __hip_atomic_fetch_add(&acc[e >> 16], (double)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    for (uint32_t p0 = 0; p0 < a.P; p0 += kPgWaves * kWave) {
      // the next 64 runs of this wave: one of every 16 parts, another of the 16 each
      // time, so that parts with more edges (skewed graphs) spread over the waves
      uint2 r = make_uint2(0, 0);
      const uint32_t q = p0 + kPgWaves * lane + ((wid ^ lane ^ (lane >> 4)) & (kPgWaves - 1u));
      if (q < a.P) r = a.run[(uint64_t)b * a.P + q];
      uint64_t some = __ballot(r.y > r.x);
      // up to 256 edges are in flight while the 256 before them are added, the next
      // run's first ones among them
      uint32_t e[4], at = 0, end = 0;
      float v[4];
      auto fetch = [&]() {
        if (at >= end && some) {
          const int l = __ffsll((unsigned long long)some) - 1;
          some &= some - 1;
          at = (uint32_t)__builtin_amdgcn_readlane((int)r.x, l);
          end = (uint32_t)__builtin_amdgcn_readlane((int)r.y, l);
        }
#pragma unroll
        for (uint32_t h = 0; h < 4; h++) {
          const uint32_t i = at + h * kWave + lane;
          e[h] = ~0u;
          v[h] = 0.f;
          if (i < end) {
            e[h] = a.E[i];
            v[h] = a.val[i];
          }
        }
      };
      fetch();
      while (at < end) {
        uint32_t ce[4];
        float cv[4];
#pragma unroll
        for (int h = 0; h < 4; h++) {
          ce[h] = e[h];
          cv[h] = v[h];
        }
        at += 4 * kWave;
        fetch();
#pragma unroll
        for (int h = 0; h < 4; h++)
          if (ce[h] != ~0u) add(ce[h], cv[h]);  // a bin has fewer than 2^16 sources
      }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < u1 - u0; i += kPgThreads) {
      const float r = base + damping * (float)acc[i];
      p[u0 + i] = r;
      if (more) {
        const uint32_t d = a.deg[u0 + i];
        a.contrib[u0 + i] = d ? r / (float)d : 0.f;
      }
    }
    __syncthreads();
  }
}

}  // namespace cpma_dev
