// F-Graph on the CPMA (Section "Evaluation on graph workloads"): one CPMA holds
// every edge (u, v) of a graph as the key u<<32 | v, so a vertex's neighbours are
// the keys of [u<<32, (u+1)<<32) and a pass over all leaves visits every edge
// grouped by source.  Delta coding elides the source except at leaf heads and
// at each vertex's first edge.
//
// The kernels below are full passes: one wave decodes one leaf (keys land in lane
// registers), gathers the per-neighbour values for all of its keys at once, then
// each lane folds its keys into runs of equal source and flushes a run with one
// atomic.  PageRank (a fixed number of iterations) runs in pull form, which on
// a symmetric edge set (an undirected graph, the case F-Graph supports) equals
// pushing p(u)/deg(u) along every edge.  BFS is level synchronous and
// direction optimising: each level passes over the leaves holding the current
// level's vertices (top-down) or the unvisited ones (bottom-up).
#pragma once
#include "leaf.hpp"

namespace cpma_dev {

struct FgArgs {
  const uint8_t* bytes;
  const uint32_t* used;
  const uint64_t* head;
  uint64_t L;
  uint32_t S;   // at most 1024: one 16-byte chunk per lane
  uint32_t nv;  // vertex ids are < nv; keys with a larger id are ignored
};

// Keys of one leaf in the lane's registers: kk[i] is valid where bit i of the
// result is set (a code or the head ends at byte i of the lane's 16 bytes).
//
// A key is the head plus the payload of every code byte before it, each byte's
// 7 bits shifted by 7 times its place in its code, so a running sum of shifted
// payloads over the bytes, read at a code's last byte, is that key's offset; the
// shift a code carries in is 7 times the lane before's run of trailing
// continuation bytes, and one wave scan of the lanes' totals gives every lane its
// start.
__device__ __forceinline__ uint32_t wave_leaf_keys(uint4 w, uint32_t used, uint64_t (&kk)[16]) {
  const int lane = lane_id();
  const uint32_t pos0 = 16u * lane;
  const uint32_t nvalid = pos0 < used ? min(16u, used - pos0) : 0u;
  uint32_t vm = nvalid >= 16u ? 0xffffu : ((1u << nvalid) - 1u);
  uint64_t lead = 0;  // the head, in lane 0
  if (lane == 0) {
    vm &= 0xff00u;  // the head is not a code
    if (used >= 8u) lead = ((uint64_t)w.y << 32) | w.x;
    w.x = 0;
    w.y = 0;
  }
  uint32_t words[4] = {w.x, w.y, w.z, w.w};
  if (nvalid < 16u) {  // values may lie past `used`
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int32_t v = (int32_t)nvalid - 4 * k;
      words[k] &= v >= 4 ? 0xffffffffu : (v <= 0 ? 0u : ((1u << (8 * v)) - 1u));
    }
  }
  const uint32_t msb = msb_byte(words[0], words[1]) | msb_byte(words[2], words[3]) << 8;
  const uint32_t cm = vm & msb;  // continuation bytes
  uint32_t sh = 7u * dpp_prev32((uint32_t)__clz((int)~(cm << 16)));
  uint64_t run = lead;
#pragma unroll
  for (int j = 0; j < 16; j++) {
    const uint32_t x = words[j >> 2];
    uint32_t c;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(c) : "v"(x), "i"(8 * (j & 3) + 7));
    run += (uint64_t)__builtin_amdgcn_ubfe(x, 8 * (j & 3), 7) << (sh & 63u);
    kk[j] = run;
    sh = (sh + 7u) & c;
  }
  const uint64_t ex = wave_incl_scan(run) - run;
#pragma unroll
  for (int j = 0; j < 16; j++) kk[j] += ex;
  return (vm & ~msb) | (lane == 0 && used >= 8u ? 1u << 7 : 0u);
}

__device__ __forceinline__ uint4 wave_leaf_bytes(const uint8_t* __restrict__ src, uint32_t used) {
  const uint32_t pos0 = 16u * lane_id();
  return pos0 < used ? *reinterpret_cast<const uint4*>(src + pos0) : make_uint4(0, 0, 0, 0);
}

__device__ __forceinline__ uint32_t wave_leaf_keys(const uint8_t* __restrict__ src, uint32_t used,
                                                   uint64_t (&kk)[16]) {
  return wave_leaf_keys(wave_leaf_bytes(src, used), used, kk);
}

__device__ __forceinline__ uint32_t src_of(uint64_t k) { return (uint32_t)(k >> 32); }
__device__ __forceinline__ uint32_t dst_of(uint64_t k) { return (uint32_t)k; }

// The leaf's first source if every key of the leaf has it (a high-degree
// vertex whose edges fill whole leaves), else UINT32_MAX.  Such leaves reduce
// across the wave first: per-lane atomics would all hit that one vertex.
__device__ __forceinline__ uint32_t fg_single_source(const FgArgs& g, uint64_t leaf, const uint64_t (&kk)[16],
                                                    uint32_t tm) {
  if (!__ballot(tm != 0)) return 0xffffffffu;  // no keys
  const uint32_t first = src_of(g.head[leaf]);  // the head is the leaf's first key
  bool other = false;
#pragma unroll
  for (int i = 0; i < 16; i++) other |= (tm & (1u << i)) && src_of(kk[i]) != first;
  return __ballot(other) ? 0xffffffffu : first;
}

template <typename T>
__device__ __forceinline__ T wave_sum_float(T x) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

// deg[u] += number of edges with source u.
__global__ void __launch_bounds__(256) k_fg_degree(FgArgs g, uint32_t* __restrict__ deg) {
  const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / kWave);
  for (uint64_t leaf = (uint64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; leaf < g.L;
       leaf += waves) {
    uint64_t kk[16];
    const uint32_t tm = wave_leaf_keys(g.bytes + leaf * (uint64_t)g.S, g.used[leaf], kk);
    const uint32_t one = fg_single_source(g, leaf, kk, tm);
    if (one != 0xffffffffu) {
      uint32_t c = 0;
#pragma unroll
      for (int i = 0; i < 16; i++) c += ((tm & (1u << i)) && dst_of(kk[i]) < g.nv) ? 1u : 0u;
      c = wave_sum(c);
      if (lane_id() == 0 && one < g.nv && c) atomicAdd(&deg[one], c);
      continue;
    }
    uint32_t run = 0xffffffffu, cnt = 0;
#pragma unroll
    for (int i = 0; i < 16; i++) {
      if (tm & (1u << i)) {
        const uint32_t s = src_of(kk[i]);
        if (s != run) {
          if (run < g.nv && cnt) atomicAdd(&deg[run], cnt);
          run = s;
          cnt = 0;
        }
        cnt += dst_of(kk[i]) < g.nv ? 1u : 0u;
      }
    }
    if (run < g.nv && cnt) atomicAdd(&deg[run], cnt);
  }
}

// acc[u] += sum over edges (u, v) of contrib[v].  T double: where the binned form,
// which sums in 64 bits, would apply too but its setup does not pay; float: graphs too
// sparse for it, where the vertices' passes are most of an iteration and 8-byte sums
// cost a quarter more (2^24 vertices, 2.6e5 edges, ten iterations: 865 and 1097 us).
template <typename T>
__global__ void __launch_bounds__(256) k_fg_pull(FgArgs g, const float* __restrict__ contrib,
                                                 T* __restrict__ acc) {
  const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / kWave);
  for (uint64_t leaf = (uint64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; leaf < g.L;
       leaf += waves) {
    uint64_t kk[16];
    const uint32_t tm = wave_leaf_keys(g.bytes + leaf * (uint64_t)g.S, g.used[leaf], kk);
    float val[16];
#pragma unroll
    for (int i = 0; i < 16; i++) {
      const uint32_t d = dst_of(kk[i]);
      val[i] = ((tm & (1u << i)) && d < g.nv) ? contrib[d] : 0.f;
    }
    const uint32_t one = fg_single_source(g, leaf, kk, tm);
    if (one != 0xffffffffu) {
      T t = 0;
#pragma unroll
      for (int i = 0; i < 16; i++) t += val[i];
      t = wave_sum_float(t);
      if (lane_id() == 0 && one < g.nv) atomicAdd(&acc[one], t);
      continue;
    }
    uint32_t run = 0xffffffffu;
    T sum = 0;
#pragma unroll
    for (int i = 0; i < 16; i++) {
      if (tm & (1u << i)) {
        const uint32_t s = src_of(kk[i]);
        if (s != run) {
          if (run < g.nv) atomicAdd(&acc[run], sum);
          run = s;
          sum = 0;
        }
        sum += val[i];
      }
    }
    if (run < g.nv) atomicAdd(&acc[run], sum);
  }
}

// BFS state besides the levels: two bitmaps over the vertices, rebuilt from the
// levels after every level (2 MB each at 2^24 vertices, so the random tests of
// a step hit L2 instead of the 4-byte level entries):
//   front: level == cur (the vertices being expanded);
//   seen:  level != unvisited.
constexpr uint32_t kUnvisited = 0xffffffffu;

struct BfsBits {
  const uint32_t* front;
  const uint32_t* seen;
};

__device__ __forceinline__ bool bit_of(const uint32_t* b, uint32_t v) { return (b[v >> 5] >> (v & 31)) & 1u; }

// Whether bits [s0, s1] of b (xor `flip`) hold a one.
__device__ __forceinline__ bool any_bit(const uint32_t* b, uint32_t flip, uint32_t s0, uint32_t s1) {
  const uint32_t w0 = s0 >> 5, w1 = s1 >> 5;
  uint32_t acc = 0;
  for (uint32_t w = w0; w <= w1; w++) {
    uint32_t x = b[w] ^ flip;
    if (w == w0) x &= ~0u << (s0 & 31);
    if (w == w1) x &= ~0u >> (31 - (s1 & 31));
    acc |= x;
  }
  return acc != 0;
}

// Whether leaf f holds a source whose bit in b (xor `flip`) is set (one lane).
// The leaf's keys lie in [head[f], head[f + 1]), so its sources lie in
// [src(head[f]), src(head[f + 1])]: a few bitmap words instead of a decode.
// Spans wider than kFgSkipSpan vertices (the last leaf, sparse id ranges) are
// not tested and count as holding one.
constexpr uint32_t kFgSkipSpan = 256;

__device__ __forceinline__ bool fg_leaf_has(const FgArgs& g, const uint32_t* b, uint32_t flip, uint64_t f) {
  const uint64_t h = g.head[f];
  if (h == kNoKey) return false;  // the empty leaf of an empty set
  const uint32_t s0 = src_of(h);
  if (s0 >= g.nv) return false;  // every key of the leaf is ignored
  if (f + 1 >= g.L) return true;
  const uint32_t s1 = min(src_of(g.head[f + 1]), g.nv - 1);
  if (s1 - s0 >= kFgSkipSpan) return true;
  return any_bit(b, flip, s0, s1);
}

// One level of a level-synchronous BFS (the hop distance of every vertex
// reached from the source).  On a symmetric edge set a vertex v joins level
// cur + 1 iff it is unvisited and some neighbour u has level cur, which can be
// found from either end of the edge (u, v):
//   top-down:  for edges (u, v) with u at level cur, mark v if unvisited;
//   bottom-up: for edges (v, u) with v unvisited, mark v if u is at level cur.
// Each direction decodes only the leaves holding a source it needs (level cur,
// resp. unvisited): a wave takes kBfsGroup leaves, each lane tests one, and the
// wave then decodes the needed ones one after another, the next one's bytes on
// their way.  A mark is a plain store of cur + 1 into the levels: every writer
// stores the same value, and the tests read only the bitmaps, which this level
// does not change.
//
// A lane's sources are few and close: two bitmap words from its first source on
// decide which of its keys matter (cand); the random reads of the other bitmap
// are then issued four at a time for those only, and bottom-up stops at the
// first hit of a source.  The leaf test cannot tell vertices without edges from
// unvisited ones, so bottom-up also notes the leaves whose sources are all
// visited (`done`, may be null), which no later level decodes.
//
// Bound by vector instructions and the rate of L2 line requests.  On a symmetric
// R-MAT graph of 2^24 vertices (1e6 leaves) the widest levels took 1060 us
// top-down and 1839, 935, 468 and 321 bottom-up with one bitmap read after
// another for each of a lane's 16 key places, 64 leaves per wave and no `done`:
// now 560 and 1390, 595, 225, 127.
constexpr uint32_t kBfsGroup = 32;
constexpr uint32_t kBfsSpan = 384;  // sources of a leaf tracked for `done`, from its first one's word on

template <bool kBottomUp>
__global__ void __launch_bounds__(256) k_fg_bfs_step(FgArgs g, BfsBits bb, uint32_t* __restrict__ level,
                                                     uint32_t cur, uint8_t* __restrict__ done) {
  __shared__ uint32_t hits[256 / kWave][kBfsSpan / 32];  // sources marked by the current leaf
  const uint32_t lane = lane_id(), wid = threadIdx.x / kWave;
  const uint32_t* __restrict__ mine = kBottomUp ? bb.seen : bb.front;   // decides on sources
  const uint32_t* __restrict__ other = kBottomUp ? bb.front : bb.seen;  // on destinations
  constexpr uint32_t kFlip = kBottomUp ? ~0u : 0u;
  const uint32_t lastw = (g.nv - 1) / 32;
  const uint64_t base = ((uint64_t)blockIdx.x * (256 / kWave) + wid) * kBfsGroup;
  const uint64_t f = base + lane;
  bool need = false;
  uint32_t used_f = 0;
  if (lane < kBfsGroup && f < g.L && !(kBottomUp && done && done[f])) {
    need = fg_leaf_has(g, mine, kFlip, f);
    used_f = g.used[f];
  }
  uint64_t m = __ballot(need);
  uint32_t at = m ? (uint32_t)(__ffsll((unsigned long long)m) - 1) : 0;
  uint32_t used = (uint32_t)__builtin_amdgcn_readlane((int)used_f, (int)at);
  uint4 w = make_uint4(0, 0, 0, 0);
  if (m) w = wave_leaf_bytes(g.bytes + (base + at) * g.S, used);
  while (m) {
    const uint64_t leaf = base + at;
    m &= m - 1;
    const uint4 wc = w;
    const uint32_t uc = used;
    if (m) {
      at = (uint32_t)(__ffsll((unsigned long long)m) - 1);
      used = (uint32_t)__builtin_amdgcn_readlane((int)used_f, (int)at);
      w = wave_leaf_bytes(g.bytes + (base + at) * g.S, used);
    }
    uint64_t kk[16];
    const uint32_t tm = wave_leaf_keys(wc, uc, kk);
    // the lane's sources lie in [src(kk[0]), src(kk[15])]: kk[0] may be part of a
    // key, which is at least the key before it
    const uint32_t w0 = src_of(kk[0]) >> 5, b0 = w0 << 5;
    const uint32_t wa = mine[min(w0, lastw)] ^ kFlip, wb = mine[min(w0 + 1, lastw)] ^ kFlip;
    const bool far = tm && (src_of(kk[15]) - b0 >= 64 || src_of(kk[15]) >= g.nv);
    uint32_t cand = 0;
    if (!__ballot(far)) {
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const uint32_t rel = src_of(kk[i]) - b0;
        const uint32_t bit = __builtin_amdgcn_ubfe(rel < 32 ? wa : wb, rel & 31u, 1);
        cand |= (dst_of(kk[i]) < g.nv ? bit : 0u) << i;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const uint32_t s = src_of(kk[i]);
        if ((tm & (1u << i)) && s < g.nv && dst_of(kk[i]) < g.nv) cand |= (((mine[s >> 5] ^ kFlip) >> (s & 31)) & 1u) << i;
      }
    }
    cand &= tm;
    if (!__ballot(cand != 0)) {
      if (kBottomUp && done && lane == 0) done[leaf] = 1;
      continue;
    }
    const uint32_t sbase = src_of(g.head[leaf]) & ~31u;
    if (kBottomUp && done) {
      if (lane < kBfsSpan / 32) hits[wid][lane] = 0;
      __builtin_amdgcn_wave_barrier();
    }
    uint32_t fs = 0xffffffffu;  // the last source marked by this lane
#pragma unroll
    for (int q = 0; q < 4; q++) {
      uint32_t fw[4];
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int i = 4 * q + j;
        const bool go = (cand & (1u << i)) && (!kBottomUp || src_of(kk[i]) != fs);
        fw[j] = kBottomUp ? 0u : ~0u;
        if (go) fw[j] = other[dst_of(kk[i]) >> 5];
      }
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int i = 4 * q + j;
        const uint32_t s = src_of(kk[i]), d = dst_of(kk[i]);
        const bool bit = (fw[j] >> (d & 31)) & 1u;
        if (kBottomUp) {
          if (bit && s != fs) {
            level[s] = cur + 1;
            fs = s;
            if (done && s - sbase < kBfsSpan) atomicOr(&hits[wid][(s - sbase) >> 5], 1u << (s & 31));
          }
        } else {
          if (!bit) level[d] = cur + 1;
        }
      }
    }
    if (kBottomUp && done) {
      __builtin_amdgcn_wave_barrier();
      bool left = false;
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const uint32_t rel = src_of(kk[i]) - sbase;
        if (cand & (1u << i)) left |= rel >= kBfsSpan || !((hits[wid][rel >> 5] >> (rel & 31)) & 1u);
      }
      if (!__ballot(left) && lane == 0) done[leaf] = 1;
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// After a level: the bitmaps for the next one (front: level == next; seen:
// level != unvisited), one 32-bit word per thread, and per block the number of
// vertices at level `next` and of unvisited vertices as one slot pair (summed by
// k_fg_fold_counts; no counter shared by all blocks).
__global__ void __launch_bounds__(256) k_fg_level_bits(const uint32_t* __restrict__ level, uint32_t nv, uint32_t next,
                                                       uint32_t* __restrict__ front, uint32_t* __restrict__ seen,
                                                       unsigned long long* __restrict__ part) {
  __shared__ uint64_t red[2][256 / kWave];
  uint64_t a = 0, b = 0;
  const uint32_t nw = (nv + 31) / 32;
  const bool vec = (reinterpret_cast<uintptr_t>(level) & 15) == 0;  // 16-byte loads of 4 levels
  for (uint32_t w = blockIdx.x * blockDim.x + threadIdx.x; w < nw; w += gridDim.x * blockDim.x) {
    uint32_t fw = 0, sw = 0;
    const uint32_t v0 = w * 32;
    if (v0 + 32 <= nv && vec) {
      const uint4* p = reinterpret_cast<const uint4*>(level + v0);
#pragma unroll
      for (int q = 0; q < 8; q++) {
        const uint4 x = p[q];
        const uint32_t l[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int j = 0; j < 4; j++) {
          fw |= (uint32_t)(l[j] == next) << (4 * q + j);
          sw |= (uint32_t)(l[j] != kUnvisited) << (4 * q + j);
        }
      }
    } else {
      for (uint32_t j = 0; v0 + j < nv; j++) {
        const uint32_t l = level[v0 + j];
        fw |= (uint32_t)(l == next) << j;
        sw |= (uint32_t)(l != kUnvisited) << j;
      }
    }
    front[w] = fw;
    seen[w] = sw;
    a += (uint32_t)__popc(fw);
    b += (uint32_t)(min(32u, nv - v0) - (uint32_t)__popc(sw));
  }
  a = wave_sum(a);
  b = wave_sum(b);
  if (lane_id() == 0) {
    red[0][threadIdx.x / kWave] = a;
    red[1][threadIdx.x / kWave] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 256 / kWave; w++) {
      a += red[0][w];
      b += red[1][w];
    }
    part[2 * blockIdx.x] = a;
    part[2 * blockIdx.x + 1] = b;
  }
}

// Sums n slot pairs into out[0], out[1] (one block; out is overwritten).
__global__ void __launch_bounds__(1024) k_fg_fold_counts(const unsigned long long* __restrict__ part, uint32_t n,
                                                         unsigned long long* __restrict__ out) {
  __shared__ uint64_t red[2][1024 / kWave];
  uint64_t a = 0, b = 0;
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    a += part[2 * i];
    b += part[2 * i + 1];
  }
  a = wave_sum(a);
  b = wave_sum(b);
  if (lane_id() == 0) {
    red[0][threadIdx.x / kWave] = a;
    red[1][threadIdx.x / kWave] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 1024 / kWave; w++) {
      a += red[0][w];
      b += red[1][w];
    }
    out[0] = a;
    out[1] = b;
  }
}

// Degree counts widened for a 64-bit prefix sum (the vertex offset array).
struct U32AsU64Fn {
  const uint32_t* p;
  __device__ uint64_t operator()(uint64_t i) const { return p[i]; }
};

// ---- connected components (label propagation with pointer jumping) -----------
// lab[u] = min(lab[u], min over edges (u, v) of lab[v]), one atomic per run of
// equal source; *changed is set when a label fell.  Labels only fall, and only
// to the label of a vertex of the same component, so the component's smallest
// id keeps its own label and, once no label falls, every vertex holds it.
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) x = min(x, (uint32_t)__shfl_xor((int)x, off, kWave));
  return x;
}

__global__ void __launch_bounds__(256) k_fg_cc_prop(FgArgs g, uint32_t* __restrict__ lab,
                                                    uint32_t* __restrict__ changed) {
  const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / kWave);
  bool ch = false;
  for (uint64_t leaf = (uint64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; leaf < g.L;
       leaf += waves) {
    uint64_t kk[16];
    const uint32_t tm = wave_leaf_keys(g.bytes + leaf * (uint64_t)g.S, g.used[leaf], kk);
    uint32_t val[16];
#pragma unroll
    for (int i = 0; i < 16; i++) {
      const uint32_t sv = src_of(kk[i]), d = dst_of(kk[i]);
      val[i] = ((tm & (1u << i)) && d < g.nv && sv < g.nv) ? lab[d] : 0xffffffffu;
    }
    const uint32_t one = fg_single_source(g, leaf, kk, tm);
    if (one != 0xffffffffu) {
      uint32_t m = 0xffffffffu;
#pragma unroll
      for (int i = 0; i < 16; i++) m = min(m, val[i]);
      m = wave_min_u32(m);
      if (lane_id() == 0 && one < g.nv && m != 0xffffffffu) ch |= atomicMin(&lab[one], m) > m;
      continue;
    }
    uint32_t run = 0xffffffffu, rmin = 0xffffffffu;
#pragma unroll
    for (int i = 0; i < 16; i++) {
      if (tm & (1u << i)) {
        const uint32_t sv = src_of(kk[i]);
        if (sv != run) {
          if (run < g.nv && rmin != 0xffffffffu) ch |= atomicMin(&lab[run], rmin) > rmin;
          run = sv;
          rmin = 0xffffffffu;
        }
        rmin = min(rmin, val[i]);
      }
    }
    if (run < g.nv && rmin != 0xffffffffu) ch |= atomicMin(&lab[run], rmin) > rmin;
  }
  if (__ballot(ch) && lane_id() == 0) *changed = 1u;  // every writer stores the same value
}

// Pointer jumping: lab[v] = lab[lab[v]] until it stops falling (every label
// on the chain is a vertex of v's component, so the result is too).
__global__ void k_fg_cc_jump(uint32_t* __restrict__ lab, uint32_t nv) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    uint32_t l = lab[v];
    for (;;) {
      const uint32_t ll = lab[l];
      if (ll >= l) break;
      l = ll;
    }
    lab[v] = l;
  }
}

__global__ void k_fg_iota(uint32_t* __restrict__ lab, uint32_t nv) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) lab[v] = v;
}

// ---- single-source betweenness (Brandes), level by level --------------------
// With BFS levels from the source known, on a symmetric edge set:
//   sigma[v] = sum over edges (v, u) with level[u] = level[v] - 1 of sigma[u]
//   delta[v] = sigma[v] * sum over edges (v, w) with level[w] = level[v] + 1 of
//              (1 + delta[w]) / sigma[w]
// A level's pass decodes only the leaves holding a source of that level (the
// `front` bitmap), folds each run of equal source and adds it with one FP64
// atomic.  kDelta selects the second formula.
template <bool kDelta>
__global__ void __launch_bounds__(256) k_fg_bc_level(FgArgs g, BfsBits bb, const uint32_t* __restrict__ level,
                                                     uint32_t cur, const double* sigma_in, const double* delta_in,
                                                     double* out) {
  const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x / kWave);
  const uint64_t wave = (uint64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const uint32_t want = kDelta ? cur + 1 : cur - 1;  // the neighbours' level
  for (uint64_t base = wave * kWave; base < g.L; base += nwaves * kWave) {
    const uint64_t f = base + (uint64_t)lane_id();
    const bool need = f < g.L && fg_leaf_has(g, bb.front, 0u, f);
    uint64_t m = __ballot(need);
    while (m) {
      const uint64_t leaf = base + (uint64_t)(__ffsll((unsigned long long)m) - 1);
      m &= m - 1;
      uint64_t kk[16];
      const uint32_t tm = wave_leaf_keys(g.bytes + leaf * (uint64_t)g.S, g.used[leaf], kk);
      uint32_t run = 0xffffffffu;
      double acc = 0.0;
      bool any = false;
#pragma unroll
      for (int i = 0; i < 16; i++) {
        if (!(tm & (1u << i))) continue;
        const uint32_t sv = src_of(kk[i]), d = dst_of(kk[i]);
        if (sv != run) {
          if (any) atomicAdd(&out[run], kDelta ? sigma_in[run] * acc : acc);
          run = sv;
          acc = 0.0;
          any = false;
        }
        if (sv < g.nv && d < g.nv && bit_of(bb.front, sv) && level[d] == want) {
          acc += kDelta ? (1.0 + delta_in[d]) / sigma_in[d] : sigma_in[d];
          any = true;
        }
      }
      if (any) atomicAdd(&out[run], kDelta ? sigma_in[run] * acc : acc);
    }
  }
}

// PageRank vertex kernels around the pulls: the first contributions contrib[u] =
// p[u] / deg[u] (0 for vertices without edges) of uniform ranks and a cleared acc; then
// p[v] = (1 - d) / N + d * acc[v] after every pull, and (more) the same for the next.
template <typename T>
__global__ void k_pr_first(const uint32_t* __restrict__ deg, uint32_t nv, float rank0, float* __restrict__ contrib,
                           T* __restrict__ acc) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    contrib[v] = deg[v] ? rank0 / (float)deg[v] : 0.f;
    acc[v] = 0;
  }
}

template <typename T>
__global__ void k_pr_update(const uint32_t* __restrict__ deg, uint32_t nv, float base, float damping,
                            float* __restrict__ p, float* __restrict__ contrib, T* __restrict__ acc, int more) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const float r = base + damping * (float)acc[v];
    p[v] = r;
    if (more) {
      contrib[v] = deg[v] ? r / (float)deg[v] : 0.f;
      acc[v] = 0;
    }
  }
}

}  // namespace cpma_dev
