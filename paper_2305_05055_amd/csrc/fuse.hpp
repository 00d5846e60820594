// One pass over a sequence of insert / delete requests (serving).
//
// The paper applies one batch of inserts or of deletes at a time (Section
// "Parallel Batch Updates in a PMA"), and a single writer applies its batches
// in order (Section "Evaluation on graph workloads").  A sequence of requests
// reduces to at most one delete batch and one insert batch with the same final
// set, and every request's count (keys it added or removed, as its own call
// would return) follows from one stable sort of all their keys:
//   * after a key's first operation in the sequence its state no longer depends
//     on the set: an insert leaves it present, a delete absent;
//   * so a later occurrence changes the key iff its kind differs from the
//     previous occurrence's, and the first changes it iff its kind differs from
//     the key's membership before the sequence;
//   * the final state follows the last occurrence's kind.
// Items are (key, value) with value = position in the concatenated requests |
// delete bit << 31; a stable sort by key keeps each key's occurrences in
// request order.
#pragma once
#include "merge_splice.hpp"
#include "query.hpp"

namespace cpma_dev {

// Request owning position p: the last r with at(r) <= p, of nreq + 1 entries in
// non-decreasing order (the last one the total).
template <typename At>
__device__ __forceinline__ uint32_t fuse_owner(At at, uint32_t nreq, uint64_t p) {
  uint32_t lo = 0, hi = nreq + 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (at(mid) <= p)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo - 1;
}
__device__ __forceinline__ uint32_t fuse_req_of(const uint64_t* off, uint32_t nreq, uint64_t p) {
  return fuse_owner([&](uint32_t r) { return off[r]; }, nreq, p);
}

// Requests differ in size by orders of magnitude, so the passes over their items
// divide positions, not requests, among the threads (a block per request: 96
// requests of 10 to 1e5 keys took 81 us to gather and 13.6 to mark; 8.9 and 8.0 now).

// Kind byte (0 insert, 1 delete) of every position, 16 per thread (kinds is
// 16-byte aligned).
__global__ void __launch_bounds__(256) k_fuse_kinds(const uint64_t* __restrict__ off,
                                                    const uint8_t* __restrict__ rdel, uint32_t nreq, uint64_t m,
                                                    uint8_t* __restrict__ kinds) {
  const uint64_t p0 = 16 * ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (p0 >= m) return;
  uint32_t r = fuse_req_of(off, nreq, p0), word[4];
  uint64_t end = off[r + 1];
#pragma unroll
  for (uint32_t j = 0; j < 16; j++) {
    if (p0 + j >= end && p0 + j < m) {
      r = fuse_req_of(off, nreq, p0 + j);
      end = off[r + 1];
    }
    const uint32_t bits = (uint32_t)rdel[r] << (8 * (j & 3));
    word[j / 4] = j & 3 ? word[j / 4] | bits : bits;
  }
  if (p0 + 16 <= m) {
    *reinterpret_cast<uint4*>(kinds + p0) = make_uint4(word[0], word[1], word[2], word[3]);
  } else {
    for (uint32_t j = 0; p0 + j < m; j++) kinds[p0 + j] = (uint8_t)(word[j / 4] >> (8 * (j & 3)));
  }
}

// Membership before the sequence of each distinct key, per leaf (large batches;
// k_contains otherwise): leaf f's distinct keys are
// keys[sbeg[f] .. sbeg[f + 1]); one wave decodes the leaf once into LDS (dynamic)
// and binary-searches each of them there.  Leaves of at most 1024 bytes whose
// keys and slice span less than 2^32 keep a 32-bit offset per byte
// (splice_parse), others their 64-bit keys (a leaf holds at most S - 7): 68 us
// for 27 000 leaves of 375 keys with 64-bit keys, 36 with offsets.
__global__ void __launch_bounds__(kWave) k_fuse_member_leaf(QueryArgs a, const uint64_t* __restrict__ keys,
                                                            const uint32_t* __restrict__ sbeg,
                                                            uint8_t* __restrict__ member) {
  extern __shared__ __align__(16) uint8_t smem[];
  const uint32_t lane = lane_id();
  for (uint64_t f = blockIdx.x; f < a.L; f += gridDim.x) {
    const uint32_t b = sbeg[f], e = sbeg[f + 1];
    if (b == e) continue;
    const uint32_t u = a.used[f];
    const uint64_t hd = a.head[f], k0 = keys[b];
    const uint64_t base = u && hd < k0 ? hd : k0;
    const uint64_t above = f + 1 < a.L ? a.head[f + 1] : ~0ull;
    const uint8_t* src = a.bytes + f * (uint64_t)a.S;
    if (a.S <= kWaveMaxS && above - base <= 1ull << 32) {
      uint32_t* K = reinterpret_cast<uint32_t*>(smem);
      uint32_t* term = K + kWaveMaxS;
      uint4 w = make_uint4(0, 0, 0, 0);
      if (16 * lane < u) w = *reinterpret_cast<const uint4*>(src + 16 * lane);
      const uint32_t tm = splice_parse(w, u, (uint32_t)(hd - base), K), tm2 = dpp_next32(tm);
      if (!(lane & 1)) term[lane / 2] = tm | tm2 << 16;
      __syncthreads();
      for (uint32_t j = b + lane; j < e; j += kWave) {
        const uint32_t x = (uint32_t)(keys[j] - base);
        uint32_t v;
        const uint32_t p = splice_find(K, u, x, &v);
        member[j] = p < u && v == x && (p < 8 || ((term[p / 32] >> (p & 31)) & 1u)) ? 1 : 0;
      }
    } else {
      uint64_t* K = reinterpret_cast<uint64_t*>(smem);
      const uint32_t nk = wave_decode_leaf(src, u, [&](uint32_t i, uint64_t x, uint64_t) { K[i] = x; });
      __syncthreads();
      for (uint32_t j = b + lane; j < e; j += kWave) {
        const uint64_t x = keys[j];
        const uint32_t lo = lds_lower_bound<uint64_t>(K, nk, x);
        member[j] = (lo < nk && K[lo] == x) ? 1 : 0;
      }
    }
    __syncthreads();
  }
}
__host__ inline uint32_t member_leaf_smem(uint32_t S) {
  const uint32_t wide = 8 * S, narrow = 4 * kWaveMaxS + 4 * (kWaveMaxS / 32);
  return wide > narrow || S > kWaveMaxS ? wide : narrow;
}

// Gather of requests that live in device memory: request r's n keys from src
// to out[dst ..), m keys in all, four positions per thread.
struct GatherReq {
  const uint64_t* src;
  uint64_t dst;
  uint64_t n;
};

__global__ void __launch_bounds__(256) k_fuse_gather(const GatherReq* __restrict__ t, uint32_t nreq, uint64_t m,
                                                     uint64_t* __restrict__ out) {
  const uint64_t base = (uint64_t)blockIdx.x * 1024 + threadIdx.x;
  auto at = [&](uint32_t r) { return r < nreq ? t[r].dst : m; };
  uint64_t end = 0, from = 0, x[4];
  const uint64_t* src = nullptr;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const uint64_t i = base + 256 * q;
    if (i < m && i >= end) {
      const GatherReq g = t[fuse_owner(at, nreq, i)];
      src = g.src;
      from = g.dst;
      end = g.dst + g.n;
    }
    x[q] = i < m ? src[i - from] : 0;
  }
#pragma unroll
  for (int q = 0; q < 4; q++)
    if (base + 256 * q < m) out[base + 256 * q] = x[q];
}

// Per sorted item: whether its request changes the key (credit, stored at the
// item's position), and per distinct key the net change of the whole sequence
// (code 1: absent before, present after; 2: present before, absent after; 0:
// unchanged).  dpos is the exclusive count of first occurrences.
__global__ void __launch_bounds__(256) k_fuse_credit(const uint64_t* __restrict__ keys,
                                                     const uint32_t* __restrict__ vals, uint64_t m,
                                                     const uint32_t* __restrict__ dpos,
                                                     const uint8_t* __restrict__ member,
                                                     uint8_t* __restrict__ credit, uint8_t* __restrict__ code) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t x = keys[i];
    const uint32_t v = vals[i];
    const uint32_t del = v >> 31;
    const bool first = i == 0 || keys[i - 1] != x;
    const uint32_t d = first ? dpos[i] : dpos[i] - 1u;
    const uint32_t was = member[d];
    // state before this item, as "absent" (the delete bit a previous item
    // would have had)
    const uint32_t prev_del = first ? (was ^ 1u) : (vals[i - 1] >> 31);
    credit[v & 0x7fffffffu] = (uint8_t)(del != prev_del);
    if (i + 1 == m || keys[i + 1] != x) code[d] = (uint8_t)(del ? (was ? 2 : 0) : (was ? 0 : 1));
  }
}

// Packed (insert, delete) flags of distinct key i: low word insert, high word
// delete; zero past nd.
struct FuseSplitFn {
  const uint8_t* code;
  const unsigned long long* nd;
  __device__ uint64_t operator()(uint64_t i) const {
    if (i >= *nd) return 0;
    const uint32_t c = code[i];
    return (uint64_t)(c == 1) | ((uint64_t)(c == 2) << 32);
  }
};

// Writes the net insert and delete batches (sorted, repeat-free) and their
// sizes (cnt[1] inserts, cnt[2] deletes).
__global__ void __launch_bounds__(256) k_fuse_split(const uint64_t* __restrict__ dkeys,
                                                    const uint8_t* __restrict__ code,
                                                    const uint64_t* __restrict__ pos,
                                                    uint64_t* __restrict__ ins, uint64_t* __restrict__ del,
                                                    unsigned long long* __restrict__ cnt) {
  const uint64_t nd = cnt[0];
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nd;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t c = code[i];
    if (c == 1) ins[(uint32_t)pos[i]] = dkeys[i];
    if (c == 2) del[pos[i] >> 32] = dkeys[i];
    if (i == 0) {
      cnt[1] = (uint32_t)pos[nd];
      cnt[2] = pos[nd] >> 32;
    }
  }
}

// Sum of the credit bytes of every request (positions are request-contiguous).
// A wave takes 1024 consecutive positions: one wave sum and one atomic when
// they belong to one request, else a run-length walk per lane over its 16.
__global__ void __launch_bounds__(256) k_fuse_reduce(const uint8_t* __restrict__ credit, uint64_t m,
                                                     const uint64_t* __restrict__ off, uint32_t nreq,
                                                     unsigned long long* __restrict__ res) {
  constexpr uint32_t kChunk = 16 * kWave;
  const int lane = lane_id();
  const uint64_t nchunks = (m + kChunk - 1) / kChunk;
  const uint64_t wstride = (uint64_t)gridDim.x * (blockDim.x / kWave);
  for (uint64_t w = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave; w < nchunks; w += wstride) {
    const uint64_t b = w * kChunk, e = min(b + kChunk, m);
    const uint32_t r0 = fuse_req_of(off, nreq, b), r1 = fuse_req_of(off, nreq, e - 1);
    if (r0 == r1) {
      uint32_t c = 0;
#pragma unroll
      for (uint32_t j = 0; j < 16; j++) {
        const uint64_t p = b + j * kWave + lane;
        if (p < e) c += credit[p];
      }
      c = wave_sum(c);
      if (lane == 0 && c) atomicAdd(&res[r0], (unsigned long long)c);
    } else {
      const uint64_t p0 = b + (uint64_t)lane * 16;
      if (p0 < e) {
        const uint64_t p1 = min(p0 + 16, e);
        uint32_t r = fuse_req_of(off, nreq, p0);
        uint64_t end = off[r + 1];
        uint32_t acc = 0;
        for (uint64_t p = p0; p < p1; p++) {
          while (p >= end) {
            if (acc) atomicAdd(&res[r], (unsigned long long)acc);
            acc = 0;
            r++;
            end = off[r + 1];
          }
          acc += credit[p];
        }
        if (acc) atomicAdd(&res[r], (unsigned long long)acc);
      }
    }
  }
}

}  // namespace cpma_dev
