// Key-value leaves (the key-value CPMA the paper names as future work for
// weighted graphs, Section "Evaluation on graph workloads").  Every key
// carries an 8-byte value.  A leaf keeps its keys exactly as the CPMA does --
// the head and the delta codes from byte 0, clen bytes -- and the values as
// 8-byte words in key order at the end of the leaf.  Its filled bytes (used,
// which the density bounds count) are clen + 8 per key, so every key costs its
// code plus 8 and at most S / 9 keys fit a leaf.
#pragma once
#include "leaf.hpp"
#include "update.hpp"

namespace cpma_dev {

// LDS of the key-value merge, sized by the leaf size: the merged keys and values
// (a merged leaf of more than `cap` keys is staged in HBM instead), whose room
// first takes the old leaf's code bytes and where each code ends; then the old
// keys (at most S / 9 + 1 fit a leaf) and the per-rank counts, whose room takes
// the new code bytes in the end.  6.1 KB at S = 1024: 26 waves on a CU.
struct KvLayout {
  uint32_t nold, cap;
  uint32_t mk, mv, raw, ends, k, c, img, total;
  __host__ __device__ explicit KvLayout(uint32_t S) {
    nold = S / 9 + 2;
    cap = 2 * nold + 64;
    mk = 0;
    mv = mk + 8 * cap;
    raw = 0;
    ends = raw + ((S + 31) & ~15u);  // a code is read as three words
    const uint32_t merged = mv + 8 * cap, codes = ends + 2 * (nold + 1);
    k = ((merged > codes ? merged : codes) + 15) & ~15u;
    c = k + 8 * nold;
    img = k;
    const uint32_t counts = c + 4 * (nold + 1), image = img + S;
    total = ((counts > image ? counts : image) + 15) & ~15u;
  }
};

// The 7-bit groups of the low n <= 8 bytes of x, joined.
__device__ __forceinline__ uint64_t join_groups(uint64_t x, uint32_t n) {
  x &= 0x7f7f7f7f7f7f7f7full >> (64u - 8u * n);
  x = (x & 0x007f007f007f007full) | ((x & 0x7f007f007f007f00ull) >> 1);
  x = (x & 0x00003fff00003fffull) | ((x & 0x3fff00003fff0000ull) >> 2);
  return (x & 0x000000000fffffffull) | ((x & 0x0fffffff00000000ull) >> 4);
}

// Keys of a key-value leaf (cl code bytes, m keys) to K, one key per lane.  A
// third of such a leaf is codes (55 keys of 3 bytes at S = 1024), so the lanes
// take 4 bytes each and write where codes end to `ends`; then lane i joins the
// code of key i from the raw bytes and a scan of the deltas gives the keys.
__device__ __forceinline__ void kv_decode_keys(const uint8_t* __restrict__ lp, uint32_t cl, uint32_t m, uint32_t* raw,
                                               uint16_t* ends, uint64_t* K) {
  const uint32_t lane = lane_id();
  uint32_t found = 1;  // key 0 is the head
  if (lane == 0) ends[0] = 8;
  for (uint32_t c0 = 0; c0 < cl; c0 += 4 * kWave) {
    const uint32_t pos = c0 + 4 * lane;
    const uint32_t w = pos < cl ? *reinterpret_cast<const uint32_t*>(lp + pos) : 0u;
    if (pos < cl) raw[pos / 4] = w;
    uint32_t t = pos >= 8 && pos < cl ? ~w & 0x80808080u : 0u;
    if (pos < cl && cl - pos < 4) t &= (1u << (8 * (cl - pos))) - 1u;
    const uint32_t n = (uint32_t)__popc(t), incl = wave_incl_scan(n);
    uint32_t at = found + incl - n;
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) {
      if (t & (0x80u << (8 * i)) && at < m) ends[at++] = (uint16_t)(pos + i + 1);
    }
    found += lane63_u32(incl);
  }
  __syncthreads();
  uint64_t run = 0;
  for (uint32_t c0 = 0; c0 < m; c0 += kWave) {
    const uint32_t i = c0 + lane;
    uint64_t d = 0;
    if (i < m) {
      const uint32_t from = i ? ends[i - 1] : 0u, n = ends[i] - from;
      const uint32_t* q = raw + from / 4;
      const uint32_t w0 = q[0], w1 = q[1], w2 = q[2], sh = 8 * (from & 3);
      const uint64_t x = (uint64_t)__builtin_amdgcn_alignbit(w2, w1, sh) << 32 | __builtin_amdgcn_alignbit(w1, w0, sh);
      if (i == 0) {
        d = x;
      } else {
        d = join_groups(x, min(n, 8u));
        if (n > 8) {
          const uint8_t* rb = reinterpret_cast<const uint8_t*>(raw) + from;
          d |= (uint64_t)(rb[8] & 0x7fu) << 56;
          if (n > 9) d |= (uint64_t)(rb[9] & 0x7fu) << 63;
        }
      }
    }
    const uint64_t incl = wave_incl_scan(d);
    if (i < m) K[i] = run + incl;
    run += lane63_u64(incl);
  }
}

// Batch merge on key-value leaves: one wave per touched leaf, any slice length.
// The old keys are decoded to LDS.  Insert: each batch key's rank by binary
// search; it goes to its rank plus the new keys before it, and so does the value
// of a key that is present (when values are given); a new key counts one at its
// rank, whose prefix sum shifts the old keys.  Delete: found keys flag their
// slot; kept keys move down.  The merged keys are then re-encoded: codes that
// fit the leaf with their values are built in LDS and copied over the old ones,
// with the values straight behind them; a larger leaf goes to the segment's
// overflow-arena region (codes, then the values from the next 8-byte boundary).
// Bound by vector instructions: 1e6 keys into 1e7 (5.5 keys into each of 180 000
// leaves, 0.37 GB at least) took 300 us with every lane parsing 16 bytes, the
// values kept in LDS three times and every code length taken twice; 149 us now.
__global__ void __launch_bounds__(kWave) k_kv_merge(MergeArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ unsigned long long stage_off;
  const uint32_t S = a.S;
  const KvLayout lay(S);
  uint64_t* K = reinterpret_cast<uint64_t*>(smem + lay.k);
  uint64_t* MK = reinterpret_cast<uint64_t*>(smem + lay.mk);
  uint64_t* MV = reinterpret_cast<uint64_t*>(smem + lay.mv);
  uint8_t* img = smem + lay.img;  // the new codes
  uint32_t* C = reinterpret_cast<uint32_t*>(smem + lay.c);
  const uint32_t lane = lane_id();
  const uint64_t T = a.ctr->T;
  const uint64_t below = (1ull << lane) - 1ull;
  unsigned long long delta = 0, alg = 0;
  for (uint64_t t = blockIdx.x; t < T; t += gridDim.x) {
    const uint4 d = a.seg_desc[t];
    const uint64_t leaf = d.x;
    const uint32_t b = d.y, e = a.seg_begin[t + 1];
    const uint32_t nb = e - b;
    const uint32_t used0 = d.z;
    const uint32_t cl0 = used0 ? a.clen[leaf] : 0u;
    const uint32_t m0 = (used0 - cl0) / 8;
    uint8_t* lp = a.bytes + leaf * (uint64_t)S;
    const uint64_t* ov = reinterpret_cast<const uint64_t*>(lp + S - 8u * m0);
    const uint64_t* Bs = a.B + b;
    // the first two rounds' old values and the first batch key come with the codes
    const uint64_t v0 = lane < m0 ? ov[lane] : 0, v1 = lane + kWave < m0 ? ov[lane + kWave] : 0;
    const uint64_t x0 = lane < nb ? Bs[lane] : 0;
    auto old_value = [&](uint32_t c0) { return c0 == 0 ? v0 : c0 == kWave ? v1 : ov[c0 + lane]; };
    for (uint32_t i = lane; i <= m0; i += kWave) C[i] = 0;
    kv_decode_keys(lp, cl0, m0, reinterpret_cast<uint32_t*>(smem + lay.raw), reinterpret_cast<uint16_t*>(smem + lay.ends),
                   K);
    __syncthreads();
    uint32_t mn = 0;
    bool ok = true, staged = false;
    uint64_t off = 0;
    // rank of batch key x among the old keys; true if it is one of them
    auto rank = [&](uint64_t x, uint32_t& r) {
      r = lds_lower_bound<uint64_t>(K, m0, x);
      return r < m0 && K[r] == x;
    };
    // places the merged keys and values at M, MVp
    auto place = [&](auto M, auto MVp, uint32_t r0, uint32_t flags0) {
      if (a.is_insert) {
        uint32_t carry = 0;
        for (uint32_t c0 = 0; c0 < m0; c0 += kWave) {
          const uint32_t i = c0 + lane;
          const uint32_t cv = i < m0 ? C[i] : 0u;
          const uint32_t incl = wave_incl_scan(cv);
          if (i < m0) {
            M[i + carry + incl] = K[i];
            MVp[i + carry + incl] = old_value(c0);
          }
          carry += lane63_u32(incl);
        }
        __threadfence_block();
        __syncthreads();  // a present key's new value comes after its old one
        uint32_t before = 0;
        for (uint32_t c0 = 0; c0 < nb; c0 += kWave) {
          const uint32_t j = c0 + lane;
          uint64_t x = x0;
          uint32_t r = r0;
          bool present = flags0 & 2u, isnew = flags0 & 1u;
          if (c0) {
            present = isnew = false;
            if (j < nb) {
              x = Bs[j];
              present = rank(x, r);
              isnew = !present;
            }
          }
          const uint64_t nm = __ballot(isnew);
          const uint32_t p = r + before + (uint32_t)__popcll(nm & below);
          if (isnew) M[p] = x;
          if (isnew || (present && a.Bv)) MVp[p] = a.Bv ? a.Bv[b + j] : 0ull;
          before += (uint32_t)__popcll(nm);
        }
      } else {
        uint32_t gone = 0;
        for (uint32_t c0 = 0; c0 < m0; c0 += kWave) {
          const uint32_t i = c0 + lane;
          const bool g = i < m0 && C[i];
          const uint64_t gm = __ballot(g);
          if (i < m0 && !g) {
            const uint32_t p = i - gone - (uint32_t)__popcll(gm & below);
            M[p] = K[i];
            MVp[p] = old_value(c0);
          }
          gone += (uint32_t)__popcll(gm);
        }
      }
    };
    uint32_t r0 = 0, flags0 = 0;  // the first round's ranks: 1 new, 2 present
    uint32_t changed = 0;         // new keys or keys gone
    for (uint32_t c0 = 0; c0 < nb; c0 += kWave) {
      const uint32_t j = c0 + lane;
      bool hit = false;
      if (j < nb) {
        uint32_t r;
        const bool present = rank(c0 ? Bs[j] : x0, r);
        hit = present != (bool)a.is_insert;
        if (hit) atomicAdd(&C[r], 1u);  // a delete's keys are distinct: C stays 0 or 1
        if (c0 == 0) {
          r0 = r;
          flags0 = present ? 2u : 1u;
        }
      }
      changed += (uint32_t)__popcll(__ballot(hit));
    }
    mn = a.is_insert ? m0 + changed : m0 - changed;
    if (mn > lay.cap) {
      if (lane == 0) stage_off = atomicAdd(&a.ctr->stage_cursor, (unsigned long long)mn);
      __syncthreads();
      off = stage_off;
      staged = true;
      ok = off + mn <= a.stage_cap;
    }
    __syncthreads();
    if (!ok) {
      if (lane == 0) atomicOr(&a.ctr->error, 1u);
      __syncthreads();
      continue;
    }
    delta += changed;
    // writes codes and values of the merged leaf; instantiated once for merged
    // keys in LDS and once for the staging buffer, so that each copy's accesses
    // have a known address space (a pointer that may be either compiles to
    // generic accesses).  False: the arena's region does not hold them.
    auto store = [&](auto M, auto MVp) {
      // codes to dst: returns their bytes; those past `room` are only counted
      auto encode = [&](auto dst, uint64_t room) {
        uint32_t run = 0;
        for (uint32_t c0 = 0; c0 < mn; c0 += kWave) {
          const uint32_t p = c0 + lane;
          const uint64_t key = p < mn ? M[p] : 0, dk = key - (p && p < mn ? M[p - 1] : 0);
          const uint32_t c = p < mn ? (p ? vlen(dk) : 8u) : 0u;
          const uint32_t incl = wave_incl_scan(c);
          if (p < mn && run + incl <= room) {
            auto q = dst + run + incl - c;
            if (p == 0)
              put_le64(q, key);
            else
              vput(q, dk);
          }
          run += lane63_u32(incl);
        }
        return run;
      };
      const uint32_t vat = 8u * mn < S ? S - 8u * mn : 0u;  // the values' place if all fits
      wave_zero(img, S);
      __syncthreads();
      const uint32_t cl = encode(img, vat);
      const uint32_t U = cl + 8u * mn;
      const bool to_arena = U > S;
      __syncthreads();
      uint64_t aoff = 0;
      if (to_arena) {
        aoff = arena_region(a, t);
        if (aoff + (((uint64_t)cl + 7) & ~7ull) + 8ull * mn > a.arena_cap) return false;
        encode(a.arena + aoff, ~0ull);
        uint64_t* vdst = reinterpret_cast<uint64_t*>(a.arena + aoff + ((cl + 7u) & ~7u));
        for (uint32_t p = lane; p < mn; p += kWave) vdst[p] = MVp[p];
      } else {
        // zeros between codes and values are already in the leaf, except where
        // old codes or old values were
        uint64_t* vdst = reinterpret_cast<uint64_t*>(lp + vat);
        for (uint32_t p = lane; p < mn; p += kWave) vdst[p] = MVp[p];
        const uint32_t low = max(cl, cl0), high = S - 8u * max(m0, mn);
        for (uint32_t o = 8u * lane; o < vat; o += 8u * kWave)
          if (o < low || o >= high) *reinterpret_cast<uint64_t*>(lp + o) = *reinterpret_cast<const uint64_t*>(img + o);
      }
      if (lane == 0) {
        if (to_arena) a.ovf[leaf] = aoff;
        a.used[leaf] = U;
        a.clen[leaf] = cl;
        a.head[leaf] = mn ? M[0] : kNoKey;
      }
      alg += used0 + U + 16ull * nb + 24;
      return true;
    };
    if (staged) {
      place(a.stage + off, a.vstage + off, r0, flags0);
      __threadfence_block();
      __syncthreads();
      ok = store(a.stage + off, a.vstage + off);
    } else {
      place(MK, MV, r0, flags0);
      __syncthreads();
      ok = store(MK, MV);
    }
    if (!ok && lane == 0) atomicOr(&a.ctr->error, 1u);
    __syncthreads();
  }
  if (lane == 0) {
    a.part[2 * blockIdx.x] = delta;
    a.part[2 * blockIdx.x + 1] = alg;
  }
}

// Keys of a sorted batch with their values: the first occurrence of each key
// (the smallest input position: the sort is stable) with the value at its
// input position.  pos: exclusive scan of first-occurrence flags.
__global__ void k_kv_compact(const uint64_t* __restrict__ a, const uint32_t* __restrict__ idx, uint64_t n,
                             const uint32_t* __restrict__ pos, const uint64_t* __restrict__ vals,
                             uint64_t* __restrict__ kout, uint64_t* __restrict__ vout,
                             unsigned long long* __restrict__ n_out) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    if (i == 0 || a[i] != a[i - 1]) {
      kout[pos[i]] = a[i];
      vout[pos[i]] = vals ? vals[idx[i] & 0x7fffffffu] : 0ull;
    }
    if (i == 0) *n_out = pos[n];
  }
}

}  // namespace cpma_dev
