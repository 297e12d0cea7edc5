// radix_small.h -- one block's stable LSD radix passes over up to kRadixSmall keys in LDS.
//
// Ranking as in radix.hip: every wave owns a contiguous part of the items and ranks them 64 at a time with one
// ballot per digit bit against its own digit counters.  A key moves with its original index (perm); the caller
// gathers values through it at the end.  A pass whose digit is the same everywhere (the exponent bits of depths)
// leaves the order alone.
#pragma once
#include "ges_internal.h"

namespace ges {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallRounds = (int)kRadixSmall / kSmallThreads;

struct SmallSort {
  uint32_t key[kRadixSmall];
  uint16_t perm[kRadixSmall];
  uint16_t cnt[kSmallWaves][256];   // per-wave digit counts, then each wave's base within its digit
  uint16_t dstart[256];
  uint32_t wsum[4];
  uint32_t kept;
};
static_assert(kRadixSmall <= 65536, "positions are 16-bit");

__device__ __forceinline__ void small_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One pass over items [0, n) of L, by the whole block; with `filter`, items whose key is kNoKey are dropped.
// Returns the items kept.
__device__ __forceinline__ uint32_t small_sort_pass(SmallSort& L, uint32_t n, int shift, int bits, bool filter) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint32_t mask = (1u << bits) - 1u;
  const int rounds = (int)((n + kSmallThreads - 1) / kSmallThreads);   // the waves share the items evenly
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (int d = lane; d < 256; d += 64) L.cnt[w][d] = 0u;
  small_fence();
  uint32_t key[kSmallRounds], rank[kSmallRounds];
  uint16_t perm[kSmallRounds];
  uint32_t validmask = 0;
#pragma unroll
  for (int r = 0; r < kSmallRounds; ++r) {
    if (r >= rounds) break;
    const uint32_t i = (uint32_t)(w * rounds + r) * 64u + (uint32_t)lane;
    const bool in = i < n;
    key[r] = in ? L.key[i] : kNoKey;
    perm[r] = in ? L.perm[i] : 0;
    const bool valid = in && !(filter && key[r] == kNoKey);
    const uint32_t dg = (key[r] >> shift) & mask;
    uint64_t peers = __ballot(valid);
    for (int bit = 0; bit < bits; ++bit) {
      const uint32_t b = (dg >> bit) & 1u;
      const uint64_t m = __ballot(b != 0u);
      peers &= b ? m : ~m;
    }
    uint32_t rk = 0u;
    if (valid) {
      const uint32_t before = L.cnt[w][dg];
      rk = before + (uint32_t)__popcll(peers & below);
      if ((peers >> lane) == 1ull) L.cnt[w][dg] = (uint16_t)(before + (uint32_t)__popcll(peers));   // last peer
      validmask |= 1u << r;
    }
    small_fence();
    rank[r] = rk;
  }
  __syncthreads();
  uint32_t tot = 0;
  if (t < 256) {
    for (int k = 0; k < kSmallWaves; ++k) {
      const uint32_t c = L.cnt[k][t];
      L.cnt[k][t] = (uint16_t)tot;
      tot += c;
    }
  }
  uint32_t s = tot;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)s, d, 64);
    if (lane >= d) s += y;
  }
  if (t < 256 && lane == 63) L.wsum[w] = s;
  // a digit that every item has: nothing moves (unless items are dropped)
  const int same = __syncthreads_or(!filter && t < 256 && tot == n);
  if (same) return n;
  if (t < 256) {
    uint32_t ls = s - tot;
    for (int k = 0; k < w; ++k) ls += L.wsum[k];
    L.dstart[t] = (uint16_t)ls;
    if (t == 255) L.kept = ls + tot;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSmallRounds; ++r) {
    if (r >= rounds) break;
    if (!((validmask >> r) & 1u)) continue;
    const uint32_t dg = (key[r] >> shift) & mask;
    const uint32_t pos = (uint32_t)L.dstart[dg] + L.cnt[w][dg] + rank[r];
    L.key[pos] = key[r];
    L.perm[pos] = perm[r];
  }
  __syncthreads();
  return L.kept;
}

}  // namespace ges
