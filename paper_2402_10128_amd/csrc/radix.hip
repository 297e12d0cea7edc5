// radix.hip -- one stable LSD radix pass over (u32 key, u32 value) items with digits of up to 8 bits.
//
// Reduce-then-scan, three launches per pass:
//   upsweep:   each block counts the digits of its items in per-wave LDS histograms and writes its 256
//              counts into the digit table ([16 digit groups][nblocks][16], see radix_tidx);
//   scan:      one block per digit turns its counts into exclusive per-block offsets and writes the
//              digit's total;
//   downsweep: each block ranks its items stably -- every wave owns a contiguous share of the block's
//              items and ranks them 64 at a time with one ballot per digit bit (lanes holding the same
//              digit) against wave-private digit counters -- places keys and then pairs in LDS in digit order, and writes
//              each digit's run to its global position (exclusive digit total prefix + the block's offset),
//              so that consecutive threads write consecutive addresses.
// A filtering pass drops items whose key is kNoKey (compaction) and stores the kept count.  Values are (u32, u32) pairs;
// the first pass makes them from a value array and the item's index (the pair sort carries each pair's slot in the
// candidate layout to the backward pass).
//
// What bounds a downsweep is the traffic of its scattered runs: the longer a run of a digit, the closer it comes to a copy,
// and with more waves per CU more lines are half written at a time.  So a block's tile grows with the input as far as
// there are blocks enough (radix_shape): 2,048 items (256 threads) up to 2M, 4,096 (512) up to 64M, 16,384 (1,024, one
// block per CU) beyond.  Tile sort of 169M slots: 2.86 ms with 2,048, 2.54 with 4,096, 2.08 with 16,384; 13.5M slots:
// 215 / 183 / 242 us (8,192) and 3.9M: 80 / 74 / 82; depth sort of 5M items 220 / 184, 3M 119 / 109, 1M 78 / 84, 200k 59 / 69.
// The two larger tiles meet at the upper line: 35M slots 428 / 459, 52M 655 / 666, 70M 882 / 876, 104M 1,336 / 1,280.
// Several tiles per block in turn (a shorter digit table), with or without the next tile's loads ahead, was slower
// than one.  Within a block the counters are read and added to without waiting between the rounds of 64, the digit's width is
// a template argument and the pairs reuse the keys' LDS: 262 -> 215 us for the 13.5M slots, 140 -> 120 for the 3M items.
// A sort of up to kRadixSmall items is one block working in LDS instead (radix_small.h).  Reading the counts of the
// blocks before by looking back over words they publish, one launch per pass, was slower except on small inputs: the
// words cross the XCDs (depth sort of 3M splats 137 -> 203 us, tile sort of 169M slots 2.98 -> 3.85 ms, of 200k splats
// 75 -> 76).
#include "ges_internal.h"

namespace ges {

// Lanes of this wave holding the same digit (valid lanes only), one ballot per digit bit.
template <int BITS>
__device__ __forceinline__ uint64_t radix_peers(bool valid, uint32_t dg) {
  const uint64_t all = __ballot(valid);
  uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
#pragma unroll
  for (int bit = 0; bit < BITS; ++bit) {
    const int32_t set = (int32_t)(dg << (31 - bit)) >> 31;   // all ones if the lane's bit is set
    const uint64_t m = __ballot(set != 0);
    lo &= ~((uint32_t)m ^ (uint32_t)set);
    hi &= ~((uint32_t)(m >> 32) ^ (uint32_t)set);
  }
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t radix_count(const RadixPass& p) {
  return p.count_dev ? *p.count_dev : p.count_host;
}

__device__ __forceinline__ uint32_t radix_digit(const RadixPass& p, uint32_t k) {
  return (k >> p.shift) & ((1u << p.bits) - 1u);
}

// The digit table holds, per block b and digit d, the block's count of d and then its exclusive prefix over
// the blocks.  Layout [d / 16][b][d % 16]: a block's 256 entries are 16 runs of 64 contiguous bytes (its
// writes in the upsweep and reads in the downsweep are whole segments; digit-major rows of 4-byte entries
// left a partial segment per entry), and a group of 16 digits is a contiguous [blocks][16] array for the
// scan.
constexpr int kScanThreads = 1024;
constexpr int kDigitGroup = 16;
__device__ __forceinline__ size_t radix_tidx(uint32_t d, uint32_t b, uint32_t nblocks) {
  return ((size_t)(d / kDigitGroup) * nblocks + b) * kDigitGroup + (d % kDigitGroup);
}

__global__ void __launch_bounds__(kRadixThreads) radix_upsweep_kernel(RadixPass p) {
  constexpr int kWaves = kRadixThreads / 64, ITEMS = kRadixItems;
  __shared__ uint32_t hist[kWaves][256];
  __shared__ unsigned long long wsum[kWaves];
  const uint32_t n = radix_count(p);
  const int w = threadIdx.x >> 6;
  unsigned long long weight = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) hist[k][threadIdx.x] = 0u;
  __syncthreads();
  const uint64_t begin = (uint64_t)blockIdx.x * p.span;
  const uint64_t end = begin + p.span < n ? begin + p.span : n;
  for (uint64_t base = begin; base < end; base += kRadixThreads * ITEMS) {
    uint32_t key[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const uint64_t i = base + (uint64_t)it * kRadixThreads + threadIdx.x;
      key[it] = i < end ? p.keys_in[i] : kNoKey;
      if (p.weights && i < end) weight += p.weights[i];   // 0 for a dropped item
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const uint64_t i = base + (uint64_t)it * kRadixThreads + threadIdx.x;
      if (i < end && !(p.filter && key[it] == kNoKey)) atomicAdd(&hist[w][radix_digit(p, key[it])], 1u);
    }
  }
  __syncthreads();
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) c += hist[k][threadIdx.x];
  p.table[radix_tidx(threadIdx.x, blockIdx.x, p.nblocks)] = c;
  if (!p.weights) return;
  for (int off = 32; off > 0; off >>= 1) weight += __shfl_xor(weight, off, 64);
  if ((threadIdx.x & 63) == 0) wsum[w] = weight;
  __syncthreads();
  if (threadIdx.x == 0) p.weight_sums[blockIdx.x] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
}

// The blocks' weight sums added up and handed out, by one block.
__device__ __forceinline__ void post_weights(const RadixPass& p) {
  __shared__ unsigned long long part[kScanThreads / 64];
  unsigned long long s = 0;
  for (uint32_t b = threadIdx.x; b < p.nblocks; b += blockDim.x) s += p.weight_sums[b];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (uint32_t k = 1; k < blockDim.x / 64; ++k) s += part[k];
    if (p.mail) post_count(p.mail, p.token, s);
    if (p.weight_total) *p.weight_total = s > 0xffffffffull ? 0xffffffffu : (uint32_t)s;
  }
}

// Few blocks: the downsweep's blocks add up the table themselves (a row of 1 KB per block, in L2), which saves
// the scan's launch (depth sort of 50k splats 71 -> 64
// us, their tile sort 37 -> 34; with 98 blocks and more the adding costs more than the launch: 73 -> 82).
constexpr uint32_t kOwnScanBlocks = 64;
__host__ __device__ inline bool radix_own_scan(const RadixPass& p) { return p.nblocks <= kOwnScanBlocks; }

// One block per digit: the exclusive scan of the digit's counts over the blocks (8 entries per thread per
// round, 1,024 threads: one round for up to 8,192 blocks), its total to totals[].  The 16 digits of a group
// share the table's 64-byte segments, so they are dealt to one XCD (blocks go to the XCDs round-robin) and
// each segment is fetched once into that XCD's L2.  Digits beyond the pass's width only clear their total.
__global__ void __launch_bounds__(kScanThreads) radix_scan_kernel(RadixPass p) {
  constexpr int kPer = 8;
  __shared__ uint32_t wsum[kScanThreads / 64];
  __shared__ uint32_t carry;
  if (blockIdx.x == 256) return post_weights(p);
  const uint32_t x = blockIdx.x & 7u, i = blockIdx.x >> 3;   // XCD, and the block's index on it
  const uint32_t d = (((i / kDigitGroup) << 3) + x) * kDigitGroup + (i % kDigitGroup);
  if (d >= (1u << p.bits)) {
    if (threadIdx.x == 0) p.totals[d] = 0u;
    return;
  }
  uint32_t* col = p.table + radix_tidx(d, 0, p.nblocks);   // entry of block b at col[16 b]
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x == 0) carry = 0u;
  __syncthreads();
  for (uint32_t base = 0; base < p.nblocks; base += kScanThreads * kPer) {
    const uint32_t j0 = base + threadIdx.x * kPer;
    uint32_t v[kPer];
    uint32_t local = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      v[k] = j0 + k < p.nblocks ? col[(size_t)(j0 + k) * kDigitGroup] : 0u;
      local += v[k];
    }
    uint32_t s = local;
#pragma unroll
    for (int dd = 1; dd < 64; dd <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)s, dd, 64);
      if (lane >= dd) s += y;
    }
    if (lane == 63) wsum[w] = s;
    __syncthreads();
    uint32_t run = carry + s - local;
    for (int k = 0; k < w; ++k) run += wsum[k];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (j0 + k < p.nblocks) col[(size_t)(j0 + k) * kDigitGroup] = run;
      run += v[k];
    }
    __syncthreads();
    if (threadIdx.x == kScanThreads - 1) carry = run;
    __syncthreads();
  }
  if (threadIdx.x == 0) p.totals[d] = carry;
}

// Inclusive sum over a wave's lanes.
__device__ __forceinline__ uint32_t radix_wave_scan(uint32_t v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v += y;
  }
  return v;
}

// Workgroups are dealt to the 8 XCDs in turn.  The first pass of a large sort gives every XCD one contiguous eighth of the
// input instead: its blocks write neighbouring pieces of each digit's run, and lines are completed in one L2 (tile sort
// of 169M slots 2.08 -> 2.01 ms; later passes read runs of their own digit order, where it gains nothing, and small
// inputs lose by it).
__device__ __forceinline__ uint32_t radix_block(bool banded, uint32_t nblocks) {
  if (!banded) return blockIdx.x;
  const uint32_t x = blockIdx.x & 7u, i = blockIdx.x >> 3, full = nblocks >> 3, rest = nblocks & 7u;
  return x * full + min(x, rest) + i;
}

template <int THREADS, int ITEMS, int BITS>
__global__ void __launch_bounds__(THREADS) radix_downsweep_kernel(RadixPass p) {
  const uint32_t block = radix_block(THREADS > kRadixThreads && p.filter, p.nblocks);
  constexpr int kWaves = THREADS / 64;
  constexpr int kTile = THREADS * ITEMS;
  constexpr int kPerWave = kTile / kWaves;   // contiguous items of one wave
  __shared__ uint2 stage[kTile];          // the tile in digit order: its keys, then its pairs
  __shared__ uint32_t cnt[kWaves][256];   // per-wave digit counts, then each wave's base within its digit
  __shared__ uint32_t dstart[256];        // block-local start of each digit
  __shared__ uint32_t gstart[256];        // global position of the block's first item of each digit
  __shared__ uint32_t wsum[2][4];
  __shared__ uint32_t kept;
  uint32_t* const sk = reinterpret_cast<uint32_t*>(stage);
  const uint32_t n = radix_count(p);
  const int lane = threadIdx.x & 63, t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  if (block != 0 && (uint64_t)block * p.span >= n) return;   // whole block
  if (block == 0 && p.weights && (p.mail || p.weight_total) && radix_own_scan(p)) post_weights(p);   // otherwise the scan has
  // the global start of the block's run of each digit: the digit's items in the whole input and in the blocks before
  uint32_t gtot = 0, before_me = 0, g = 0;
  const bool digits = THREADS == 256 || t < 256;   // the threads that have a digit: whole waves
  if (digits) {
    if (radix_own_scan(p)) {
      for (uint32_t b0 = 0; b0 < p.nblocks; b0 += 16) {
        uint32_t c[16];
#pragma unroll
        for (uint32_t e = 0; e < 16; ++e) c[e] = b0 + e < p.nblocks ? p.table[radix_tidx(t, b0 + e, p.nblocks)] : 0u;
#pragma unroll
        for (uint32_t e = 0; e < 16; ++e) {
          gtot += c[e];
          if (b0 + e < block) before_me += c[e];
        }
      }
    } else {
      gtot = p.totals[t];
      before_me = p.table[radix_tidx(t, block, p.nblocks)];
    }
    g = radix_wave_scan(gtot);
    if (lane == 63) wsum[1][w] = g;
  }
  __syncthreads();
  if (digits) {
    uint32_t gs = g - gtot;
    for (int k = 0; k < w; ++k) gs += wsum[1][k];
    gstart[t] = gs + before_me;
    if (block == 0 && t == 255 && p.filter && p.count_out) *p.count_out = gs + gtot;
  }
  // the wave's items; a wave past the end reads the first item and counts none
  const uint64_t at = (uint64_t)block * kTile + (uint64_t)(w * kPerWave);
  const uint32_t left = at >= n ? 0u : (n - at < kPerWave ? (uint32_t)(n - at) : (uint32_t)kPerWave);
  const uint64_t from = left ? at : 0;
  const uint32_t last = left ? left - 1 : 0;
  if (n == 0u) return;   // whole block (the first one)
#pragma unroll
  for (int k = 0; k < 4; ++k) cnt[w][lane + 64 * k] = 0u;
  uint32_t key[ITEMS], rank[ITEMS];
  uint2 val[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) key[r] = (p.keys_in + from)[min((uint32_t)(r * 64 + lane), last)];
  if (p.pvals_in) {
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) val[r] = (p.pvals_in + from)[min((uint32_t)(r * 64 + lane), last)];
  } else {
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const uint32_t o = min((uint32_t)(r * 64 + lane), last);
      val[r] = make_uint2((p.vals_in + from)[o], (uint32_t)from + o);
    }
  }
  // ranks: the lanes of a digit read the wave's count of it, then one of them adds theirs; LDS takes a wave's accesses in
  // order, so no round waits for the one before
  uint32_t validmask = 0;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool valid = (uint32_t)(r * 64 + lane) < left && !(p.filter && key[r] == kNoKey);
    const uint32_t dg = radix_digit(p, key[r]);
    const uint64_t peers = radix_peers<BITS>(valid, dg);
    const uint32_t ahead = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
    validmask |= valid ? 1u << r : 0u;
    rank[r] = __hip_atomic_load(&cnt[w][dg], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT) + ahead;
    if (valid && ahead == 0u)
      __hip_atomic_fetch_add(&cnt[w][dg], (uint32_t)__popcll(peers), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  __syncthreads();
  // per digit: each wave's base within the digit and the tile's digit counts scanned over the digits
  uint32_t tot = 0, s = 0;
  if (digits) {
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
      const uint32_t c = cnt[k][t];
      cnt[k][t] = tot;
      tot += c;
    }
    s = radix_wave_scan(tot);
    if (lane == 63) wsum[0][w] = s;
  }
  __syncthreads();
  if (digits) {
    uint32_t ls = s - tot;
    for (int k = 0; k < w; ++k) ls += wsum[0][k];
    dstart[t] = ls;
    if (t == 255) kept = ls + tot;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t dg = radix_digit(p, key[r]);
    rank[r] += dstart[dg] + cnt[w][dg];
    if ((validmask >> r) & 1u) sk[rank[r]] = key[r];
  }
  __syncthreads();
  const uint32_t m = kept;
  uint32_t dst[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t j = t + r * THREADS;
    const uint32_t k = sk[j];   // what an earlier phase left, past the tile's last
    const uint32_t dg = radix_digit(p, k);
    dst[r] = gstart[dg] + (j - dstart[dg]);
    if (j < m) p.keys_out[dst[r]] = k;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if ((validmask >> r) & 1u) stage[rank[r]] = val[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t j = t + r * THREADS;
    if (j < m) p.pvals_out[dst[r]] = stage[j];
  }
}

template <int THREADS, int ITEMS>
static void launch_downsweep(const RadixPass& p, dim3 grid, hipStream_t stream) {
  const dim3 block(THREADS);
  if (p.bits <= 5) hipLaunchKernelGGL((radix_downsweep_kernel<THREADS, ITEMS, 5>), grid, block, 0, stream, p);
  else if (p.bits == 6) hipLaunchKernelGGL((radix_downsweep_kernel<THREADS, ITEMS, 6>), grid, block, 0, stream, p);
  else if (p.bits == 7) hipLaunchKernelGGL((radix_downsweep_kernel<THREADS, ITEMS, 7>), grid, block, 0, stream, p);
  else hipLaunchKernelGGL((radix_downsweep_kernel<THREADS, ITEMS, 8>), grid, block, 0, stream, p);
}

hipError_t launch_radix_sort(const RadixSort& s, hipStream_t stream) {
  if (s.nblocks == 0) return hipSuccess;
  if (s.passes < 1 || s.passes > kRadixMaxPasses || s.shape.tile() < 1) return hipErrorInvalidValue;
  for (int k = 0; k < s.passes; ++k) {
    if (s.bits[k] < 1 || s.bits[k] > 8) return hipErrorInvalidValue;
    RadixPass p{};
    p.bits = s.bits[k];
    p.shift = s.shift[k];
    p.filter = k == 0;
    p.span = (uint32_t)s.shape.tile();
    p.nblocks = s.nblocks;
    p.keys_in = k == 0 ? s.keys : s.key_buf[(k + 1) & 1];
    p.vals_in = s.vals;
    p.pvals_in = k == 0 ? nullptr : s.pair_buf[(k + 1) & 1];
    p.keys_out = s.key_buf[k & 1];
    p.pvals_out = s.pair_buf[k & 1];
    p.count_dev = k == 0 ? s.count_dev : s.kept;
    p.count_host = s.count_host;
    p.table = s.table;
    p.totals = s.totals;
    p.count_out = s.kept;
    p.weights = k == 0 ? s.weights : nullptr;
    p.weight_sums = s.weight_sums;
    p.mail = s.mail;
    p.token = s.token;
    p.weight_total = k == 0 ? s.weight_total : nullptr;
    const dim3 grid(s.nblocks);
    hipLaunchKernelGGL(radix_upsweep_kernel, grid, dim3(kRadixThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!radix_own_scan(p)) {
      hipLaunchKernelGGL(radix_scan_kernel, dim3(p.weights && (p.mail || p.weight_total) ? 257 : 256), dim3(kScanThreads), 0, stream, p);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    if (s.shape.threads == 1024)
      launch_downsweep<1024, 16>(p, grid, stream);
    else if (s.shape.threads == 512)
      launch_downsweep<512, 8>(p, grid, stream);
    else
      launch_downsweep<256, 8>(p, grid, stream);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ges
