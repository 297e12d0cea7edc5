// binning.hip -- (tile, splat) pairs of a batch, ordered by (tile, depth, splat index), and tile ranges.
//
// The 3DGS lineage the paper builds on (Sec. 5.2 keeps its design choices) duplicates every splat once
// per tile it covers and sorts the pairs by (tile, depth).  Here the depth part of that order is settled
// once per splat instead of once per pair, and only the tile part is sorted over the pairs:
//   1. depth sort (in ges_preprocess): the listed splats of every view, keyed by the depth bits the
//      preprocess writes, in four stable 8-bit LSD radix passes carrying (candidate count, item); the first
//      pass drops unlisted splats.  Stability keeps equal depths in index order.
//      The first pass also adds up the candidates of all splats and posts the sum to the host, which has the
//      key capacity a frame needs while the sort goes on.
//   2. key scan: every listed splat owns one slot per candidate tile (tile_geom.h), laid out along the
//      depth order; the offset of each 256-splat chunk and the batch's slot count.
//   3. duplicate (render): each wave takes 64 consecutive splats of the depth order, expands their
//      candidates and tests one per lane; every slot receives (batch tile, splat index) or a dropped key.
//      Slots are written in order, so the writes are contiguous.
//   4. tile sort: stable LSD radix passes on the batch tile id (two for up to 65,536 tiles); the first
//      drops the empty slots.  Pairs of one tile keep the depth order of step 3, hence (depth, index).
//   5. ranges: each tile's [start, end) from the boundaries of the sorted tile ids (empty tiles (0, 0)).
// Up to 8,192 items, steps 1 and 2 are one block working in LDS, and up to 8,192 slots so are 4 and 5.
// HBM: per listed splat its record (64 B, gathered in depth order) and a few words; per slot 8 B written
// by the duplication and 12 B read and written per radix pass.
#include <algorithm>

#include "ges_internal.h"
#include "radix_small.h"
#include "tile_geom.h"

namespace ges {

constexpr int kDepthPasses = 4;   // 31 key bits (positive binary32 depths)

// No splat: no sort runs, so nothing else would write the counts.
__global__ void clear_cells_kernel(uint32_t* cells, unsigned long long* mail, uint32_t token) {
  if (threadIdx.x < 4) cells[threadIdx.x] = 0u;
  if (threadIdx.x == 0 && mail) post_count(mail, token, 0ull);
}

// Words a coming render starts from: per view its header (keys, error word, pair statistics) and tile ranges.
__device__ __forceinline__ void clear_views(const DeviceBatch* db, int64_t first, int64_t stride) {
  for (int v = 0; v < db->nviews; ++v) {
    const ViewDesc& V = db->views[v];
    const int64_t T = (int64_t)V.tiles_x * V.tiles_y;
    for (int64_t t = first; t < T; t += stride) V.ranges[t] = make_uint2(0u, 0u);
    if (first < 4) V.header[first] = 0ull;
  }
}

// Up to so many items the chunk sums are not scanned: each block of the duplication adds up those before its own (at most
// 8 per thread), which saves the scan's launch.  The slot count comes from the depth sort then and the views are
// cleared here.  Key scan of 50k to 500k items 10.4 -> 6.4 us, the duplication as before.
constexpr int64_t kUnscannedItems = 2048 * 256;
inline bool chunks_unscanned(const Batch& b) { return b.items > kRadixSmall && b.items <= kUnscannedItems; }

// The depth sort and key scan of up to kRadixSmall items as one block: the keys and their order in LDS.  A
// launch takes about 4.6 us on the stream however little it does, and the general path has ten to fourteen (1k
// splats at 64x64: depth sort and scan 73 -> 16 us, tile sort 24 -> 10).
__global__ void __launch_bounds__(kSmallThreads) small_depth_kernel(const DeviceBatch* __restrict__ db, uint32_t items,
                                                                    const uint32_t* __restrict__ keys,
                                                                    const uint32_t* __restrict__ cand, uint2* order,
                                                                    uint32_t* chunk_off, uint32_t* cells,
                                                                    unsigned long long* mail, uint32_t token) {
  __shared__ SmallSort L;
  __shared__ unsigned long long wave_sum[kSmallThreads / 64];
  __shared__ unsigned long long chunk_sum[kRadixSmall / 256];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  unsigned long long sum = 0;
  for (uint32_t i = t; i < items; i += kSmallThreads) {
    L.key[i] = keys[i];
    L.perm[i] = (uint16_t)i;
    sum += cand[i];   // 0 for an unlisted item
  }
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if (lane == 0) wave_sum[w] = sum;
  __syncthreads();
  sum = 0;
  for (int k = 0; k < kSmallThreads / 64; ++k) sum += wave_sum[k];
  if (t == 0 && mail) post_count(mail, token, sum);   // the host goes on while the sort runs
  uint32_t n = items;
  for (int pass = 0; pass < kDepthPasses; ++pass) n = small_sort_pass(L, n, 8 * pass, 8, pass == 0);
  // the order, and the slots before each chunk of 256 splats of it
  for (uint32_t j0 = 0; j0 < n; j0 += kSmallThreads) {
    const uint32_t j = j0 + t;
    uint32_t c = 0;
    if (j < n) {
      const uint32_t i = L.perm[j];
      c = cand[i];
      order[j] = make_uint2(c, i);
    }
    unsigned long long s = c;
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    __syncthreads();
    if (lane == 0) wave_sum[w] = s;
    __syncthreads();
    if (t < kSmallThreads / 256)
      chunk_sum[j0 / 256 + t] = ((wave_sum[4 * t] + wave_sum[4 * t + 1]) + wave_sum[4 * t + 2]) + wave_sum[4 * t + 3];
  }
  __syncthreads();
  if (t * 256u < n) {
    unsigned long long before = 0;
    for (int k = 0; k < t; ++k) before += chunk_sum[k];
    chunk_off[t] = before > 0xffffffffull ? 0xffffffffu : (uint32_t)before;
  }
  if (t == 0) {
    cells[0] = n;
    cells[1] = sum >= 0xffffffffull ? 0xffffffffu : (uint32_t)sum;
    cells[2] = 0u;
    cells[3] = 0u;
  }
  clear_views(db, threadIdx.x, blockDim.x);
}

hipError_t launch_depth_sort(const DeviceBatch* dbatch, Batch& b, hipStream_t stream) {
  SortWs& w = b.sw;
  w.depth_final = (kDepthPasses - 1) & 1;   // the buffer of the last pass
  if (b.items == 0) {
    hipLaunchKernelGGL(clear_cells_kernel, dim3(1), dim3(64), 0, stream, w.cells, b.mail.slot, b.mail.token);
    return hipGetLastError();
  }
  if (b.items <= kRadixSmall) {
    hipLaunchKernelGGL(small_depth_kernel, dim3(1), dim3(kSmallThreads), 0, stream, dbatch, (uint32_t)b.items,
                       w.item_key, w.item_cand, w.dv[w.depth_final], w.chunk_off, w.cells, b.mail.slot, b.mail.token);
    return hipGetLastError();
  }
  // the values are (candidate count, item) pairs, made by the first pass from the counts and the item
  // indices, so that the key scan and the duplication read the counts in depth order
  RadixSort s{};
  s.passes = kDepthPasses;
  for (int k = 0; k < kDepthPasses; ++k) { s.bits[k] = 8; s.shift[k] = 8 * k; }
  s.keys = w.item_key;
  s.vals = w.item_cand;
  for (int k = 0; k < 2; ++k) { s.key_buf[k] = w.dk[k]; s.pair_buf[k] = w.dv[k]; }
  s.count_host = (uint32_t)b.items;
  s.shape = radix_shape((uint64_t)b.items);
  s.nblocks = s.shape.blocks((uint64_t)b.items);
  s.table = w.table;
  s.totals = w.totals;
  s.kept = &w.cells[0];
  s.weights = w.item_cand;
  s.weight_sums = w.weights;
  s.mail = b.mail.slot;
  s.token = b.mail.token;
  s.weight_total = chunks_unscanned(b) ? &w.cells[1] : nullptr;
  return launch_radix_sort(s, stream);
}

// Which view owns batch item j (linear scan over at most kMaxViews views).
__device__ __forceinline__ int view_of_item(const DeviceBatch* db, int64_t j) {
  return view_of_block(db->item_prefix, db->nviews, j);
}

// Candidate slots of each 256-splat chunk of the depth order (before its exclusive scan).
__global__ void __launch_bounds__(256) chunk_sum_kernel(const DeviceBatch* __restrict__ db, int unscanned,
                                                        const uint2* __restrict__ order, uint32_t* cells,
                                                        uint32_t* chunk_off) {
  __shared__ uint32_t wsum[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t listed = cells[0];
  const int64_t base = (int64_t)blockIdx.x * 256;
  if (unscanned) {
    clear_views(db, base + threadIdx.x, (int64_t)gridDim.x * 256);
    if (blockIdx.x == 0 && threadIdx.x < 2) cells[2 + threadIdx.x] = 0u;
  }
  if (base >= (int64_t)listed) return;   // whole block
  const int64_t k = base + threadIdx.x;
  uint32_t c = k < (int64_t)listed ? order[k].x : 0u;
  for (int off = 32; off > 0; off >>= 1) c += (uint32_t)__shfl_xor((int)c, off, 64);
  if (lane == 0) wsum[w] = c;
  __syncthreads();
  if (threadIdx.x == 0) chunk_off[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// One block: exclusive scan of the chunk sums (saturating at 2^32 - 1, which the host reports as
// capacity exceeded); the batch's slot count into cells[1]; the per-view header words and ranges cleared
// for the coming render.  Each thread scans kPer consecutive sums of a round in registers, so a round takes
// one block-wide scan of the thread totals.
__global__ void __launch_bounds__(1024) chunk_scan_kernel(const DeviceBatch* __restrict__ db, uint32_t* chunk_off,
                                                          uint32_t* cells) {
  constexpr int kPer = 8;
  __shared__ unsigned long long wsum[16];
  __shared__ unsigned long long carry;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t listed = cells[0];
  const int64_t nchunks = ((int64_t)listed + 255) / 256;
  if (threadIdx.x == 0) carry = 0ull;
  __syncthreads();
  for (int64_t base = 0; base < nchunks; base += 1024 * kPer) {
    const int64_t c0 = base + (int64_t)threadIdx.x * kPer;   // this thread's kPer consecutive entries
    uint32_t x[kPer];
    unsigned long long local = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      x[k] = c0 + k < nchunks ? chunk_off[c0 + k] : 0u;
      local += x[k];
    }
    unsigned long long s = local;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned long long y = __shfl_up(s, d, 64);
      if (lane >= d) s += y;
    }
    if (lane == 63) wsum[wid] = s;
    __syncthreads();
    unsigned long long run = carry + s - local;
    for (int q = 0; q < wid; ++q) run += wsum[q];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (c0 + k < nchunks) chunk_off[c0 + k] = run > 0xffffffffull ? 0xffffffffu : (uint32_t)run;
      run += x[k];
    }
    __syncthreads();
    if (threadIdx.x == 1023) carry = run;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    cells[1] = carry >= 0xffffffffull ? 0xffffffffu : (uint32_t)carry;
    cells[2] = 0u;
    cells[3] = 0u;
  }
  clear_views(db, threadIdx.x, blockDim.x);
}

hipError_t launch_key_scan(const DeviceBatch* dbatch, const Batch& b, hipStream_t stream) {
  const SortWs& w = b.sw;
  if (b.items > 0 && b.items <= kRadixSmall) return hipSuccess;   // part of the depth sort
  const int64_t chunks = (b.items + 255) / 256;
  if (chunks > 0) {
    hipLaunchKernelGGL(chunk_sum_kernel, dim3((unsigned)chunks), dim3(256), 0, stream, dbatch, chunks_unscanned(b) ? 1 : 0,
                       w.dv[w.depth_final], w.cells, w.chunk_off);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || chunks_unscanned(b)) return e;
  }
  hipLaunchKernelGGL(chunk_scan_kernel, dim3(1), dim3(1024), 0, stream, dbatch, w.chunk_off, w.cells);
  return hipGetLastError();
}

// Per-wave LDS staging of 64 splats and of 64 of their tile rows for the flattened candidate walk.
struct __attribute__((aligned(16))) WaveSplats {
  float4 conic[64];      // u, v, a, b
  float4 edge[64];       // c, 1/a, 1/c, q_max
  uint4 at[64];          // splat index in its view, the view's first batch tile, its tiles per row, width | height << 16
  uint4 row[64];         // the current rows that have candidates: owning splat (lane), tile row, column less position, -
  uint32_t rexcl[64];    // exclusive prefix of the splats' tile rows
  uint32_t filled[64];   // candidates enumerated so far (checked against the splat's slots)
  uint32_t hits[64];
  int32_t tx0[64], tx1[64], ty0[64];
  uint32_t spans[64];
  float q2[64], det[64], Xe[64], Y[64], ra[64];
  uint32_t begins[64];   // of the 64 candidates at hand, the first ones of their rows
};

__device__ __forceinline__ void dup_wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Last index j in [0, 64) with ex[j] <= x (ex non-decreasing, ex[0] = 0 <= x).
__device__ __forceinline__ int owner_of(const uint32_t* ex, uint32_t x) {
  int j = 0;
#pragma unroll
  for (int step = 32; step > 0; step >>= 1)
    if (ex[j + step] <= x) j += step;
  return j;
}

// Each wave takes 64 consecutive splats of the depth order and fills their slots: the splats' tile rows are
// flattened 64 at a time (each lane computes one row's span of candidate columns), then the candidates of
// those rows 64 at a time, one per lane; each slot receives (batch tile, splat index) when the exact test
// admits the tile (always for SQUARE), else a dropped key.  Also per splat its tile count and visibility
// bit, and per view its number of keys.  What bounds it is VALU issue, the exact test above all; a candidate finds its
// row by the rows that began up to it (a ballot, where a search of the rows' prefix took six dependent reads), reads its
// splat 16 bytes at a time, and hits are counted by the lanes that own the rows, from the ballot of a batch, not by
// an atomic per candidate: 169M slots 1252 -> 995 us, 5M of large splats 162 -> 117, 13.5M 140 -> 128.
template <bool PACK>
__global__ void __launch_bounds__(256) duplicate_kernel(DeviceBatch* __restrict__ db, const ViewPack pack,
                                                        const uint2* __restrict__ order,
                                                        const uint32_t* __restrict__ chunk_off, int unscanned,
                                                        uint32_t* cells, uint32_t* keys, uint32_t* vals, uint64_t capacity,
                                                        int ellipse) {
  __shared__ WaveSplats wave_lds[4];
  __shared__ uint32_t view_keys[kMaxViews];
  __shared__ uint32_t wave_total[4];
  __shared__ unsigned long long chunks_before[4];   // slots of the chunks before the block's, by wave
  const Views<PACK> views{db, pack};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (PACK && blockIdx.x == 0) write_views(db, pack);
  for (int v = threadIdx.x; v < kMaxViews; v += 256) view_keys[v] = 0u;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const uint32_t slots = cells[1];
    cells[3] = (uint64_t)slots > capacity ? (uint32_t)capacity : slots;   // slots written below
    if ((uint64_t)slots > capacity) atomicOr(&views[0].header[1], 1ull);
  }
  __syncthreads();
  const uint32_t listed = cells[0];
  if (unscanned && (int64_t)blockIdx.x * 256 < (int64_t)listed) {
    unsigned long long before = 0;
    for (uint32_t c = threadIdx.x; c < blockIdx.x; c += 256) before += chunk_off[c];
    for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, 64);
    if (lane == 0) chunks_before[wave] = before;
  }
  const int64_t chunk = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;   // 64 splats per wave
  WaveSplats& W = wave_lds[wave];
  int v = 0;
  int64_t i = 0;
  uint32_t nslots = 0u, nrows = 0u;
  bool live = false;
  uint32_t flags = 0u;
  const bool busy = chunk * 64 < (int64_t)listed;   // wave-uniform
  if (busy) {
    const int64_t k = chunk * 64 + lane;
    if (k < (int64_t)listed) {
      const uint2 cj = order[k];   // (candidate count, item)
      const uint32_t j = cj.y;
      v = PACK ? (int)(j / (uint32_t)pack.items) : view_of_item(db, j);
      const ViewDesc& V = views[v];
      i = (int64_t)j - (PACK ? v * pack.items : db->item_prefix[v]);
      const float4 r3 = V.rec[4 * i + 3];
      const uint32_t lo = __float_as_uint(r3.y), hi = __float_as_uint(r3.z);
      flags = (uint32_t)__float_as_int(r3.x) >> 24;
      const float4 r0 = V.rec[4 * i + 0];
      const float4 r1 = V.rec[4 * i + 1];
      SplatTiles s;
      candidate_tiles(r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, (int)(lo & 0xffffu), (int)(lo >> 16), (int)(hi & 0xffffu),
                      (int)(hi >> 16), ellipse != 0, s);
      live = true;
      // the splat's slots are the ones the key scan counted (the preprocess ran candidate_count on the same
      // values); its rows are enumerated until they are filled
      nslots = cj.x;
      nrows = nslots ? s.rows : 0u;
      W.filled[lane] = 0u;
      W.tx0[lane] = s.tx0; W.tx1[lane] = s.tx1; W.ty0[lane] = s.ty0;
      W.spans[lane] = s.spans ? 1u : 0u;
      W.conic[lane] = make_float4(s.u, s.v, s.a, s.b);
      W.edge[lane] = make_float4(s.c, s.inv_a, s.inv_c, s.qm);
      W.at[lane] = make_uint4((uint32_t)i, (uint32_t)(PACK ? v * pack.tiles : db->tile_prefix[v]), (uint32_t)V.tiles_x,
                              (uint32_t)(V.width | (V.height << 16)));
      W.q2[lane] = s.q2; W.det[lane] = s.det; W.Xe[lane] = s.Xe; W.Y[lane] = s.Y; W.ra[lane] = s.ra;
    }
  }
  // slots of the wave's splats: the block's offset (one 256-splat chunk) plus the earlier waves' counts
  uint32_t sincl = nslots, rincl = nrows;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)sincl, d, 64);
    const uint32_t z = (uint32_t)__shfl_up((int)rincl, d, 64);
    if (lane >= d) { sincl += y; rincl += z; }
  }
  // wave totals as scalars: the loops below then keep their control on the scalar unit
  const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane(__shfl((int)sincl, 63, 64));
  const uint32_t rtotal = (uint32_t)__builtin_amdgcn_readfirstlane(__shfl((int)rincl, 63, 64));
  if (lane == 0) wave_total[wave] = total;
  __syncthreads();
  if (busy) {
    W.rexcl[lane] = rincl - nrows;
    W.hits[lane] = 0u;
    dup_wave_fence();
    uint64_t slot0 = unscanned ? (chunks_before[0] + chunks_before[1]) + (chunks_before[2] + chunks_before[3])
                               : chunk_off[blockIdx.x];
    for (int q = 0; q < wave; ++q) slot0 += wave_total[q];
    uint32_t done = 0;   // slots filled by the rows before this round
    for (uint32_t r0 = 0; r0 < rtotal; r0 += 64) {
      // one tile row per lane: its span of candidate columns
      const uint32_t r = r0 + (uint32_t)lane;
      uint32_t width = 0u;
      int j = 0, ty = 0, clo = 0;
      if (r < rtotal) {
        j = owner_of(W.rexcl, r);
        ty = W.ty0[j] + (int)(r - W.rexcl[j]);
        SplatTiles s;
        s.tx0 = W.tx0[j]; s.tx1 = W.tx1[j]; s.ty0 = W.ty0[j];
        s.spans = W.spans[j] != 0u;
        const float4 conic = W.conic[j], edge = W.edge[j];
        s.u = conic.x; s.v = conic.y; s.a = conic.z; s.b = conic.w;
        s.c = edge.x; s.inv_a = edge.y; s.inv_c = edge.z; s.qm = edge.w;
        s.q2 = W.q2[j]; s.det = W.det[j]; s.Xe = W.Xe[j]; s.Y = W.Y[j];
        s.ra = W.ra[j];
        int chi;
        row_span(s, ty, (int)(W.at[j].w >> 16), clo, chi);
        width = chi >= clo ? (uint32_t)(chi - clo + 1) : 0u;
      }
      uint32_t wincl = width;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)wincl, d, 64);
        if (lane >= d) wincl += y;
      }
      const uint32_t ctotal = (uint32_t)__builtin_amdgcn_readfirstlane(__shfl((int)wincl, 63, 64));
      const uint32_t wexcl = wincl - width;
      const uint64_t some = __ballot(width != 0u);   // the rows that have candidates, listed without gaps
      if (width) {
        W.row[__builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u))] =
            make_uint4((uint32_t)j, (uint32_t)ty, (uint32_t)clo - wexcl, 0u);
        atomicAdd(&W.filled[j], width);
      }
      uint32_t row_hits = 0u;
      for (uint32_t c0 = 0; c0 < ctotal; c0 += 64) {
        const uint32_t c = c0 + (uint32_t)lane;
        // a candidate's row: as many as began up to it
        W.begins[lane] = 0u;
        dup_wave_fence();
        if (width && wexcl - c0 < 64u) W.begins[wexcl - c0] = 1u;
        dup_wave_fence();
        const uint64_t begins = __ballot(W.begins[lane] != 0u);
        const uint32_t before = (uint32_t)__popcll(__ballot(width && wexcl < c0));
        const uint32_t q = before - 1u + ((uint32_t)(begins >> lane) & 1u) +
                           __builtin_amdgcn_mbcnt_hi((uint32_t)(begins >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)begins, 0u));
        const uint32_t pos = done + c;   // position among the wave's slots
        bool hit = false;
        if (c < ctotal && pos < total) {
          const uint4 row = W.row[q];
          const int js = (int)row.x, tyy = (int)row.y, txx = (int)(row.z + c);
          const uint4 at = W.at[js];
          const float4 conic = W.conic[js], edge = W.edge[js];
          hit = !ellipse || ellipse_hits_tile(conic.x, conic.y, conic.z, conic.w, edge.x, edge.y, edge.z, edge.w, txx, tyy,
                                              (int)(at.w & 0xffffu), (int)(at.w >> 16));
          const uint64_t slot = slot0 + pos;
          if (slot < capacity) {
            keys[slot] = hit ? at.y + (uint32_t)(tyy * (int)at.z + txx) : kNoKey;
            vals[slot] = at.x;
          }
        }
        // the hits among this lane's row's candidates
        const uint64_t mask = __ballot(hit);
        const int lo = max((int)wexcl - (int)c0, 0), hi = min((int)wincl - (int)c0, 64);
        if (lo < hi) row_hits += (uint32_t)__popcll((mask >> lo) & (~0ull >> (64 - (hi - lo))));
      }
      if (row_hits) atomicAdd(&W.hits[j], row_hits);
      done += ctotal;
      dup_wave_fence();
    }
    if (live && W.filled[lane] != nslots) atomicOr(&views[0].header[1], 2ull);   // never expected
    if (live) {
      // the preprocess left the candidate count in tiles_touched and the visibility bit set when it is
      // non-zero: rewrite them only where the exact count differs (scattered 4-byte stores)
      const ViewDesc& V = views[v];
      const uint32_t h = W.hits[lane];
      if (h != nslots) reinterpret_cast<uint32_t*>(V.rec)[16 * i + R_TOUCHED] = h;
      if (h == 0u && nslots != 0u) V.vis[i] = flags;
      const uint64_t first = slot0 + (sincl - nslots);   // the splat's first slot (its rows in the backward)
      V.slot_off[i] = first > 0xffffffffull ? 0xffffffffu : (uint32_t)first;
      if (h) atomicAdd(&view_keys[v], h);
    }
  }
  __syncthreads();
  for (int vv = threadIdx.x; vv < views.count(); vv += 256)
    if (view_keys[vv]) atomicAdd(&views[vv].header[0], (unsigned long long)view_keys[vv]);
}

hipError_t launch_duplicate(DeviceBatch* dbatch, const Batch& b, hipStream_t stream) {
  const SortWs& w = b.sw;
  const int64_t chunks = (b.items + 255) / 256;
  if (chunks == 0 || b.key_capacity == 0) return launch_views(dbatch, b, stream);
  const int X = b.dup_buffer;
  auto kernel = b.pack ? duplicate_kernel<true> : duplicate_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)chunks), dim3(256), 0, stream, dbatch, b.pack ? *b.pack : ViewPack{},
                     w.dv[w.depth_final], w.chunk_off, chunks_unscanned(b) ? 1 : 0, w.cells, b.kw.key[X],
                     reinterpret_cast<uint32_t*>(b.kw.pv[X]),
                     b.key_capacity, b.tile_cull == GES_TILES_ELLIPSE ? 1 : 0);
  return hipGetLastError();
}

// After the backward raster: each splat's 2-D gradient, the sum of the rows the raster stored at its
// candidate slots (one per tile in which some pixel composited it; about a tenth of the slots, as the tiles'
// walks end where their pixels saturate), added in binary64 in slot order -- the same order on every run,
// so the backward is deterministic.  A wave takes 8 or 32 words of the row marks (32 slots each): it lists their marked
// slots in LDS, loads 64 rows at a time (one per lane; a row carries its splat's batch item and first
// candidate slot) and each run of one splat's rows is added from LDS, carrying an unfinished run into the next 64
// and, past the wave's words, through the rest of the splat's slot range.
// The run at the start of the range belongs to the wave holding the splat's first row if that lies before
// the range.  The splat's 2-D gradient is written and kRowBit set in its visibility word (the preprocess
// backward takes zero without it).
//
// What bounds it is the latency of a wave's steps and, of those, the sums.  A chunk of 64 rows with many runs (splats
// of one or two rows) is added a run per lane; one with few runs a component per lane, 6 runs of 10 at a time, or
// the few lanes with a run would add ten numbers per row, one row after the other.
// Both add in the same order.  A run per lane for every chunk, and 8 words per wave for every frame, took 587 us for
// 169M slots, 215 for 5M of large splats, 102 for 13.5M and 77 for 3.9M; now 251, 59, 65 and 42.
constexpr uint32_t kNoItem = 0xffffffffu;
// More slots than this: ranges of 32 words per wave, as a tenth of the slots of such a frame has a row and a wave should
// have some tens of them.  8 words against 32: 169M slots 422 / 251 us, 35M 138 / 88, 21M 103 / 70; where most slots have a
// row, 24M 208 / 194, 12M 144 / 152, 6M 95 / 122, 5M of large splats 59 / 72.
constexpr uint64_t kReduceWide = 1ull << 25;
constexpr int kReduceRuns = 6;        // runs that are added together, a component per lane
constexpr int kReduceFew = 2 * kReduceRuns;   // up to so many runs in 64 rows (1M splats: 6 43, 12 42, 24 42 us; 50k: 19, 19, 25)

template <int WORDS>
struct ReduceLds {
  uint32_t slot[WORDS * 32];          // marked slots, in order
  float row[64][kRowFloats];          // the current 64 rows
  uint32_t owner[64];
  uint32_t start[64 + 1];             // first rows of the runs, and the end of the last
  double carry[10];                   // sums of the run left open by the last 64 rows
  uint32_t carry_owner;
};

__device__ __forceinline__ void reduce_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double* grad2d_of(const DeviceBatch* db, uint32_t item, uint32_t*& vis) {
  const int v = view_of_item(db, item);
  const ViewDesc& V = db->views[v];
  const int64_t i = (int64_t)item - db->item_prefix[v];
  vis = V.vis + i;
  return V.grad2d + (int64_t)kGradStride * i;
}

__device__ __forceinline__ void write_grad2d(const DeviceBatch* db, uint32_t item, const double* g) {
  uint32_t* vis;
  double2* gs = reinterpret_cast<double2*>(grad2d_of(db, item, vis));
#pragma unroll
  for (int c = 0; c < 5; ++c) gs[c] = make_double2(g[2 * c], g[2 * c + 1]);
  __hip_atomic_fetch_or(vis, kRowBit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Component c of it, by the lane that has it.
__device__ __forceinline__ void write_grad2d(const DeviceBatch* db, uint32_t item, int c, double g) {
  uint32_t* vis;
  grad2d_of(db, item, vis)[c] = g;
  if (c == 0) __hip_atomic_fetch_or(vis, kRowBit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The marked slots of words [w0, w0 + WORDS) below `end` into L.slot, in order; returns their count.
template <int WORDS>
__device__ __forceinline__ uint32_t list_marks(const GlobalU32* bits, uint64_t w0, uint64_t nwords, uint64_t end,
                                               ReduceLds<WORDS>& L, int lane) {
  const uint64_t q = w0 + (uint64_t)lane;
  uint32_t m = 0u;
  if (lane < WORDS && q < nwords && q * 32 < end) {
    m = bits[q];
    if (end - q * 32 < 32) m &= (1u << (uint32_t)(end - q * 32)) - 1u;
  }
  const uint32_t cnt = (uint32_t)__builtin_popcount(m);
  uint32_t incl = cnt;
#pragma unroll
  for (int d = 1; d < WORDS; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)incl, d, 64);
    if (lane >= d) incl += y;
  }
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, WORDS - 1);
  uint32_t p = incl - cnt;
  while (m) {
    L.slot[p++] = (uint32_t)(q * 32) + (uint32_t)__builtin_ctz(m);
    m &= m - 1u;
  }
  reduce_fence();
  return total;
}

// Lane-per-row load of rows [c0, c0 + n) of the list into LDS; returns the lane's row's item and first slot.
template <int WORDS>
__device__ __forceinline__ void load_rows(const GlobalVec4* rows, ReduceLds<WORDS>& L, uint32_t c0, uint32_t n, int lane,
                                          uint32_t& item, uint32_t& first) {
  item = kNoItem;
  first = 0u;
  if ((uint32_t)lane < n) {
    const GlobalVec4* r = rows + (uint64_t)L.slot[c0 + lane] * (kRowFloats / 4);
    const Vec4 a0 = r[0], a1 = r[1], a2 = r[2];
    item = __float_as_uint(a2[2]);
    first = __float_as_uint(a2[3]);
    Vec4* to = reinterpret_cast<Vec4*>(L.row[lane]);
    to[0] = a0;
    to[1] = a1;
    to[2] = a2;
  }
  L.owner[lane] = item;
}

template <int WORDS>
__global__ void __launch_bounds__(256) row_reduce_kernel(const DeviceBatch* __restrict__ db,
                                                         const float* __restrict__ rows_,
                                                         const uint32_t* __restrict__ bits_, uint64_t nslots) {
  __shared__ __align__(16) ReduceLds<WORDS> lds[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  ReduceLds<WORDS>& L = lds[wave];
  const uint64_t nwords = (nslots + 31) / 32;
  const uint64_t w0 = ((uint64_t)blockIdx.x * 4 + wave) * WORDS;
  if (w0 >= nwords) return;
  const uint64_t wend = min<uint64_t>((w0 + WORDS) * 32, nslots);   // first slot after the range
  const GlobalU32* bits = (const GlobalU32*)bits_;
  const GlobalVec4* rows = (const GlobalVec4*)rows_;
  const uint32_t total = list_marks(bits, w0, nwords, wend, L, lane);
  if (total == 0) return;
  if (lane == 0) L.carry_owner = kNoItem;
  uint32_t skip = kNoItem;
  const int run = lane / 10, comp = lane - 10 * run;   // a component per lane
  for (uint32_t c0 = 0; c0 < total; c0 += 64) {
    const uint32_t n = min<uint32_t>(64u, total - c0);
    uint32_t o, lo;
    load_rows(rows, L, c0, n, lane, o, lo);
    if (c0 == 0) {
      // the first run's splat is summed by the wave of its first row: is that before this range?
      const uint32_t o0 = (uint32_t)__shfl((int)o, 0, 64);
      const uint64_t lo0 = (uint32_t)__shfl((int)lo, 0, 64);
      bool earlier = false;
      for (uint64_t q0 = lo0 >> 5; q0 < w0 && !earlier; q0 += 64) {
        const uint64_t q = q0 + (uint64_t)lane;
        uint32_t m = 0u;
        if (q < w0) {
          m = bits[q];
          if (q == lo0 >> 5) m &= ~0u << (uint32_t)(lo0 & 31u);
        }
        earlier = __ballot(m != 0u) != 0ull;
      }
      if (earlier) skip = o0;
    }
    reduce_fence();
    const uint32_t co = L.carry_owner;
    // a run left open by the previous 64 rows goes on here, or ended with them
    const bool goes_on = co != kNoItem && co == L.owner[0];
    if (co != kNoItem && !goes_on && lane < 10) write_grad2d(db, co, lane, L.carry[lane]);
    const bool head = (uint32_t)lane < n && (lane == 0 || L.owner[lane - 1] != o);
    const uint64_t heads = __ballot(head);
    const uint32_t nruns = (uint32_t)__builtin_popcountll(heads);
    if (head)
      L.start[__builtin_amdgcn_mbcnt_hi((uint32_t)(heads >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)heads, 0u))] = lane;
    if (lane == 0) L.start[nruns] = n;
    reduce_fence();
    if (nruns <= (uint32_t)kReduceFew) {
      for (uint32_t r0 = 0; r0 < nruns; r0 += kReduceRuns) {
        const uint32_t r = r0 + (uint32_t)run;
        if (run < kReduceRuns && r < nruns) {
          const uint32_t k0 = L.start[r], k1 = L.start[r + 1], ow = L.owner[k0];
          double g = r == 0 && goes_on ? L.carry[comp] : 0.0;
          if (ow != skip) {
#pragma unroll 4
            for (uint32_t k = k0; k < k1; ++k) g += (double)L.row[k][comp];
          }
          if (k1 == n) {
            L.carry[comp] = g;
            if (comp == 0) L.carry_owner = ow == skip ? kNoItem : ow;
          } else if (ow != skip) {
            write_grad2d(db, ow, comp, g);
          }
        }
      }
    } else if (head) {
      double g[10];
#pragma unroll
      for (int k = 0; k < 10; ++k) g[k] = lane == 0 && goes_on ? L.carry[k] : 0.0;
      uint32_t k = (uint32_t)lane;
      if (o != skip) {
        for (; k < n && L.owner[k] == o; ++k) {
#pragma unroll
          for (int c = 0; c < 10; ++c) g[c] += (double)L.row[k][c];
        }
      } else {
        while (k < n && L.owner[k] == o) ++k;
      }
      if (k == n) {
#pragma unroll
        for (int c = 0; c < 10; ++c) L.carry[c] = g[c];
        L.carry_owner = o == skip ? kNoItem : o;
      } else if (o != skip) {
        write_grad2d(db, o, g);
      }
    }
    reduce_fence();
  }
  // the last run: finished here, or continued through the rest of its splat's slots
  const uint32_t co = L.carry_owner;
  if (co == kNoItem) return;
  double g = lane < 10 ? L.carry[lane] : 0.0;
  uint64_t hi;
  {
    const int v = view_of_item(db, co);
    const ViewDesc& V = db->views[v];
    const int64_t i = (int64_t)co - db->item_prefix[v];
    hi = min<uint64_t>((uint64_t)V.slot_off[i] + V.item_cand[i], nslots);
  }
  for (uint64_t q0 = w0 + WORDS; q0 * 32 < hi; q0 += WORDS) {
    reduce_fence();
    const uint32_t cnt = list_marks(bits, q0, nwords, hi, L, lane);
    for (uint32_t c0 = 0; c0 < cnt; c0 += 64) {
      const uint32_t n = min<uint32_t>(64u, cnt - c0);
      uint32_t o, lo;
      load_rows(rows, L, c0, n, lane, o, lo);
      reduce_fence();
      if (lane < 10) {
#pragma unroll 4
        for (uint32_t k = 0; k < n; ++k) g += (double)L.row[k][lane];
      }
      reduce_fence();
    }
  }
  if (lane < 10) write_grad2d(db, co, lane, g);
}

hipError_t launch_row_reduce(const DeviceBatch* dbatch, const Batch& b, const float* rows, const uint32_t* bits,
                             uint64_t nslots, hipStream_t stream) {
  (void)b;
  if (nslots == 0) return hipSuccess;
  const uint64_t nwords = (nslots + 31) / 32;
  if (nslots > kReduceWide)
    hipLaunchKernelGGL(row_reduce_kernel<32>, dim3((unsigned)((nwords + 127) / 128)), dim3(256), 0, stream, dbatch, rows,
                       bits, nslots);
  else
    hipLaunchKernelGGL(row_reduce_kernel<8>, dim3((unsigned)((nwords + 31) / 32)), dim3(256), 0, stream, dbatch, rows,
                       bits, nslots);
  return hipGetLastError();
}

// Tile ranges from the boundaries of the sorted tile ids (ranges were cleared by the key scan).  Each thread
// reads 4 consecutive ids as one 16-byte load; the ids either side come from the neighbouring lanes.
__global__ void __launch_bounds__(256) tile_ranges_kernel(const DeviceBatch* __restrict__ db,
                                                          const uint32_t* __restrict__ tiles,
                                                          const uint32_t* __restrict__ cells, int64_t total_tiles) {
  const uint64_t K = cells[2];
  const int lane = threadIdx.x & 63;
  const uint64_t k0 = ((uint64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (k0 - 4 * (uint64_t)lane >= K) return;   // the whole wave lies past the keys
  uint32_t t[4] = {~0u, ~0u, ~0u, ~0u};
  if (k0 + 4 <= K) {
    const uint4 q = reinterpret_cast<const uint4*>(tiles)[k0 >> 2];
    t[0] = q.x; t[1] = q.y; t[2] = q.z; t[3] = q.w;
  } else {
    for (int e = 0; e < 4; ++e)
      if (k0 + e < K) t[e] = tiles[k0 + e];
  }
  uint32_t prev = (uint32_t)__shfl_up((int)t[3], 1, 64), next = (uint32_t)__shfl_down((int)t[0], 1, 64);
  if (lane == 0) prev = k0 > 0 && k0 <= K ? tiles[k0 - 1] : ~0u;
  if (lane == 63) next = k0 + 4 < K ? tiles[k0 + 4] : ~0u;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint64_t k = k0 + e;
    if (k >= K) break;
    const uint32_t tt = t[e];
    if ((int64_t)tt >= total_tiles) continue;   // not a tile of the batch (never written by the duplication)
    const uint32_t before = e == 0 ? prev : t[e - 1];
    const uint32_t after = e == 3 ? next : t[e + 1];
    const bool first = k == 0 || before != tt;
    const bool last = k + 1 == K || after != tt;
    if (!first && !last) continue;
    const int v = view_of_block(db->tile_prefix, db->nviews, (int64_t)tt);
    uint2* r = db->views[v].ranges + ((int64_t)tt - db->tile_prefix[v]);
    if (first) r->x = (uint32_t)k;
    if (last) r->y = (uint32_t)(k + 1);
  }
}

// The tile sort of up to kRadixSmall slots and its ranges as one block (see small_depth_kernel).  The last
// buffer may be the one the duplication wrote: everything read from it is read before the first write.
__global__ void __launch_bounds__(kSmallThreads) small_tile_kernel(const DeviceBatch* __restrict__ db, uint32_t* cells,
                                                                   int tile_bits, int passes, const uint32_t* keys,
                                                                   const uint32_t* ids, uint32_t* keys_out,
                                                                   uint2* pairs_out, int64_t total_tiles) {
  __shared__ SmallSort L;
  const int t = threadIdx.x;
  uint32_t n = min(cells[3], kRadixSmall);
  for (uint32_t i = t; i < n; i += kSmallThreads) {
    L.key[i] = keys[i];
    L.perm[i] = (uint16_t)i;
  }
  __syncthreads();
  int shift = 0;
  for (int pass = 0; pass < passes; ++pass) {
    const int left = passes - pass, bits = (tile_bits - shift + left - 1) / left;
    n = small_sort_pass(L, n, shift, bits, pass == 0);
    shift += bits;
  }
  uint32_t id[kRadixSmall / kSmallThreads];
#pragma unroll
  for (uint32_t r = 0; r < kRadixSmall / kSmallThreads; ++r) {
    const uint32_t j = r * kSmallThreads + t;
    id[r] = j < n ? ids[L.perm[j]] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < kRadixSmall / kSmallThreads; ++r) {
    const uint32_t j = r * kSmallThreads + t;
    if (j >= n) break;
    const uint32_t tile = L.key[j];
    keys_out[j] = tile;
    pairs_out[j] = make_uint2(id[r], L.perm[j]);
    if ((int64_t)tile >= total_tiles) continue;   // not a tile of the batch (never written by the duplication)
    const bool first = j == 0 || L.key[j - 1] != tile, last = j + 1 == n || L.key[j + 1] != tile;
    if (!first && !last) continue;
    const int v = view_of_block(db->tile_prefix, db->nviews, (int64_t)tile);
    uint2* g = db->views[v].ranges + ((int64_t)tile - db->tile_prefix[v]);
    if (first) g->x = j;
    if (last) g->y = j + 1;
  }
  if (t == 0) cells[2] = n;
}

hipError_t launch_tile_sort(const DeviceBatch* dbatch, const Batch& b, hipStream_t stream) {
  if (b.key_capacity == 0 || b.items == 0) return hipSuccess;   // no pair: the ranges are clear
  const SortWs& w = b.sw;
  const KeyWs& k = b.kw;
  const int X = b.dup_buffer;
  if (((X + b.tile_passes) & 1) != 0 || b.tile_passes > kRadixMaxPasses) return hipErrorInvalidValue;
  // the tile bits split evenly over the passes (13 bits: 7 + 6), so that no pass scatters to more digit
  // runs than it must
  int bits = 1;
  while (bits < 32 && ((int64_t)1 << bits) < b.total_tiles) ++bits;
  if (b.key_capacity <= kRadixSmall) {
    hipLaunchKernelGGL(small_tile_kernel, dim3(1), dim3(kSmallThreads), 0, stream, dbatch, w.cells, bits,
                       b.tile_passes, k.key[X], reinterpret_cast<const uint32_t*>(k.pv[X]), k.key[0], k.pv[0],
                       b.total_tiles);
    return hipGetLastError();
  }
  RadixSort s{};
  s.passes = b.tile_passes;
  int shift = 0;
  for (int pass = 0; pass < s.passes; ++pass) {
    const int left = s.passes - pass;
    s.bits[pass] = (bits - shift + left - 1) / left;
    s.shift[pass] = shift;
    shift += s.bits[pass];
  }
  s.keys = k.key[X];
  s.vals = reinterpret_cast<const uint32_t*>(k.pv[X]);   // the first pass pairs each splat index with its slot
  for (int e = 0; e < 2; ++e) { s.key_buf[e] = k.key[X ^ 1 ^ e]; s.pair_buf[e] = k.pv[X ^ 1 ^ e]; }
  s.count_dev = &w.cells[3];
  s.shape = radix_shape(b.key_capacity);
  s.nblocks = s.shape.blocks(b.key_capacity);
  s.table = k.table;
  s.totals = k.totals;
  s.kept = &w.cells[2];
  hipError_t e = launch_radix_sort(s, stream);
  if (e != hipSuccess) return e;
  const uint64_t rblocks = (b.key_capacity + 1023) / 1024;
  hipLaunchKernelGGL(tile_ranges_kernel, dim3((unsigned)rblocks), dim3(256), 0, stream, dbatch,
                     k.key[0], w.cells, b.total_tiles);
  return hipGetLastError();
}

}  // namespace ges
