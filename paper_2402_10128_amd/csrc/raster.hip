// raster.hip -- per-tile front-to-back compositing of GES splats and its reverse-mode pass.
//
// Compositing is the discrete form of the volume-rendering integral (GES Sec. 4.2, Eq. transimttance):
// for every pixel, over its tile's splats in (depth, index) order,
//   q = a dx^2 + 2 b dx dy + c dy^2 with (dx,dy) = mean2D - pixel centre   (binary32, fixed order:
//       t = fma(a, dx, (2b) dy); q = fma(t, dx, (c dy) dy) -- identical on every machine)
//   skip unless q <= q_max (alpha >= 1/255);   falloff G = exp(-q/2) (PHI) or exp(-q^(beta/2)/2) (GEF)
//   alpha = min(0.99, o G);  t = T (1 - alpha);  stop before compositing when t < 1e-4
//   C += alpha T rgb;  T = t.
// Launch shape (gfx950): the forward pass gives a 16x16 tile four wave64s, one 8x8 quadrant each with one pixel
// per lane; a wave skips the splats that cannot reach its quadrant (see raster_forward_kernel).  The backward
// pass, whose issue rate is saturated on large frames, keeps one wave per tile with 4 pixels per lane (rows
// y, y+4, y+8, y+12), so each splat read from LDS is used four times per lane.  Records are staged in LDS and
// read back as broadcasts.  A wave stops as soon as no lane has a live pixel; the forward block once no wave
// has.  Tiles are dealt to the 8 XCDs in groups of 8 neighbours (see xcd_tile).
// The backward pass walks each pixel's contributors back to front, recovering the transmittance
// before splat j as T_j = T_(j+1) / (1 - alpha_j) from the stored final T, so no per-pixel lists are
// kept.  A long walk is cut into segments that several waves take at once (a wave needs about 0.5 us per splat,
// and a 64x64 frame has 16 tiles): backward_prepare_kernel plans them and raster_recover_kernel leaves the
// state at their boundaries.
// Per splat, the 4 pixels of a lane are summed in registers and each row of 16 lanes by a DPP
// reduce-scatter; the row's lanes park the row sums in LDS, and every 32 splats each lane finishes one
// parked splat (4 row sums) and stores the tile's ten sums of the splat as a row at the pair's candidate
// slot, marking the slot; a row reduction then adds each splat's rows in binary64 in slot order (the
// cross-tile sums of a splat often cancel; binary32 accumulation would lose accuracy there), with no
// atomics, so the backward is deterministic.
// Factors of 2 common to a splat's terms (the mean2D and b gradients) are applied once per (tile, splat).
#include <type_traits>

#include "ges_internal.h"

namespace ges {

constexpr float kNegHalfLog2e = -0.72134752044448170368f;   // -log2(e)/2: exp(-q/2) = 2^(kNegHalfLog2e q)

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// max(q, 0) for q that is not NaN, as one integer max of the bits (a negative q, -0 included, has a negative
// bit pattern); fmaxf costs a canonicalisation besides under IEEE mode.
__device__ __forceinline__ float clamp_q(float q) { return __int_as_float(max(__float_as_int(q), 0)); }

__device__ __forceinline__ float pair_q(float u, float v, float a, float bb, float c, float px, float py,
                                        float& dx, float& dy) {
  dx = u - px;
  dy = v - py;
  float t = bb * dy;
  t = __builtin_fmaf(a, dx, t);
  float w = c * dy;
  w = w * dy;
  return __builtin_fmaf(t, dx, w);
}

// Map a block to a global tile.  Blocks are dealt to the 8 XCDs round-robin (block index mod 8); tiles
// are dealt to them in groups of kXcdGroup horizontally adjacent tiles, group g to XCD g mod 8.  A group
// shares splats in one XCD's L2, and the dealing spreads the heavy centre of the image over all XCDs
// (contiguous bands per XCD left the busiest XCD with 1.16x the mean backward work and about 1.36x the
// mean forward work on the 3M-splat frame).  Measured on that frame: groups of 8 gave 2.25 ms per
// training step against 2.27 (groups of 4 and 16), 2.30 (bands) and 2.32 (single tiles).
constexpr int kXcdGroup = 8;
__device__ __forceinline__ int64_t xcd_tile(int64_t blk) {
  const int64_t i = blk >> 3;   // index of the block within its XCD
  return ((blk & 7) + 8 * (i / kXcdGroup)) * kXcdGroup + (i % kXcdGroup);
}

// The backward pass of a single view deals groups of kXcdGroup tiles in the order group_order gives (its
// heaviest walks first, so that the longest waves start at once and the light ones fill in behind them),
// group by group to the XCDs as xcd_tile does.  Returns -1 past the last tile.
__device__ __forceinline__ int64_t ordered_tile(int64_t blk, const uint32_t* group_order, int64_t tiles) {
  const int64_t i = blk >> 3;
  const int64_t gi = (blk & 7) + 8 * (i / kXcdGroup);
  const int64_t ngroups = (tiles + kXcdGroup - 1) / kXcdGroup;
  if (gi >= ngroups) return -1;
  const uint32_t g = group_order[gi];
  if (g >= ngroups) return -1;
  const int64_t t = (int64_t)g * kXcdGroup + (i % kXcdGroup);
  return t < tiles ? t : -1;
}

// Forward pass: one block of four wave64s per 16x16 tile, each wave owning one 8x8 quadrant with one pixel per
// lane.  What bounds it is the serial walk down a tile's list, not arithmetic, wherever the frame has fewer
// tiles than the device has room for, and in the last tiles of every frame; most of what a walk meets misses
// most of the tile (200k splats at 512x512: 12 % of the examined pairs composite).  So
//   - each wave first tests 64 listed splats against its quadrant, one per lane (box_may_hit), and walks only
//     those that may reach it (a bit mask in scalar registers);
//   - it takes them kFwdGroup at a time: their falloffs are independent of one another and overlap, only the
//     short transmittance recurrence is serial;
//   - the next kFwdBatch records are loaded while the current ones are composited (two LDS buffers, one
//     barrier per batch).
// The arithmetic of a pair, and the order of a pixel's pairs, do not depend on any of this.  Measured against two
// waves per tile with two pixels per lane, walking every splat: 1k splats at 64x64 102 -> 36 us, 200k at 512x512
// 363 -> 130, GEF 300k at 801x533 443 -> 304, 1M at 1600x1040 233 -> 188, 3M at 1920x1080 243 -> 221, 5M of heavy
// overlap 828 -> 642.  Other group sizes (with the next records still waited for at their loads: 36, 133, 329, 189, 229,
// 666 us): 2 everywhere 41, 139, 349, 185, 228, 659; one splat at a time with a branch per decision 51, 169, 478,
// 251, 304, 905.
constexpr int kFwdWaves = 4;
constexpr int kFwdBatch = 128;              // records staged per barrier: threads 0-127 load words 0-7 of
                                            // one record each, threads 128-255 words 8-11
static_assert(kFwdBatch * 2 == 64 * kFwdWaves, "half the block per record part");

// Whether a splat's alpha-floor ellipse may reach a pixel centre of the box (dx, dy: mean minus the box's
// edges).  False only if pair_q exceeds q_max at every pixel of the box: the least q over the box (on an edge
// unless the mean lies inside; there a quadratic, least at the clamped stationary point) is compared with
// q_max plus 4e-6 of the largest term magnitude a pixel of the box can have, which covers the binary32
// rounding of pair_q (5 roundings, 3e-7 of the magnitude) and of this minimum (below 1e-6 of it).
__device__ __forceinline__ float box_edge(float a, float b, float c, float rc, float e, float lo, float hi) {
  const float y = fminf(fmaxf(-(b * e) * rc, lo), hi);
  return __builtin_fmaf(__builtin_fmaf(a, e, 2.f * b * y), e, c * y * y);
}
__device__ __forceinline__ bool box_may_hit(float a, float b, float c, float qm, float dxlo, float dxhi, float dylo,
                                            float dyhi) {
  if (dxlo <= 0.f && dxhi >= 0.f && dylo <= 0.f && dyhi >= 0.f) return true;
  const float ra = fast_rcp(a), rc = fast_rcp(c);
  const float m = fminf(fminf(box_edge(a, b, c, rc, dxlo, dylo, dyhi), box_edge(a, b, c, rc, dxhi, dylo, dyhi)),
                        fminf(box_edge(c, b, a, ra, dylo, dxlo, dxhi), box_edge(c, b, a, ra, dyhi, dxlo, dxhi)));
  const float ax = fmaxf(fabsf(dxlo), fabsf(dxhi)), ay = fmaxf(fabsf(dylo), fabsf(dyhi));
  const float mag = __builtin_fmaf(__builtin_fmaf(a, ax, 2.f * fabsf(b) * ay), ax, c * ay * ay);
  return !(m > __builtin_fmaf(4e-6f, mag, qm));
}

__device__ __forceinline__ float scalar_f32(float x) {   // of a wave-uniform value
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// The lanes whose comparison holds, as a scalar mask (one compare; NaN compares false).
__device__ __forceinline__ uint64_t lanes_le(float x, float y) { return __builtin_amdgcn_fcmpf(x, y, 5); }
__device__ __forceinline__ uint64_t lanes_lt(float x, float y) { return __builtin_amdgcn_fcmpf(x, y, 4); }

// An empty instruction that takes a group's record words: their LDS reads are issued together before it.
template <int N>
__device__ __forceinline__ void group_loaded(Vec4 (&A)[N], Vec4 (&B)[N]) {
  static_assert(N == 2 || N == 4, "one operand list per size");
  if constexpr (N == 4)
    asm volatile("" : "+v"(A[0]), "+v"(A[1]), "+v"(A[2]), "+v"(A[3]), "+v"(B[0]), "+v"(B[1]), "+v"(B[2]), "+v"(B[3]));
  else
    asm volatile("" : "+v"(A[0]), "+v"(A[1]), "+v"(B[0]), "+v"(B[1]));
}

template <int FALLOFF, int kFwdGroup>
__global__ void __launch_bounds__(64 * kFwdWaves) raster_forward_kernel(const DeviceBatch* __restrict__ db,
                                                             const uint2* __restrict__ sorted_pairs,
                                                             int64_t total_tiles,
                                                             uint64_t capacity) {
  __shared__ Vec4 stage[2][3][kFwdBatch];   // record words 0-3 (b doubled), 4-7 and 8-11
  __shared__ uint32_t live[2][kFwdWaves];
  __shared__ unsigned long long red[kFwdWaves][2];
  __shared__ uint32_t red_m[kFwdWaves];
  const int64_t gt = xcd_tile(blockIdx.x);
  if (gt >= total_tiles) return;   // the whole block
  const int v = view_of_block(db->tile_prefix, db->nviews, gt);
  const ViewDesc& V = db->views[v];
  const int lt = (int)(gt - db->tile_prefix[v]);
  const int tx = lt % V.tiles_x, ty = lt / V.tiles_x;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qx = tx * kTile + (w & 1) * 8, qy = ty * kTile + (w >> 1) * 8;   // the wave's quadrant
  const int px = qx + (lane & 7), py = qy + (lane >> 3);
  const bool inside = px < V.width && py < V.height;
  uint64_t alive = __ballot(inside);   // pixels still compositing
  // a pixel that has stopped takes a NaN centre: its q is NaN and fails the alpha-floor test of every splat
  float pxf = inside ? (float)px : __builtin_nanf("");
  const float pyf = (float)py;
  // pixel centres of the quadrant, in scalar registers
  const float bx0 = scalar_f32((float)qx), bx1 = scalar_f32((float)min(qx + 7, V.width - 1));
  const float by0 = scalar_f32((float)qy), by1 = scalar_f32((float)min(qy + 7, V.height - 1));
  float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
  uint32_t last = 0u;
  // wave totals (scalars): pairs examined by pixels that terminated (1 + the terminating position each), and
  // pairs composited
  uint64_t n_exam = 0;
  uint32_t n_blend = 0;
  const uint2 rg = V.ranges[lt];
  // a range beyond the key buffer (inconsistent key count) renders as background; the list length is made
  // a scalar, so that the batch and splat loop control runs on the scalar unit
  const int n = __builtin_amdgcn_readfirstlane((uint64_t)rg.y <= capacity ? (int)(rg.y - rg.x) : 0);
  const GlobalRec* rec = (const GlobalRec*)(V.rec);
  const uint2* list = sorted_pairs + rg.x;
  // staging: this thread's record of a batch, and which part of it
  const int sj = threadIdx.x & (kFwdBatch - 1);
  const bool part0 = w < kFwdWaves / 2;
  const int first_word = part0 ? 0 : 2;
  uint32_t id = 0;
  Vec4 r0 = {0.f, 0.f, 0.f, 0.f}, r1 = r0;
  auto load_id = [&](int base) {
    if (base + sj < n) id = list[base + sj].x;
  };
  auto load_rec = [&](int base) {
    if (base + sj < n) {
      // without a branch on the part: assigned in both of its arms, the words went through scratch memory, and their
      // loads were waited for on the spot (3M splats at 1920x1080: 105 MB more written, forward 234 -> 221 us; GEF 300k at 801x533 332 -> 304)
      r0 = rec[4 * (size_t)id + first_word];
      r1 = rec[4 * (size_t)id + (part0 ? 1 : 2)];
    }
  };
  auto store_rec = [&](int buf) {
    if (part0) {
      stage[buf][0][sj] = Vec4{r0.x, r0.y, r0.z, r0.w + r0.w};
      stage[buf][1][sj] = r1;
    } else {
      stage[buf][2][sj] = r0;
    }
  };
  if (n > 0) {
    load_id(0);
    load_rec(0);
    load_id(kFwdBatch);
    store_rec(0);
    __syncthreads();
  }
  int buf = 0;
  for (int base = 0; base < n; base += kFwdBatch, buf ^= 1) {
    const int cnt = min(kFwdBatch, n - base);
    load_rec(base + kFwdBatch);       // the records of the next batch, and the list entries of the one after,
    load_id(base + 2 * kFwdBatch);    // arrive while this one is composited
    const Vec4(*st)[kFwdBatch] = stage[buf];
    if (alive) {                      // wave-uniform: a wave whose pixels have all stopped only stages
      for (int c0 = 0; c0 < cnt; c0 += 64) {
        bool hit = false, inf = false;
        if (c0 + lane < cnt) {
          const Vec4 A = st[0][c0 + lane];
          const Vec4 B = st[1][c0 + lane];
          const Vec4 Cl = st[2][c0 + lane];
          inf = !(fabsf(Cl.x) + fabsf(Cl.y) + fabsf(Cl.z) < __builtin_inff());
          hit = box_may_hit(A.z, 0.5f * A.w, B.x, B.y, A.x - bx1, A.x - bx0, A.y - by1, A.y - by0);
        }
        uint64_t mask = __ballot(hit);
        const uint64_t odd = __ballot(inf);   // a colour that is not finite (or a sum of magnitudes that is not)
        while (mask) {
          // the next kFwdGroup splats (a short last group repeats its first, switched off)
          int js[kFwdGroup];
          uint64_t have[kFwdGroup];
#pragma unroll
          for (int e = 0; e < kFwdGroup; ++e) {
            have[e] = mask ? ~0ull : 0ull;
            js[e] = mask ? c0 + (int)__builtin_ctzll(mask) : js[0];
            mask &= mask - 1ull;   // 0 stays 0
          }
          Vec4 A[kFwdGroup], B[kFwdGroup], Cc[kFwdGroup];
#pragma unroll
          for (int e = 0; e < kFwdGroup; ++e) {
            A[e] = st[0][js[e]];
            B[e] = st[1][js[e]];
            Cc[e] = st[2][js[e]];
          }
          group_loaded(A, B);   // all the group's LDS reads before the first use
          float q[kFwdGroup], alpha[kFwdGroup];
          uint64_t ok[kFwdGroup], some = 0ull;   // lanes whose pixel takes the splat (a stopped pixel's q is NaN)
#pragma unroll
          for (int e = 0; e < kFwdGroup; ++e) {
            float dx, dy;
            q[e] = pair_q(A[e].x, A[e].y, A[e].z, A[e].w, B[e].x, pxf, pyf, dx, dy);
            ok[e] = lanes_le(q[e], B[e].y) & have[e];
            some |= ok[e];
          }
          if (!some) continue;
#pragma unroll
          for (int e = 0; e < kFwdGroup; ++e) {
            const float qc = clamp_q(q[e]);
            float G;
            if constexpr (FALLOFF == GES_FALLOFF_PHI) {
              G = fast_exp2(kNegHalfLog2e * qc);
            } else {
              const float qb = fast_exp2(0.5f * B[e][3] * fast_log2(qc));
              G = fast_exp2(kNegHalfLog2e * qb);
            }
            alpha[e] = fminf(kAlphaMax, B[e].z * G);
          }
          // transmittance behind each splat of the group, a pixel that does not take one keeping its own
          float t[kFwdGroup + 1], a0[kFwdGroup];
          t[0] = T;
#pragma unroll
          for (int e = 0; e < kFwdGroup; ++e) {
            a0[e] = __builtin_amdgcn_inverse_ballot_w64(ok[e]) ? alpha[e] : 0.f;
            t[e + 1] = t[e] * (1.f - a0[e]);   // exactly t[e] where the splat is not taken
          }
          if (!((lanes_lt(t[kFwdGroup], kTMin) & alive) | odd)) {
            // no pixel stops in this group (t never grows) and every colour is finite, so a weight of 0 adds
            // exactly nothing: straight-line for the whole wave
#pragma unroll
            for (int e = 0; e < kFwdGroup; ++e) {
              const float wgt = a0[e] * t[e];
              C0 = __builtin_fmaf(wgt, Cc[e].x, C0);
              C1 = __builtin_fmaf(wgt, Cc[e].y, C1);
              C2 = __builtin_fmaf(wgt, Cc[e].z, C2);
              last = __builtin_amdgcn_inverse_ballot_w64(ok[e]) ? (uint32_t)(base + js[e] + 1) : last;
              n_blend += (uint32_t)__builtin_popcountll(ok[e]);
            }
            T = t[kFwdGroup];
            continue;
          }
#pragma unroll
          for (int e = 0; e < kFwdGroup; ++e) {   // splat by splat, a pixel stopping at its own
            const uint32_t pos1 = (uint32_t)(base + js[e] + 1);
            const float te = T * (1.f - alpha[e]);
            const uint64_t ended = lanes_lt(te, kTMin) & ok[e] & alive;
            if (ended) {
              alive &= ~ended;
              n_exam += (uint64_t)pos1 * (uint32_t)__builtin_popcountll(ended);
              pxf = __builtin_amdgcn_inverse_ballot_w64(ended) ? __builtin_nanf("") : pxf;
            }
            const uint64_t blend = ok[e] & alive;
            n_blend += (uint32_t)__builtin_popcountll(blend);
            if (__builtin_amdgcn_inverse_ballot_w64(blend)) {
              const float wgt = alpha[e] * T;
              C0 = __builtin_fmaf(wgt, Cc[e].x, C0);
              C1 = __builtin_fmaf(wgt, Cc[e].y, C1);
              C2 = __builtin_fmaf(wgt, Cc[e].z, C2);
              T = te;
              last = pos1;
            }
          }
          if (!alive) break;
        }
        if (!alive) break;
      }
    }
    // the block stops once every pixel of the tile has (the same decision in every wave, taken after the
    // barrier that also ends the reads of this batch)
    if (lane == 0) live[buf][w] = alive ? 1u : 0u;
    store_rec(buf ^ 1);
    __syncthreads();
    uint32_t any_live = 0;
#pragma unroll
    for (int k = 0; k < kFwdWaves; ++k) any_live |= live[buf][k];
    if (!any_live) break;
  }
  {
    // pair statistics of the tile: pairs examined (each pixel up to and including its terminating splat)
    // and composited, stored per tile and summed by raster_stats_kernel.  (Device-scope atomics from
    // every tile into one counter serialise across the XCDs: two per tile cost about 50 us per frame.)
    // pixels still alive examined the whole list (out-of-image pixels were never alive)
    const unsigned long long e = n_exam + (unsigned long long)__builtin_popcountll(alive) * (uint32_t)n;
    const unsigned long long b = n_blend;
    // and the length of the backward walk over the tile: its last composited position
    uint32_t m = last;
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
    if (lane == 0) { red[w][0] = e; red[w][1] = b; red_m[w] = m; }
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long se = 0, sb = 0;
      uint32_t sm = 0;
#pragma unroll
      for (int q = 0; q < kFwdWaves; ++q) {
        se += red[q][0];
        sb += red[q][1];
        sm = max(sm, red_m[q]);
      }
      V.tile_stats[2 * lt] = se;
      V.tile_stats[2 * lt + 1] = sb;
      V.tile_work[lt] = sm;
    }
  }
  if (inside) {
    const size_t pix = (size_t)py * V.width + px;
    V.out_rgb[3 * pix + 0] = __builtin_fmaf(T, V.bg[0], C0);
    V.out_rgb[3 * pix + 1] = __builtin_fmaf(T, V.bg[1], C1);
    V.out_rgb[3 * pix + 2] = __builtin_fmaf(T, V.bg[2], C2);
    if (V.final_T) V.final_T[pix] = T;
    if (V.n_contrib) V.n_contrib[pix] = last;
  }
}

// ---- sums with DPP: quad swaps and row rotations
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xf, false);
  return x + __int_as_float(y);
}

// Sum over each row of 16 lanes (every lane of the row ends with its row's total).
__device__ __forceinline__ float row_sum(float x) {
  x = dpp_add<0xB1, 0xf>(x);    // quad_perm [1,0,3,2]
  x = dpp_add<0x4E, 0xf>(x);    // quad_perm [2,3,0,1]
  x = dpp_add<0x124, 0xf>(x);   // row_ror:4
  x = dpp_add<0x128, 0xf>(x);   // row_ror:8
  return x;
}

// One exchange step of a reduce-scatter inside rows of 16 lanes: the lane pairs with the lane that the
// involution CTRL maps it to (row_mirror: l^15, row_half_mirror: l^7, quad_perm [2,3,0,1]: l^2); the lane
// with the bit set keeps the second operand's partial sum and sends the first, its partner the reverse.
template <int CTRL>
__device__ __forceinline__ float xstep(float lo, float hi, bool upper) {
  const float keep = upper ? hi : lo;
  const float send = upper ? lo : hi;
  return keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), CTRL, 0xf, 0xf, false));
}

// Row sums of 8 values in 8 DPP adds and 14 selects instead of 32 DPP adds: the partner masks 15, 7, 2, 1
// span the 16 lanes of a row, and lane l ends with the sum of value (l >> 1) & 7 over its row.
__device__ __forceinline__ float row_scatter8(float a0, float a1, float a2, float a3, float a4, float a5, float a6,
                                              float a7, int lane) {
  const bool u3 = lane & 8, u2 = lane & 4, u1 = lane & 2;
  const float b0 = xstep<0x140>(a0, a4, u3), b1 = xstep<0x140>(a1, a5, u3);   // row_mirror
  const float b2 = xstep<0x140>(a2, a6, u3), b3 = xstep<0x140>(a3, a7, u3);
  const float c0 = xstep<0x141>(b0, b2, u2), c1 = xstep<0x141>(b1, b3, u2);   // row_half_mirror
  const float d0 = xstep<0x4E>(c0, c1, u1);                                    // quad_perm [2,3,0,1]
  return dpp_add<0xB1, 0xf>(d0);                                               // quad_perm [1,0,3,2]
}

constexpr int kFlush = 32;   // splats whose row partials are parked in LDS before one flush of rows

// Words of the backward's plan (b.kw.plan): where each XCD's work items start, the number of tiles whose walk
// is cut, and the list positions per segment.
enum : int { P_STARTS = 0, P_CUT = 9, P_SEG = 10 };

// Walks the cut tiles back to front only to leave, at every segment boundary, the transmittance and the colour
// behind it: the recurrences of the backward pass, the same operations in the same order (so that cutting a walk
// changes no bit of the gradients), without its sums.  Launch shape and walk as in the forward pass: a quadrant
// per wave, only the splats that can reach it, kRecGroup at a time; a splat that a pixel does not take has alpha
// 0, which leaves its transmittance and colour exactly as they are (a colour that is not finite is taken as 0 there, in
// a walk of its own: with a branch for it in the one walk, two views of 52x474 take 1,224 us instead of 1,174, and the two
// need the bound of 6 waves per SIMD, GEF 300k at 801x533 758 without, 745 with).
constexpr int kRecGroup = 4;
template <int FALLOFF>
__global__ void __launch_bounds__(64 * kFwdWaves, 6) raster_recover_kernel(const DeviceBatch* __restrict__ db,
                                                             const uint2* __restrict__ sorted_pairs,
                                                             const uint32_t* __restrict__ cut_tiles,
                                                             const uint32_t* __restrict__ plan) {
  __shared__ Vec4 stage[2][3][kFwdBatch];   // record words 0-3 (b doubled), 4-7 and 8-11
  if (blockIdx.x >= plan[P_CUT]) return;   // the whole block
  const int64_t gt = cut_tiles[blockIdx.x];
  const int v = view_of_block(db->tile_prefix, db->nviews, gt);
  const ViewDesc& V = db->views[v];
  const int lt = (int)(gt - db->tile_prefix[v]);
  const int tx = lt % V.tiles_x, ty = lt / V.tiles_x;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qx = tx * kTile + (w & 1) * 8, qy = ty * kTile + (w >> 1) * 8;   // the wave's quadrant
  const int px = qx + (lane & 7), py = qy + (lane >> 3);
  const float pxf = (float)px, pyf = (float)py;
  const float bx0 = scalar_f32((float)qx), bx1 = scalar_f32((float)min(qx + 7, V.width - 1));
  const float by0 = scalar_f32((float)qy), by1 = scalar_f32((float)min(qy + 7, V.height - 1));
  float T = 1.f, S0 = 0.f, S1 = 0.f, S2 = 0.f;
  uint32_t last = 0u;
  if (px < V.width && py < V.height) {
    const size_t pix = (size_t)py * V.width + px;
    T = V.final_T[pix];
    last = V.n_contrib[pix];
  }
  uint32_t wl = last;
  for (int off = 32; off > 0; off >>= 1) wl = max(wl, (uint32_t)__shfl_xor((int)wl, off, 64));
  const int wlast = __builtin_amdgcn_readfirstlane((int)wl);   // the wave's own walk
  const int n = __builtin_amdgcn_readfirstlane((int)V.tile_work[lt]);
  const int seg = __builtin_amdgcn_readfirstlane((int)plan[P_SEG]);
  int bound = (n - 1) / seg * seg;   // the next boundary on the way down
  GlobalVec4* ck = (GlobalVec4*)V.ckpt + (size_t)V.tile_ckpt[lt] * kTilePx + ((w >> 1) * 8 + (lane >> 3)) * kTile +
                   (w & 1) * 8 + (lane & 7);   // the pixel's entry at the tile's first boundary
  const GlobalRec* rec = (const GlobalRec*)(V.rec);
  const uint2* list = sorted_pairs + V.ranges[lt].x;
  const int sj = threadIdx.x & (kFwdBatch - 1);
  const bool part0 = w < kFwdWaves / 2;
  const int first_word = part0 ? 0 : 2;
  uint32_t id = 0;
  Vec4 r0 = {0.f, 0.f, 0.f, 0.f}, r1 = r0;
  auto load_id = [&](int base) {
    if (base >= 0 && base + sj < n) id = list[base + sj].x;
  };
  auto load_rec = [&](int base) {
    if (base >= 0 && base + sj < n) {
      r0 = rec[4 * (size_t)id + first_word];   // no branch on the part (see the forward)
      r1 = rec[4 * (size_t)id + (part0 ? 1 : 2)];
    }
  };
  auto store_rec = [&](int buf) {
    if (part0) {
      stage[buf][0][sj] = Vec4{r0.x, r0.y, r0.z, r0.w + r0.w};
      stage[buf][1][sj] = r1;
    } else {
      stage[buf][2][sj] = r0;
    }
  };
  const int top = (n - 1) / kFwdBatch * kFwdBatch;
  load_id(top);
  load_rec(top);
  load_id(top - kFwdBatch);
  store_rec(0);
  __syncthreads();
  int buf = 0;
  for (int base = top; base >= 0 && base + kFwdBatch >= seg; base -= kFwdBatch, buf ^= 1) {   // to the first boundary
    load_rec(base - kFwdBatch);
    load_id(base - 2 * kFwdBatch);
    const Vec4(*st)[kFwdBatch] = stage[buf];
    for (int c0 = kFwdBatch - 64; c0 >= 0; c0 -= 64) {
      const int lo = base + c0;
      if (lo + 64 == bound) {
        if (wlast > bound) ck[(size_t)(bound / seg - 1) * kTilePx] = Vec4{T, S0, S1, S2};
        bound -= seg;
      }
      if (wlast <= lo) continue;   // the quadrant's pixels all stopped before these splats
      bool hit = false, inf = false;
      if (lo + lane < wlast) {
        const Vec4 A = st[0][c0 + lane];
        const Vec4 B = st[1][c0 + lane];
        const Vec4 Cl = st[2][c0 + lane];
        inf = !(fabsf(Cl.x) + fabsf(Cl.y) + fabsf(Cl.z) < __builtin_inff());
        hit = box_may_hit(A.z, 0.5f * A.w, B.x, B.y, A.x - bx1, A.x - bx0, A.y - by1, A.y - by0);
      }
      uint64_t mask = __ballot(hit);
      const bool odd = __ballot(inf) != 0ull;   // a colour that is not finite (or a sum of magnitudes that is not)
      auto walk = [&](auto wild) {
        while (mask) {
          // the next kRecGroup splats from the back (a short last group repeats its first, switched off)
          int js[kRecGroup];
          uint64_t have[kRecGroup];
#pragma unroll
          for (int e = 0; e < kRecGroup; ++e) {
            have[e] = mask ? ~0ull : 0ull;
            js[e] = mask ? 63 - (int)__builtin_clzll(mask) : js[0];
            mask &= ~(1ull << js[e]);   // 0 stays 0
          }
          Vec4 A[kRecGroup], B[kRecGroup], Cc[kRecGroup];
#pragma unroll
          for (int e = 0; e < kRecGroup; ++e) {
            A[e] = st[0][c0 + js[e]];
            B[e] = st[1][c0 + js[e]];
            Cc[e] = st[2][c0 + js[e]];
          }
          group_loaded(A, B);
          float alpha[kRecGroup], inv[kRecGroup];
          uint64_t take[kRecGroup];
#pragma unroll
          for (int e = 0; e < kRecGroup; ++e) {
            float dx, dy;
            const float q0 = pair_q(A[e].x, A[e].y, A[e].z, A[e].w, B[e].x, pxf, pyf, dx, dy);
            take[e] = lanes_le(q0, B[e].y) & have[e] &
                      __builtin_amdgcn_uicmp((uint32_t)(lo + js[e]), last, 36);   // position < last
            const float q = clamp_q(q0);
            float G;
            if (FALLOFF == GES_FALLOFF_PHI) {
              G = fast_exp2(kNegHalfLog2e * q);
            } else {
              const float qb = fast_exp2(0.5f * B[e].w * fast_log2(q));
              G = fast_exp2(kNegHalfLog2e * qb);
            }
            const float oG = B[e].z * G;
            const float full = oG > kAlphaMax ? kAlphaMax : oG;
            alpha[e] = __builtin_amdgcn_inverse_ballot_w64(take[e]) ? full : 0.f;
            inv[e] = __builtin_amdgcn_inverse_ballot_w64(take[e]) ? fast_rcp(1.f - alpha[e]) : 1.f;
          }
          if constexpr (decltype(wild)::value) {   // 0 times an infinite colour would not leave S as it is
#pragma unroll
            for (int e = 0; e < kRecGroup; ++e)
              if (!__builtin_amdgcn_inverse_ballot_w64(take[e])) Cc[e] = Vec4{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int e = 0; e < kRecGroup; ++e) {
            T = T * inv[e];
            S0 = __builtin_fmaf(alpha[e], Cc[e].x - S0, S0);
            S1 = __builtin_fmaf(alpha[e], Cc[e].y - S1, S1);
            S2 = __builtin_fmaf(alpha[e], Cc[e].z - S2, S2);
          }
        }
      };
      if (odd) walk(std::true_type{});
      else walk(std::false_type{});
    }
    store_rec(buf ^ 1);
    __syncthreads();
  }
}

// The bands of 4 pixel rows of the tile at (x0, y0) that a splat may reach (box_may_hit of each).  A wave asks this of 64
// splats at a time, one per lane, and walks the ones that reach a band, looking at those bands only: 1M splats at
// 1600x1040 352 -> 336 us, 5M of heavy overlap 1322 -> 1265, 3M at 1920x1080 416 -> 407, four views of 200k at 512x512
// 570 -> 524.
__device__ __forceinline__ uint32_t bands_reached(float u, float v, float a, float b, float c, float qm, float x0,
                                                  float y0) {
  uint32_t m = 0u;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    m |= box_may_hit(a, b, c, qm, u - (x0 + 15.f), u - x0, v - (y0 + (float)(4 * k + 3)), v - (y0 + (float)(4 * k)))
             ? 1u << k : 0u;
  return m;
}

// One block of one wave per work item.  SEGMENTED: an item is a segment of a tile's walk (see
// backward_prepare_kernel), and a block takes further items in turn; it starts from the transmittance behind the
// segment and the colour behind it, which are the pixel's final transmittance and nothing where its last
// composited splat lies in the segment, else what raster_recover_kernel left at the boundary.  Otherwise an item
// is a whole tile, dealt by ordered_tile or xcd_tile.
template <int FALLOFF, bool SEGMENTED>
__global__ void __launch_bounds__(64) raster_backward_kernel(const DeviceBatch* __restrict__ db,
                                                             const uint2* __restrict__ sorted_pairs,
                                                             int64_t total_tiles, const uint2* __restrict__ items,
                                                             const uint32_t* __restrict__ plan) {
  __shared__ float4 sA[64], sB[64], sC[64];
  __shared__ float sRed[kFlush][4][10];   // [parked splat][lane row][component]
  __shared__ uint32_t sSlot[kFlush];      // the parked splat's slot: its row of this tile's sums
  __shared__ uint32_t sItem[kFlush];      // the parked splat's batch item and first candidate slot (written
  __shared__ uint32_t sFirst[kFlush];     // into its row)
  __shared__ uint32_t sIdx[64];           // batch item and first candidate slot of each staged splat
  __shared__ uint32_t sLo[64];
  const int lane = threadIdx.x;
  const int row = lane >> 4;
  const uint32_t xcd = blockIdx.x & 7u;
  const uint32_t end = SEGMENTED ? plan[P_STARTS + xcd + 1] : 1u;
  for (uint32_t it = SEGMENTED ? plan[P_STARTS + xcd] + (blockIdx.x >> 3) : 0u; it < end;
       it += SEGMENTED ? gridDim.x >> 3 : 1u) {
    const uint2 item = SEGMENTED ? items[it] : make_uint2(0u, 0u);   // batch tile, segment
    const int64_t gt = SEGMENTED ? (int64_t)item.x
                       : db->nviews == 1 ? ordered_tile(blockIdx.x, db->views[0].group_order, total_tiles)
                                         : xcd_tile(blockIdx.x);
    if (gt < 0 || gt >= total_tiles) return;
    const int v = view_of_block(db->tile_prefix, db->nviews, gt);
    const ViewDesc& V = db->views[v];
    const int lt = (int)(gt - db->tile_prefix[v]);
    const int tx = lt % V.tiles_x, ty = lt / V.tiles_x;
    const int px = tx * kTile + (lane & 15);
    const int py0 = ty * kTile + (lane >> 4);
    const float pxf = (float)px;
    const uint2 rg = V.ranges[lt];
    const uint32_t seg = SEGMENTED ? plan[P_SEG] : 0u;
    const uint32_t first_pos = item.y * seg, end_pos = SEGMENTED ? first_pos + seg : ~0u;
    float pyf[4], T[4], TfB[4], g[4][3], S[4][3];
    uint32_t last[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int py = py0 + 4 * k;
      pyf[k] = (float)py;
      S[k][0] = S[k][1] = S[k][2] = 0.f;
      if (px < V.width && py < V.height) {
        const size_t pix = (size_t)py * V.width + px;
        T[k] = V.final_T[pix];
        last[k] = V.n_contrib[pix];
        g[k][0] = V.dL_drgb[3 * pix];
        g[k][1] = V.dL_drgb[3 * pix + 1];
        g[k][2] = V.dL_drgb[3 * pix + 2];
      } else {
        T[k] = 1.f;
        last[k] = 0u;
        g[k][0] = g[k][1] = g[k][2] = 0.f;
      }
      // T_final (bg . g): the background's share of dL/dalpha, divided by (1 - alpha) per splat
      TfB[k] = T[k] * (V.bg[0] * g[k][0] + V.bg[1] * g[k][1] + V.bg[2] * g[k][2]);
    }
    if constexpr (SEGMENTED) {
      const GlobalRec* ck = (const GlobalRec*)V.ckpt + ((size_t)V.tile_ckpt[lt] + item.y) * kTilePx + lane;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (last[k] > end_pos) {   // the walk of this pixel, 16 (row + 4 k) + column, goes on behind the segment
          const Vec4 c = ck[64 * k];
          T[k] = c.x;
          S[k][0] = c.y;
          S[k][1] = c.z;
          S[k][2] = c.w;
          last[k] = end_pos;
        } else if (last[k] <= first_pos) {
          last[k] = 0u;
        }
      }
    }
    // wave max of the last contributor position per band of 4 rows and over the tile, made scalars: the walk's
    // loop control (positions, the parked-splat count, the flush test) then runs on the scalar unit instead of
    // taking VALU issue slots, and a band skips the splats behind all of its pixels' last ones
    // the logarithm of q's floor by the instruction that takes the others
    float q_floor = 1e-12f;
    asm volatile("" : "+v"(q_floor));
    const float lq_floor = FALLOFF == GES_FALLOFF_GEF ? fast_log2(q_floor) : 0.f;
    uint32_t band_last[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t m = last[k];
      for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
      band_last[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
    }
    const uint32_t maxlast = max(max(band_last[0], band_last[1]), max(band_last[2], band_last[3]));
    const GlobalRec* rec = (const GlobalRec*)(V.rec);
    // global address space: the row stores then count only against vmcnt, and the LDS waits of the following
    // splats do not wait for them (flat stores count against lgkmcnt too)
    GlobalVec4* rows = (GlobalVec4*)(V.grad_rows);
    GlobalU32* bits = (GlobalU32*)(V.grad_bits);
    int nslot = 0;
    const int stop = __builtin_amdgcn_readfirstlane((int)first_pos);
    auto flush = [&]() {
      // one lane per parked splat: add the four row sums and store the tile's sums of the splat, the splat's
      // batch item and its first candidate slot in the row of its slot (the row reduction adds a splat's rows
      // in slot order), marking the slot
      __syncthreads();
      if (lane < nslot) {   // entries 0 .. nslot-1 hold row partials
        const uint32_t slot = sSlot[lane];
        float val[10];
#pragma unroll
        for (int c = 0; c < 10; ++c)
          val[c] = (sRed[lane][0][c] + sRed[lane][1][c]) + (sRed[lane][2][c] + sRed[lane][3][c]);
        val[0] = 2.f * val[0];   // dL/du = 2 sum dq (a dx + b dy)
        val[1] = 2.f * val[1];   // dL/dv = 2 sum dq (b dx + c dy)
        val[3] = 2.f * val[3];   // dL/db = 2 sum dq dx dy
        if (FALLOFF != GES_FALLOFF_GEF) val[9] = 0.f;
        GlobalVec4* r = rows + (size_t)slot * (kRowFloats / 4);
        Vec4 v0, v1, v2;
        v0[0] = val[0]; v0[1] = val[1]; v0[2] = val[2]; v0[3] = val[3];
        v1[0] = val[4]; v1[1] = val[5]; v1[2] = val[6]; v1[3] = val[7];
        v2[0] = val[8]; v2[1] = val[9]; v2[2] = __uint_as_float(sItem[lane]); v2[3] = __uint_as_float(sFirst[lane]);
        r[0] = v0;
        r[1] = v1;
        r[2] = v2;
        __hip_atomic_fetch_or(bits + (slot >> 5), 1u << (slot & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      nslot = 0;
    };
    for (int hi = (int)maxlast; hi > stop; hi -= 64) {
      const int lo = max(stop, hi - 64);
      const int cnt = hi - lo;
      uint32_t reach = 0u;   // of this lane's splat: the bands it may reach
      if (lane < cnt) {
        const uint2 pr = sorted_pairs[rg.x + lo + lane];   // (splat index, slot)
        const float4 a = rec_load(rec, 4 * (size_t)pr.x);
        const float4 b = rec_load(rec, 4 * (size_t)pr.x + 1);
        const float4 c = rec_load(rec, 4 * (size_t)pr.x + 2);
        sA[lane] = make_float4(a.x, a.y, a.z, a.w);
        sB[lane] = b;
        sC[lane] = make_float4(c.x, c.y, c.z, __uint_as_float(pr.y));
        sIdx[lane] = (uint32_t)db->item_prefix[v] + pr.x;
        sLo[lane] = V.slot_off[pr.x];
        reach = bands_reached(a.x, a.y, a.z, a.w, b.x, b.y, (float)(tx * kTile), (float)(ty * kTile));
      }
      uint64_t band[4], walk = 0ull;   // the splats a band has to look at: those before the last of its pixels'
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t n = band_last[k] > (uint32_t)lo ? band_last[k] - (uint32_t)lo : 0u;
        band[k] = __ballot((reach >> k) & 1u) & (n >= 64u ? ~0ull : (1ull << n) - 1ull);
        walk |= band[k];
      }
      __syncthreads();
      while (walk) {
        const int j = 63 - (int)__builtin_clzll(walk);
        walk &= ~(1ull << j);
        const float4 A = sA[j];
        const float4 B = sB[j];
        const float4 Cc = sC[j];
        const uint32_t pos = (uint32_t)(lo + j);
        const float bb = A.w + A.w;
        // per lane: sums over its pixels of dq (a dx + b dy), dq (b dx + c dy), dq dx^2, dq dx dy, dq dy^2
        // (dq = dL/dq; halves of the mean2D and b gradients), of G dL/dalpha (opacity), of alpha T g
        // (colour) and, for GEF, of dL/dbeta
        float su = 0.f, sv = 0.f, pa = 0.f, pb = 0.f, pc = 0.f, po = 0.f, pr = 0.f, pg = 0.f, pbl = 0.f, pbeta = 0.f;
        bool entered = false;   // wave-uniform: some row band had a pixel that took the splat
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (!((band[k] >> j) & 1ull)) continue;   // scalar
          float dx, dy;
          const float q0 = pair_q(A.x, A.y, A.z, bb, B.x, pxf, pyf[k], dx, dy);
          const bool valid = (pos < last[k]) && (q0 <= B.y);
          if (!__any(valid)) continue;   // wave-uniform: no pixel of this row band took the splat
          entered = true;
          // straight-line for every lane; a pixel that did not take the splat gets alpha = 0 (T, S and every
          // accumulated term are then unchanged: 1/(1 - 0) = 1 exactly)
          const float q = clamp_q(q0);
          float G, qb = 0.f, lq = 0.f;
          if (FALLOFF == GES_FALLOFF_PHI) {
            G = fast_exp2(kNegHalfLog2e * q);
          } else {
            lq = fast_log2(q);
            qb = fast_exp2(0.5f * B.w * lq);
            G = fast_exp2(kNegHalfLog2e * qb);
          }
          const float oG = B.z * G;
          const bool clamped = oG > kAlphaMax;
          const float alpha = valid ? (clamped ? kAlphaMax : oG) : 0.f;
          const float inv = valid ? fast_rcp(1.f - alpha) : 1.f;
          T[k] = T[k] * inv;                 // transmittance before this splat (unchanged: inv = 1 exactly)
          const float w = alpha * T[k];
          pr = __builtin_fmaf(w, g[k][0], pr);
          pg = __builtin_fmaf(w, g[k][1], pg);
          pbl = __builtin_fmaf(w, g[k][2], pbl);
          const float d0 = Cc.x - S[k][0], d1 = Cc.y - S[k][1], d2 = Cc.z - S[k][2];
          float dalpha = __builtin_fmaf(d0, g[k][0], __builtin_fmaf(d1, g[k][1], d2 * g[k][2]));
          dalpha = __builtin_fmaf(dalpha, T[k], -TfB[k] * inv);
          S[k][0] = __builtin_fmaf(alpha, d0, S[k][0]);
          S[k][1] = __builtin_fmaf(alpha, d1, S[k][1]);
          S[k][2] = __builtin_fmaf(alpha, d2, S[k][2]);
          // below the clamp: dL/do = G dL/dalpha and G dL/dG = alpha dL/dalpha = o (G dL/dalpha); above it
          // both are 0.  Per pixel only gd = G dL/dalpha is formed: the opacity o and the constant of dG/dq
          // are common to the splat's terms and multiply its row sums once (dq below is dL/dq / (o k)).
          const float gd = (valid && !clamped) ? G * dalpha : 0.f;
          po += gd;
          float dq;
          if (FALLOFF == GES_FALLOFF_PHI) {
            dq = q0 >= 0.f ? gd : 0.f;   // dG/dq = -G/2: k = -1/2
          } else {
            // dG/dq = -(beta/4) q^(beta/2 - 1) G  (q floored at 1e-12): k = -beta/4;
            // dG/dbeta = -(1/4) q^(beta/2) ln q G: the row sum of q^(beta/2) log2 q gd takes -(ln 2)/4 o
            const float qpow = fast_exp2((0.5f * B.w - 1.f) * (q >= 1e-12f ? lq : lq_floor));   // q >= +0
            dq = q0 >= 0.f ? qpow * gd : 0.f;
            pbeta = __builtin_fmaf(q > 0.f ? qb * lq : 0.f, gd, pbeta);
          }
          const float dqdx = dq * dx, dqdy = dq * dy;
          su = __builtin_fmaf(dq, __builtin_fmaf(A.z, dx, A.w * dy), su);
          sv = __builtin_fmaf(dq, __builtin_fmaf(A.w, dx, B.x * dy), sv);
          pa = __builtin_fmaf(dqdx, dx, pa);
          pb = __builtin_fmaf(dqdx, dy, pb);
          pc = __builtin_fmaf(dqdy, dy, pc);
        }
        if (entered) {
          // rows of 16 lanes reduce in registers: the first 8 sums by a reduce-scatter (after it, lanes 2i and
          // 2i+1 of a row hold row sum i), the blue and beta sums by a full row sum; the row's lanes then park
          // the 10 sums in LDS, each scaled by the splat's common factor (o k for the dq sums, o for dL/dbeta)
          const float e = row_scatter8(su, sv, pa, pb, pc, po, pr, pg, lane);
          const float r8 = row_sum(pbl);
          const float r9 = FALLOFF == GES_FALLOFF_GEF ? row_sum(pbeta) : 0.f;
          const float kq = FALLOFF == GES_FALLOFF_PHI ? -0.5f * B.z : (-0.25f * B.w) * B.z;
          float* d = sRed[nslot][row];
          const int idx = (lane >> 1) & 7;
          if ((lane & 1) == 0) d[idx] = idx < 5 ? kq * e : e;
          if ((lane & 15) == 15) {
            d[8] = r8;
            d[9] = FALLOFF == GES_FALLOFF_GEF ? (-0.25f * 0.69314718055994531f * B.z) * r9 : 0.f;
          }
          if (lane == 0) {
            sSlot[nslot] = __float_as_uint(Cc.w);
            sItem[nslot] = sIdx[j];
            sFirst[nslot] = sLo[j];
          }
          ++nslot;
        }
        if (nslot == kFlush) flush();
      }
      __syncthreads();
    }
    if (nslot > 0) flush();
  }
}

// Bucket of a tile group for the backward order: 0 holds the heaviest walks (1,023 positions or more).
constexpr int kOrderBuckets = 1024;
static_assert(kXcdGroup == 8, "a tile group's work words are read as two 16-byte loads");
__device__ __forceinline__ int group_bucket(const uint32_t* work, int64_t g, int64_t tiles) {
  uint32_t w = 0;
  if ((g + 1) * kXcdGroup <= tiles) {   // a whole group (the work array is 256-byte aligned)
    const uint4 a = reinterpret_cast<const uint4*>(work)[2 * g];
    const uint4 b = reinterpret_cast<const uint4*>(work)[2 * g + 1];
    w = max(max(max(a.x, a.y), max(a.z, a.w)), max(max(b.x, b.y), max(b.z, b.w)));
  } else {
    for (int64_t t = g * kXcdGroup; t < tiles; ++t) w = max(w, work[t]);
  }
  return kOrderBuckets - 1 - (int)min(w, (uint32_t)(kOrderBuckets - 1));
}

// One block per view: its per-tile pair statistics summed into its header ([2] examined, [3] composited);
// for a single view, also the order of its tile groups for the backward pass: a counting sort on the
// group's longest walk, heaviest first (the order within a bucket is immaterial).
__global__ void __launch_bounds__(1024) raster_stats_kernel(const DeviceBatch* __restrict__ db) {
  __shared__ unsigned long long part[2][16];
  __shared__ uint32_t cursor[kOrderBuckets];
  __shared__ uint32_t wsum[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const ViewDesc& V = db->views[blockIdx.x];
  {
    const int T = V.tiles_x * V.tiles_y;
    unsigned long long e = 0, c = 0;
    for (int t = threadIdx.x; t < T; t += 1024) {
      e += V.tile_stats[2 * t];
      c += V.tile_stats[2 * t + 1];
    }
    for (int off = 32; off > 0; off >>= 1) {
      e += __shfl_xor(e, off, 64);
      c += __shfl_xor(c, off, 64);
    }
    if (lane == 0) { part[0][w] = e; part[1][w] = c; }
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long se = 0, sc = 0;
      for (int k = 0; k < 16; ++k) { se += part[0][k]; sc += part[1][k]; }
      V.header[2] = se;
      V.header[3] = sc;
    }
  }
  if (db->nviews != 1) return;
  const int64_t tiles = (int64_t)V.tiles_x * V.tiles_y;
  const int64_t ngroups = (tiles + kXcdGroup - 1) / kXcdGroup;
  const int tid = threadIdx.x;
  cursor[tid] = 0u;   // one bucket per thread
  __syncthreads();
  for (int64_t g = tid; g < ngroups; g += 1024) atomicAdd(&cursor[group_bucket(V.tile_work, g, tiles)], 1u);
  __syncthreads();
  const uint32_t c = cursor[tid];   // exclusive scan of the bucket counts
  uint32_t s = c;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)s, d, 64);
    if (lane >= d) s += y;
  }
  if (lane == 63) wsum[w] = s;
  __syncthreads();
  uint32_t pre = 0;
  for (int k = 0; k < w; ++k) pre += wsum[k];
  cursor[tid] = pre + s - c;
  __syncthreads();
  for (int64_t g = tid; g < ngroups; g += 1024) {
    const uint32_t pos = atomicAdd(&cursor[group_bucket(V.tile_work, g, tiles)], 1u);
    V.group_order[pos] = (uint32_t)g;
  }
}

// Before the backward raster: the blocks past the first clear the row marks; block 0 plans the walks of a frame
// that may be cut (items not NULL).  Cutting pays where the longest walk, at about 0.5 us a splat, outlasts the walks of
// all tiles spread over the device's 1,024 SIMDs, at about 0.27 ns a position, by a factor of two (kCutShare), and where
// there are fewer than two tiles a SIMD (kCutTiles); elsewhere
// a segment is as long as the longest walk, and no tile is cut.  Over 112 frames of 64 to 6,144 tiles and one to six
// views, from 50k to 2M splats, times without the cut and with it: below the factor, from 3,072 tiles on, 1.09 to 0.71
// (GEF 150k at 1536x1024 1,433 : 2,023 us, clusters of 1M there 339 : 446), and 820 : 766 for GEF 150k at 801x533 (1,734
// tiles); from a factor of 2.1 on 1.03 up to 6 (200k in one dense cluster at 1536x1024
// 1,472 : 415).  A segment that is cut is the length that gives about kItemTarget items (a multiple of 64, the
// backward's staged batch), and every piece is a work item.  Tile groups
// (tiles, in a frame of few) go to the XCDs in turn, heaviest walks first where the forward ordered them, so
// that a group's records meet in one L2 and the last items to start are short; the items of XCD x are
// items[plan[P_STARTS + x], plan[P_STARTS + x + 1]).  There are at most as many items as walked list positions,
// and a boundary stands for at least 64 of them, so items and cut tiles fit the buffers of the tile sort.
constexpr uint32_t kCutShare = 926;   // part of the walks' sum that the longest may have: 2 x 0.27 ns / 0.5 us
constexpr uint32_t kCutTiles = 2048;
constexpr uint32_t kOrderTiles = 2048;
// Targets of 2,560 / 4,096 / 8,192 / 16,384: four views of 512x512 686 / 602 / 561 / 568 us, GEF 300k at 801x533
// 1,025 / 868 / 864 / 845; smaller frames reach the shortest segment with any.
constexpr uint32_t kItemTarget = kMaxCheckpoints;   // boundaries <= walked positions / segment <= this
template <bool PACK>
__global__ void __launch_bounds__(1024) backward_prepare_kernel(DeviceBatch* __restrict__ db,
                                                                const ViewPack pack, uint2* items,
                                                                uint32_t* cut_tiles, uint32_t* plan, uint32_t* bits,
                                                                size_t nwords) {
  if (blockIdx.x > 0) {
    const size_t n4 = nwords / 4, step = (size_t)(gridDim.x - 1) * 1024;
    const size_t i0 = (size_t)(blockIdx.x - 1) * 1024 + threadIdx.x;
    for (size_t i = i0; i < n4; i += step) reinterpret_cast<uint4*>(bits)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (i0 < nwords - 4 * n4) bits[4 * n4 + i0] = 0u;
    return;
  }
  if (PACK) write_views(db, pack);
  if (!items) return;
  const Views<PACK> views{db, pack};
  __shared__ unsigned long long wsum[16];
  __shared__ uint32_t wmax[16];
  __shared__ unsigned long long carry;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const bool one = views.count() == 1;
  const uint32_t view_tiles = (uint32_t)(PACK ? pack.tiles : db->tile_prefix[1]), tiles = views.count() * view_tiles;
  const uint32_t* work0 = views[0].tile_work;
  auto walk = [&](uint32_t t) -> uint32_t {   // the views of a backward share a resolution
    const uint32_t v = one ? 0u : t / view_tiles;
    return (one ? work0 : views[v].tile_work)[t - v * view_tiles];
  };
  unsigned long long sum = 0;   // walked positions
  uint32_t longest = 0;
  for (uint32_t t = threadIdx.x; t < tiles; t += 1024) {
    const uint32_t n = walk(t);
    sum += n;
    longest = max(longest, n);
  }
  for (int off = 32; off > 0; off >>= 1) {
    sum += __shfl_xor(sum, off, 64);
    longest = max(longest, (uint32_t)__shfl_xor((int)longest, off, 64));
  }
  if (lane == 0) { wsum[w] = sum; wmax[w] = longest; }
  if (threadIdx.x == 0) carry = 0ull;
  __syncthreads();
  sum = 0;
  for (int k = 0; k < 16; ++k) {
    sum += wsum[k];
    longest = max(longest, wmax[k]);
  }
  __syncthreads();
  const uint32_t whole = (longest + 63u) / 64u;   // batches of the longest walk
  const uint32_t piece = (uint32_t)max(1ull, (sum + 64ull * kItemTarget - 1) / (64ull * kItemTarget));
  const bool cuts = tiles < kCutTiles || (unsigned long long)longest * kCutShare > sum;
  const uint32_t seg = (cuts ? piece : max(piece, whole)) * 64u;
  // positions of the list order: XCD by XCD, a padded run of groups each; one tile per thread and round
  const uint32_t gs = tiles < kOrderTiles ? 1u : (uint32_t)kXcdGroup;   // tiles dealt to an XCD together
  const uint32_t ngroups = (tiles + gs - 1) / gs, run = (ngroups + 7) / 8 * gs;
  const uint32_t* order = one && gs > 1 ? views[0].group_order : nullptr;
  for (uint32_t o0 = 0; o0 < 8 * run; o0 += 1024) {
    const uint32_t o = o0 + threadIdx.x, x = o / run, i = o - x * run;
    uint32_t g = 8 * (i / gs) + x, t = tiles, ns = 0;
    if (x < 8 && g < ngroups) {
      if (order) g = order[g];
      t = g < ngroups ? g * gs + i % gs : tiles;
      if (t < tiles) ns = (walk(t) + seg - 1u) / seg;
    }
    // items, walks and cut walks before this tile (at most 2^32, 2^16 and 2^16: see cut_walks)
    const unsigned long long mine = ((unsigned long long)ns << 32) | (ns ? 1u << 16 : 0u) | (ns > 1 ? 1u : 0u);
    unsigned long long s = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned long long y = __shfl_up(s, d, 64);
      if (lane >= d) s += y;
    }
    if (lane == 63) wsum[w] = s;
    __syncthreads();
    unsigned long long at = carry + s - mine;
    for (int k = 0; k < w; ++k) at += wsum[k];
    const uint32_t first = (uint32_t)(at >> 32), walks = (uint32_t)at >> 16, cut = (uint32_t)at & 0xffffu;
    if (x < 8 && i == 0) plan[P_STARTS + x] = first;
    if (ns > 1) {
      const uint32_t v = one ? 0u : t / view_tiles;
      cut_tiles[cut] = t;
      views[v].tile_ckpt[t - v * view_tiles] = first - walks;   // the boundaries of the walks before it
    }
    for (uint32_t k = 0; k < ns; ++k) items[first + k] = make_uint2(t, k);
    __syncthreads();
    if (threadIdx.x == 1023) carry = at + mine;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    plan[P_STARTS + 8] = (uint32_t)(carry >> 32);
    plan[P_CUT] = (uint32_t)carry & 0xffffu;
    plan[P_SEG] = seg;
  }
}

// Frames whose walks may be cut (the device decides, see backward_prepare_kernel): up to 6,144 tiles.  Beyond, a frame with
// one dense cluster would gain too (8,160 tiles 1,088 : 333 us), others lose by the shared segment length (306 : 452).
static bool cut_walks(const Batch& b) { return b.total_tiles <= 6144; }

hipError_t launch_backward_prepare(DeviceBatch* dbatch, const Batch& b, uint32_t* bits, size_t nwords,
                                   hipStream_t stream) {
  const size_t clear = std::min<size_t>(1024, (nwords + 4095) / 4096);
  auto kernel = b.pack ? backward_prepare_kernel<true> : backward_prepare_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(1 + clear)), dim3(1024), 0, stream, dbatch,
                     b.pack ? *b.pack : ViewPack{}, cut_walks(b) ? b.kw.pv[1] : nullptr, b.kw.table, b.kw.plan, bits, nwords);
  return hipGetLastError();
}

hipError_t launch_raster_forward(const DeviceBatch* dbatch, const Batch& b, hipStream_t stream) {
  if (b.total_tiles == 0) return hipSuccess;
  const int64_t span = 8 * kXcdGroup;   // the grid covers whole rounds of groups
  const dim3 grid((unsigned)((b.total_tiles + span - 1) / span * span));
  // every view of a batch shares the falloff (the server fixes it per instance).  Splats per group: 4 shorten
  // the serial walk, 2 leave registers for more waves per SIMD, which counts once the frame fills the device
  // (4 against 2, with the statistics pass: 512x512 153 / 162 us, 801x533 GEF 318 / 361; clusters of 1M splats and 200k in
  // one dense cluster at 4,096 tiles 183 / 177, 649 / 675, at 5,120 170 / 167, 493 / 524, at 6,500 168 / 162, 367 / 392, at
  // 8,160 165 / 156, 267 / 291; heavy overlap 710 / 678)
  const bool phi = b.falloff != GES_FALLOFF_GEF, few = b.total_tiles <= 4096;   // PHI and PHI_EXACT: Gaussian
  void (*kernel)(const DeviceBatch*, const uint2*, int64_t, uint64_t) =
      phi ? (few ? raster_forward_kernel<GES_FALLOFF_PHI, 4> : raster_forward_kernel<GES_FALLOFF_PHI, 2>)
          : (few ? raster_forward_kernel<GES_FALLOFF_GEF, 4> : raster_forward_kernel<GES_FALLOFF_GEF, 2>);
  hipLaunchKernelGGL(kernel, grid, dim3(64 * kFwdWaves), 0, stream, dbatch, b.sorted_pairs, b.total_tiles,
                     b.key_capacity);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(raster_stats_kernel, dim3((unsigned)b.nviews), dim3(1024), 0, stream, dbatch);
  return hipGetLastError();
}

hipError_t launch_raster_backward(const DeviceBatch* dbatch, const Batch& b, hipStream_t stream) {
  if (b.total_tiles == 0) return hipSuccess;
  const bool phi = b.falloff != GES_FALLOFF_GEF;
  if (!cut_walks(b)) {
    const int64_t span = 8 * kXcdGroup;   // the grid covers whole rounds of groups
    const dim3 grid((unsigned)((b.total_tiles + span - 1) / span * span));
    hipLaunchKernelGGL((phi ? raster_backward_kernel<GES_FALLOFF_PHI, false>
                            : raster_backward_kernel<GES_FALLOFF_GEF, false>),
                       grid, dim3(64), 0, stream, dbatch, b.sorted_pairs, b.total_tiles, nullptr, nullptr);
    return hipGetLastError();
  }
  const int64_t most = max_checkpoints(b.key_capacity);   // boundaries, hence cut tiles
  if (most > 0) {
    const dim3 grid((unsigned)std::min<int64_t>(b.total_tiles, most));
    hipLaunchKernelGGL((phi ? raster_recover_kernel<GES_FALLOFF_PHI> : raster_recover_kernel<GES_FALLOFF_GEF>), grid,
                       dim3(64 * kFwdWaves), 0, stream, dbatch, b.sorted_pairs, b.kw.table, b.kw.plan);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // a block per item, whichever XCD it belongs to, up to a few rounds of the device (the item counts are known
  // there only): blocks past the items leave at once, items past the blocks are taken in turn
  const int64_t blocks = std::min<int64_t>(8 * (b.total_tiles + most), 8192);
  hipLaunchKernelGGL((phi ? raster_backward_kernel<GES_FALLOFF_PHI, true> : raster_backward_kernel<GES_FALLOFF_GEF, true>),
                     dim3((unsigned)blocks), dim3(64), 0, stream, dbatch, b.sorted_pairs, b.total_tiles, b.kw.pv[1],
                     b.kw.plan);
  return hipGetLastError();
}

}  // namespace ges
