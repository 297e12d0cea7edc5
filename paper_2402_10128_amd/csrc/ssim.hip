// ssim.hip -- SSIM term of the GES training loss (lambda_ssim L_ssim, Sec. 4.4, Eq. final) and its gradient.
//
// Gaussian-weighted SSIM (Wang et al., 2004): 11x11 window (sigma 1.5, unit sum), each colour channel on its
// own, zero padding so the map has the image's size, C1 = 0.01^2, C2 = 0.03^2; L_ssim = 1 - mean SSIM over
// every pixel and channel.  The gradient goes through the five local statistics: with A, B, Cxy the
// derivatives of SSIM(p) with respect to w*x, w*x^2 and w*xy at p, d(sum_p SSIM)/dx(q) =
// (w*A)(q) + 2 x(q) (w*B)(q) + y(q) (w*Cxy)(q), w symmetric and zero-padded.
//
// Two tiled passes over tiles of 64 x 32 pixels of one channel, each staging the tile plus a 5-pixel halo in LDS and filtering
// separably (11 taps across, then 11 down; every sum in the order of the taps):
//   forward: the five statistics -> SSIM (summed per block) and the maps A, B, Cxy;
//   backward: the three maps filtered again -> dL/dI, added to the caller's gradient; one more block adds the
//            per-block sums in a fixed order to the loss.
// The statistics are taken of x - 1/2 and y - 1/2 (padding becomes -1/2): variances and covariances do not
// change under a common shift, and the second moments of values in [-1/2, 1/2] lose four times less to
// the cancellation in E[x^2] - E[x]^2.
//
// A thread filters 8 neighbouring outputs at a time: across, from 20 staged values by five 16-byte reads, so that the
// products x^2, y^2, xy are taken 18 times for 8 outputs; down, a column of 18 values.  Two statistics (one map) are
// filtered at a time, which keeps a block to 48 KB (24 KB) of LDS.  What bounds the forward is VALU issue (110
// multiply-adds per pixel and channel, 134 with the halo rows, about 230 instructions with the rest: 46 us at 1080p if every
// SIMD issued each cycle); the backward, latency of memory and LDS (175 MB at 1080p, 34 us at a copy's rate).  At 1080p the
// forward went from 64 us (32 x 32 tiles, a block's three channels in turn, staging indices divided out per value)
// to 58, the backward from 56 to 43, and the sum's own launch of 4.3 went away; at 512 x 512 it is
// 16.5 -> 16.0 and 13.0 -> 11.4.  The four quotients are IEEE divisions: reciprocals and one remainder step without their
// scaling took 56 us, and gave 0 where a denominator's reciprocal is subnormal.  Filtering down first, straight from memory in registers, and the sum of the
// variances as one statistic takes 39 + 34 us, but rounds differently: through Adam's moments a training step's
// result then moves by up to 1e-3.
//
// Memory per pixel and channel: the forward reads x, y (8 B) and writes three maps (12 B); the backward
// reads the maps (12 B), x, y and the gradient (12 B) and writes the gradient (4 B).  Tiles are dealt to the
// XCDs in bands so the halo re-reads, and a tile's channels' shares of its lines, hit L2.
#include <algorithm>
#include <cmath>

#include "ges_internal.h"

namespace ges {

constexpr int kSsimR = 5;
constexpr int kSsimTaps = 2 * kSsimR + 1;
constexpr int kSsimW = 64, kSsimH = 32;          // output tile
constexpr int kSsimInH = kSsimH + 2 * kSsimR;    // staged rows (42, of 74)
constexpr int kSsimRaw = 76;                     // pitch of a staged row: 16-byte aligned, neighbouring rows 12 banks apart
constexpr int kSsimMid = 68;                     // pitch of a row filtered across: 4 banks apart
constexpr int kSsimThreads = 256;
constexpr int kSsimHalo = 2 * kSsimR * kSsimInH;   // staged values beyond a wave's 64 columns
constexpr int kSsimRowsPer = (kSsimInH + 3) / 4, kSsimHaloPer = (kSsimHalo + kSsimThreads - 1) / kSsimThreads;
constexpr int kSsimStage = kSsimRowsPer + kSsimHaloPer;   // staged values per thread
constexpr int kSsimOut = 8;                      // neighbouring outputs of a thread, across and down
constexpr int kSsimSpan = kSsimOut + 2 * kSsimR; // values they read (18)
static_assert(kSsimW * kSsimH / kSsimOut == kSsimThreads && kSsimW == 64, "a thread's outputs down: a wave is a row");
constexpr float kSsimC1 = 0.01f * 0.01f, kSsimC2 = 0.03f * 0.03f;
constexpr float kSsimShift = 0.5f;

struct SsimWeights {
  float w[kSsimTaps];
};

// Workgroups are dealt to the 8 XCDs in turn (block b runs on XCD b mod 8), and each XCD has its own L2.
// Block b takes tile (b mod 8) * per + b / 8, so every XCD walks one contiguous band of tile rows and the
// halos that neighbouring tiles share are read through the same L2.  Returns -1 for the spare blocks.
// The channel is the fastest of them.
__device__ __forceinline__ int ssim_tile(int b, int ntiles, int& c) {
  const int per = (ntiles + 7) / 8;
  const int j = b >> 3, tile = (b & 7) * per + j / 3;
  c = j % 3;
  return (j < 3 * per && tile < ntiles) ? tile : -1;
}

// A thread's share of a staged tile: a wave takes every fourth row's first 64 columns (the row's address and its being
// inside the image are scalars), the last 10 columns of all rows are dealt out after them.  f(j, row, column, index of
// the image's row, x, inside) for each; row and x are 0 outside.
template <class F>
__device__ __forceinline__ void ssim_staged(int x0, int y0, int w, int h, const F& f) {
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const bool in_x = x0 + lane >= 0 && x0 + lane < w;
  const int ox = in_x ? x0 + lane : 0;
#pragma unroll
  for (int j = 0; j < kSsimRowsPer; ++j) {
    const int r = wave + 4 * j, gy = y0 + r;
    const bool in_y = gy >= 0 && gy < h && r < kSsimInH;
    f(j, r, lane, (int64_t)(in_y ? gy : 0) * w, ox, in_x && in_y);
  }
#pragma unroll
  for (int j = 0; j < kSsimHaloPer; ++j) {
    const int e = t + j * kSsimThreads, r = e / (2 * kSsimR), col = 64 + e % (2 * kSsimR);
    const int gx = x0 + col, gy = y0 + r;
    const bool in = e < kSsimHalo && gx >= 0 && gx < w && gy >= 0 && gy < h;
    f(kSsimRowsPer + j, r, col, (int64_t)(in ? gy : 0) * w, in ? gx : 0, in);
  }
}

// The 8 outputs across of value f(column) over 18 columns.
template <class F>
__device__ __forceinline__ void ssim_taps(const SsimWeights& wt, const F& f, float (&o)[kSsimOut]) {
  float v[kSsimSpan];
#pragma unroll
  for (int k = 0; k < kSsimSpan; ++k) v[k] = f(k);
#pragma unroll
  for (int q = 0; q < kSsimOut; ++q) {
    float acc = 0.f;
#pragma unroll
    for (int k = 0; k < kSsimTaps; ++k) acc = __builtin_fmaf(wt.w[k], v[q + k], acc);
    o[q] = acc;
  }
}

__device__ __forceinline__ void ssim_read(const float* row, float (&v)[20]) {
#pragma unroll
  for (int k = 0; k < 5; ++k) *reinterpret_cast<float4*>(&v[4 * k]) = *reinterpret_cast<const float4*>(row + 4 * k);
}

// One row's 8 outputs across: statistic S (0 x, 1 y, 2 x^2, 3 y^2, 4 xy).
template <int S>
__device__ __forceinline__ void ssim_across(const SsimWeights& wt, const float* x, const float* y, float* mid) {
  float a[20], b[20], o[kSsimOut];
  ssim_read(S == 1 || S == 3 ? y : x, a);
  if (S == 4) ssim_read(y, b);
  ssim_taps(wt, [&](int k) { return S < 2 ? a[k] : (S < 4 ? a[k] * a[k] : a[k] * b[k]); }, o);
  *reinterpret_cast<float4*>(mid) = make_float4(o[0], o[1], o[2], o[3]);
  *reinterpret_cast<float4*>(mid + 4) = make_float4(o[4], o[5], o[6], o[7]);
}

constexpr int kSsimStrips = kSsimInH * (kSsimW / kSsimOut);   // of 8 outputs across (336)

// Two statistics across (or S1 < 0: one), their strips dealt to the threads one after the other.
template <int S0, int S1>
__device__ __forceinline__ void ssim_rows(const SsimWeights& wt, const float (*sx)[kSsimRaw], const float (*sy)[kSsimRaw],
                                          float (*mid)[kSsimInH][kSsimMid]) {
  for (int i = threadIdx.x; i < (S1 < 0 ? 1 : 2) * kSsimStrips; i += kSsimThreads) {
    const bool second = i >= kSsimStrips;
    const int e = second ? i - kSsimStrips : i;
    const int r = e / (kSsimW / kSsimOut), col0 = kSsimOut * (e % (kSsimW / kSsimOut));
    if (!second) ssim_across<S0>(wt, &sx[r][col0], &sy[r][col0], &mid[0][r][col0]);
    else if (S1 >= 0) ssim_across<(S1 < 0 ? 0 : S1)>(wt, &sx[r][col0], &sy[r][col0], &mid[1][r][col0]);
  }
}

__device__ __forceinline__ void ssim_down(const SsimWeights& wt, const float (*mid)[kSsimMid], float (&o)[kSsimOut]) {
  const int col = threadIdx.x & 63, row0 = kSsimOut * (threadIdx.x >> 6);
  ssim_taps(wt, [&](int k) { return mid[row0 + k][col]; }, o);
}

__global__ void __launch_bounds__(kSsimThreads) ssim_fwd_kernel(const float* __restrict__ img,
                                                                const float* __restrict__ tgt, int w, int h,
                                                                const SsimWeights wt, float* __restrict__ maps,
                                                                double* __restrict__ partial, int tiles_x,
                                                                int ntiles) {
  __shared__ __align__(16) float sx[kSsimInH][kSsimRaw];
  __shared__ __align__(16) float sy[kSsimInH][kSsimRaw];
  __shared__ __align__(16) float mid[2][kSsimInH][kSsimMid];
  __shared__ double red[kSsimThreads / 64];
  int c;
  const int tile = ssim_tile(blockIdx.x, ntiles, c);
  if (tile < 0) return;
  const int t = threadIdx.x;
  const int x0 = (tile % tiles_x) * kSsimW - kSsimR, y0 = (tile / tiles_x) * kSsimH - kSsimR;
  const size_t plane = (size_t)w * h;
  {
    float ra[kSsimStage], rb[kSsimStage];
    ssim_staged(x0, y0, w, h, [&](int j, int, int, int64_t row, int x, bool in) {   // all loads first, then the LDS stores
      const float a = (img + 3 * row + c)[3u * (unsigned)x], b = (tgt + 3 * row + c)[3u * (unsigned)x];
      ra[j] = (in ? a : 0.f) - kSsimShift;   // padding is 0, i.e. -1/2 after the shift
      rb[j] = (in ? b : 0.f) - kSsimShift;
    });
    ssim_staged(x0, y0, w, h, [&](int j, int r, int col, int64_t, int, bool) {
      if (r < kSsimInH) {
        sx[r][col] = ra[j];
        sy[r][col] = rb[j];
      }
    });
  }
  __syncthreads();
  float st[5][kSsimOut];
  ssim_rows<0, 1>(wt, sx, sy, mid);
  __syncthreads();
  ssim_down(wt, mid[0], st[0]);
  ssim_down(wt, mid[1], st[1]);
  __syncthreads();
  ssim_rows<2, 3>(wt, sx, sy, mid);
  __syncthreads();
  ssim_down(wt, mid[0], st[2]);
  ssim_down(wt, mid[1], st[3]);
  __syncthreads();
  ssim_rows<4, -1>(wt, sx, sy, mid);
  __syncthreads();
  ssim_down(wt, mid[0], st[4]);
  float ssum = 0.f;
  const int gx = x0 + kSsimR + (t & 63), gy0 = y0 + kSsimR + kSsimOut * (t >> 6);
#pragma unroll
  for (int q = 0; q < kSsimOut; ++q) {
    if (gx >= w || gy0 + q >= h) continue;
    const float ex = st[0][q], ey = st[1][q], exx = st[2][q], eyy = st[3][q], exy = st[4][q];
    // shifted moments -> variances/covariance; means of the unshifted images
    const float vx = exx - ex * ex, vy = eyy - ey * ey, cxy = exy - ex * ey;
    const float mx = ex + kSsimShift, my = ey + kSsimShift;
    const float n1 = 2.f * mx * my + kSsimC1, n2 = 2.f * cxy + kSsimC2;
    const float d1 = mx * mx + my * my + kSsimC1, d2 = vx + vy + kSsimC2;
    const float inv = 1.f / (d1 * d2);
    const float s = n1 * n2 * inv;
    ssum += s;
    // derivatives with respect to the shifted statistics (the shift moves the mean term only)
    const float dA = 2.f * my * n2 * inv - 2.f * mx * s / d1 + 2.f * ex * s / d2 - 2.f * ey * n1 * inv;
    const float dB = -s / d2;
    const float dC = 2.f * n1 * inv;
    const size_t o = c * plane + (size_t)(gy0 + q) * w + gx;
    maps[o] = dA;
    maps[o + 3 * plane] = dB;
    maps[o + 6 * plane] = dC;
  }
  double d = (double)ssum;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) d += __shfl_xor(d, off, 64);
  if ((t & 63) == 0) red[t >> 6] = d;
  __syncthreads();
  if (t == 0) partial[3 * tile + c] = ((red[0] + red[1]) + red[2]) + red[3];
}

// loss += lam (1 - sum / count), the block sums added in a fixed order
__device__ __forceinline__ void ssim_final(const double* __restrict__ partial, int nb, double count, float lam,
                                           float* __restrict__ loss, double* red) {
  double s = 0.0;
  for (int k = threadIdx.x; k < nb; k += kSsimThreads) s += partial[k];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double total = ((red[0] + red[1]) + red[2]) + red[3];
    *loss = (float)((double)*loss + (double)lam * (1.0 - total / count));
  }
}

__global__ void __launch_bounds__(kSsimThreads) ssim_bwd_kernel(const float* __restrict__ img,
                                                                const float* __restrict__ tgt, int w, int h,
                                                                const SsimWeights wt, const float* __restrict__ maps,
                                                                float scale, float* __restrict__ dL, int tiles_x,
                                                                int ntiles, const double* __restrict__ partial,
                                                                double count, float lam, float* __restrict__ loss) {
  __shared__ __align__(16) float sm[kSsimInH][kSsimRaw];
  __shared__ __align__(16) float mid[1][kSsimInH][kSsimMid];
  if (blockIdx.x == gridDim.x - 1) {
    ssim_final(partial, 3 * ntiles, count, lam, loss, reinterpret_cast<double*>(sm));
    return;
  }
  int c;
  const int tile = ssim_tile(blockIdx.x, ntiles, c);
  if (tile < 0) return;
  const int t = threadIdx.x;
  const int x0 = (tile % tiles_x) * kSsimW - kSsimR, y0 = (tile / tiles_x) * kSsimH - kSsimR;
  const size_t plane = (size_t)w * h;
  float rv[kSsimStage];
  auto load = [&](int m) {
    const float* p = maps + (3 * m + c) * plane;
    ssim_staged(x0, y0, w, h, [&](int j, int, int, int64_t row, int x, bool in) {
      const float v = (p + row)[(unsigned)x];
      rv[j] = in ? v : 0.f;   // the maps are zero outside the image
    });
  };
  load(0);
  // the images and the gradient of the thread's outputs
  const int gx = x0 + kSsimR + (t & 63), gy0 = y0 + kSsimR + kSsimOut * (t >> 6);
  float xs[kSsimOut], ys[kSsimOut], gs[kSsimOut], f[3][kSsimOut];
#pragma unroll
  for (int q = 0; q < kSsimOut; ++q) {
    const size_t o = gx < w && gy0 + q < h ? 3 * ((size_t)(gy0 + q) * w + gx) + c : 0;
    xs[q] = img[o];
    ys[q] = tgt[o];
    gs[q] = dL[o];
  }
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    ssim_staged(x0, y0, w, h, [&](int j, int r, int col, int64_t, int, bool) {
      if (r < kSsimInH) sm[r][col] = rv[j];
    });
    __syncthreads();   // and the map before has been filtered down
    if (m < 2) load(m + 1);
    ssim_rows<0, -1>(wt, sm, sm, mid);
    __syncthreads();
    ssim_down(wt, mid[0], f[m]);
  }
#pragma unroll
  for (int q = 0; q < kSsimOut; ++q) {
    if (gx >= w || gy0 + q >= h) continue;
    const float x_ = xs[q] - kSsimShift, y_ = ys[q] - kSsimShift;
    const float g = f[0][q] + 2.f * x_ * f[1][q] + y_ * f[2][q];
    dL[3 * ((size_t)(gy0 + q) * w + gx) + c] = gs[q] - scale * g;
  }
}

static size_t ssim_tiles(int w, int h) {
  return (size_t)((w + kSsimW - 1) / kSsimW) * (size_t)((h + kSsimH - 1) / kSsimH);
}

size_t ssim_scratch_bytes(int w, int h) {
  const size_t maps = 9 * (size_t)w * h * sizeof(float);
  return ((maps + 255) / 256) * 256 + 3 * ssim_tiles(w, h) * sizeof(double);
}

hipError_t launch_ssim_loss(const float* img, const float* target, int w, int h, float lam, void* scratch,
                            float* loss, float* dL, hipStream_t stream) {
  SsimWeights wt;
  double g[kSsimTaps], sum = 0.0;
  for (int k = 0; k < kSsimTaps; ++k) {
    const double d = (double)(k - kSsimR);
    g[k] = std::exp(-d * d / (2.0 * 1.5 * 1.5));
    sum += g[k];
  }
  for (int k = 0; k < kSsimTaps; ++k) wt.w[k] = (float)(g[k] / sum);
  float* maps = reinterpret_cast<float*>(scratch);
  const size_t maps_bytes = ((9 * (size_t)w * h * sizeof(float) + 255) / 256) * 256;
  double* partial = reinterpret_cast<double*>(reinterpret_cast<char*>(scratch) + maps_bytes);
  const int tiles_x = (w + kSsimW - 1) / kSsimW;
  const int ntiles = (int)ssim_tiles(w, h);
  const unsigned blocks = 3 * 8 * ((ntiles + 7) / 8);
  const double count = 3.0 * (double)w * (double)h;
  hipLaunchKernelGGL(ssim_fwd_kernel, dim3(blocks), dim3(kSsimThreads), 0, stream, img, target, w, h, wt, maps, partial,
                     tiles_x, ntiles);
  hipLaunchKernelGGL(ssim_bwd_kernel, dim3(blocks + 1), dim3(kSsimThreads), 0, stream, img, target, w, h, wt,
                     (const float*)maps, (float)((double)lam / count), dL, tiles_x, ntiles, (const double*)partial, count,
                     lam, loss);
  return hipGetLastError();
}

}  // namespace ges
