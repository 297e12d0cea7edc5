// ssim.hip -- SSIM term of the GES training loss (lambda_ssim L_ssim, Sec. 4.4, Eq. final) and its gradient.
//
// Gaussian-weighted SSIM (Wang et al., 2004): 11x11 window (sigma 1.5, unit sum), each colour channel on its
// own, zero padding so the map has the image's size, C1 = 0.01^2, C2 = 0.03^2; L_ssim = 1 - mean SSIM over
// every pixel and channel.  The gradient goes through the five local statistics: with A, B, Cxy the
// derivatives of SSIM(p) with respect to w*x, w*x^2 and w*xy at p, d(sum_p SSIM)/dx(q) =
// (w*A)(q) + 2 x(q) (w*B)(q) + y(q) (w*Cxy)(q), w symmetric and zero-padded.
//
// Two tiled passes over tiles of 160 x 8 pixels, each filtering separably (11 taps down, then 11 across):
//   forward: four statistics of every channel (w*x, w*y, w*(x^2+y^2), w*xy: SSIM and its derivatives take the two
//            variances as their sum) -> SSIM (summed per block) and the maps A, B, Cxy;
//   backward: the three maps filtered -> dL/dI, added to the caller's gradient; one more block adds the
//            per-block sums in a fixed order to the loss.
// The statistics are taken of x - 1/2 and y - 1/2 (padding becomes -1/2): variances and covariances do not
// change under a common shift, and the second moments of values in [-1/2, 1/2] lose four times less to
// the cancellation in E[x^2] - E[x]^2.
//
// The pass down runs straight from memory in registers: a thread owns one staged column of one channel (160 + 10
// columns x 3 channels = 510 of 512 threads; for the images these are 510 neighbouring floats of each row) and adds every
// row it reads to the up to 8 outputs the row is a tap of, so no value is staged twice and the products x^2 + y^2 and
// xy are taken once.  Its results go to LDS by channel, where the pass across reads 16 values by four 16-byte
// reads for 4 outputs.  What bounds the forward is its arithmetic (88 multiply-adds per pixel and channel, about 140
// instructions with the rest, 28 us at 1080p if every SIMD issued each cycle); the backward, memory (maps, images
// and gradient, 175 MB at 1080p, at 5.1 TB/s).  At 1080p the forward went from 60 us (32 x 32 tiles staged a channel at a
// time, across first, five statistics) to 39, the backward from 55 to 34 and the sum's own launch of 4.3 went away;
// at 512 x 512 it is 16.4 -> 9.5 and 13.7 -> 8.1.  Tiles of 4 or 6 rows took as long together; sending the backward's
// results through LDS once more, to meet images and gradient in memory's order, gained nothing.
//
// Memory per pixel and channel: the forward reads x, y (8 B) and writes three maps (12 B); the backward
// reads the maps (12 B), x, y and the gradient (12 B) and writes the gradient (4 B).  Tiles are dealt to the
// XCDs in bands so the halo re-reads hit L2.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "ges_internal.h"

namespace ges {

constexpr int kSsimR = 5;
constexpr int kSsimTaps = 2 * kSsimR + 1;
constexpr int kSsimT = 160, kSsimRows = 8;       // output tile
constexpr int kSsimCols = kSsimT + 2 * kSsimR;   // its columns with the halo (170)
constexpr int kSsimThreads = 512;
constexpr int kSsimIn = kSsimRows + 2 * kSsimR;  // rows a column is read over (18)
constexpr int kSsimPitch = 172;                  // of a row in LDS, 16-byte aligned
// Distance of the channels' planes in LDS.  The pass down writes (column, channel) = (t / 3, t mod 3) and the pass across
// reads 16 bytes at (quad, channel) alike, so three planes are in use at a time: 20 banks of 64 apart, the 22
// columns or 3 quads of a group of lanes fall on different banks in each.
constexpr int kSsimPlane = kSsimRows * kSsimPitch + 52;
static_assert(kSsimPlane % 64 == 20 && kSsimPitch >= kSsimCols + 2 && 3 * kSsimCols <= kSsimThreads, "");
constexpr int kSsimQuads = kSsimT / 4;
constexpr int kSsimTasks = 3 * kSsimQuads * kSsimRows;   // 4 neighbouring outputs of a channel each
constexpr float kSsimC1 = 0.01f * 0.01f, kSsimC2 = 0.03f * 0.03f;
constexpr float kSsimShift = 0.5f;

struct SsimWeights {
  float w[kSsimTaps];
};

// Workgroups are dealt to the 8 XCDs in turn (block b runs on XCD b mod 8), and each XCD has its own L2.
// Block b takes tile (b mod 8) * per + b / 8, so every XCD walks one contiguous band of tile rows and the
// halos that neighbouring tiles share are read through the same L2.  Returns -1 for the spare blocks.
__device__ __forceinline__ int ssim_tile(int b, int ntiles) {
  const int per = (ntiles + 7) / 8;
  const int j = b >> 3, tile = (b & 7) * per + j;
  return (j < per && tile < ntiles) ? tile : -1;
}

// Adds the value of input row k to the outputs it is a tap of.
template <int K, int N>
__device__ __forceinline__ void ssim_tap(const SsimWeights& wt, const float (&v)[N], float (&acc)[N][kSsimRows]) {
#pragma unroll
  for (int q = 0; q < kSsimRows; ++q)
    if (K - q >= 0 && K - q < kSsimTaps) {
#pragma unroll
      for (int s = 0; s < N; ++s) acc[s][q] = __builtin_fmaf(wt.w[K - q], v[s], acc[s][q]);
    }
}

// The pass across for the 4 outputs from column col0 (a multiple of 4) of a row in LDS.
__device__ __forceinline__ void ssim_across(const SsimWeights& wt, const float* row, float (&o)[4]) {
  float v[16];
#pragma unroll
  for (int k = 0; k < 4; ++k) *reinterpret_cast<float4*>(&v[4 * k]) = *reinterpret_cast<const float4*>(row + 4 * k);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float acc = 0.f;
#pragma unroll
    for (int k = 0; k < kSsimTaps; ++k) acc = __builtin_fmaf(wt.w[k], v[q + k], acc);
    o[q] = acc;
  }
}

template <int K>
struct SsimRow {   // rows 0 .. K of a column, in order
  template <class F>
  static __device__ __forceinline__ void each(const F& f) {
    SsimRow<K - 1>::each(f);
    f(std::integral_constant<int, K>());
  }
};
template <>
struct SsimRow<-1> {
  template <class F>
  static __device__ __forceinline__ void each(const F&) {}
};

__global__ void __launch_bounds__(kSsimThreads) ssim_fwd_kernel(const float* __restrict__ img,
                                                                const float* __restrict__ tgt, int w, int h,
                                                                const SsimWeights wt, float* __restrict__ maps,
                                                                int pitch, double* __restrict__ partial, int tiles_x,
                                                                int ntiles) {
  __shared__ __align__(16) float hs[4 * 3 * kSsimPlane];
  __shared__ double red[kSsimThreads / 64];
  const int tile = ssim_tile(blockIdx.x, ntiles);
  if (tile < 0) return;
  const int t = threadIdx.x;
  const int x0 = (tile % tiles_x) * kSsimT, y0 = (tile / tiles_x) * kSsimRows;
  const size_t line = 3 * (size_t)w;
  if (t < 3 * kSsimCols) {   // down
    const int64_t fx = 3 * (int64_t)(x0 - kSsimR) + t;
    const bool in_x = fx >= 0 && fx < (int64_t)line;
    const unsigned fo = in_x ? (unsigned)fx : 0u;
    float xv[kSsimIn], yv[kSsimIn];
#pragma unroll
    for (int k = 0; k < kSsimIn; ++k) {
      const int gy = min(max(y0 - kSsimR + k, 0), h - 1);
      xv[k] = (img + gy * line)[fo];
      yv[k] = (tgt + gy * line)[fo];
    }
    float acc[4][kSsimRows] = {};
    SsimRow<kSsimIn - 1>::each([&](auto K) {
      constexpr int k = decltype(K)::value;
      const int gy = y0 - kSsimR + k;
      const bool in = in_x && gy >= 0 && gy < h;   // padding is 0, i.e. -1/2 after the shift
      const float x = (in ? xv[k] : 0.f) - kSsimShift, y = (in ? yv[k] : 0.f) - kSsimShift;
      const float v[4] = {x, y, __builtin_fmaf(x, x, y * y), x * y};
      ssim_tap<k>(wt, v, acc);
    });
    const int c = t % 3, col = t / 3;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int q = 0; q < kSsimRows; ++q) hs[(s * 3 + c) * kSsimPlane + q * kSsimPitch + col] = acc[s][q];
  }
  __syncthreads();
  const size_t plane = (size_t)pitch * h;
  float ssum = 0.f;
  for (int i = t; i < kSsimTasks; i += kSsimThreads) {   // across
    const int c = i % 3, col0 = 4 * (i / 3 % kSsimQuads), row = i / (3 * kSsimQuads);
    const int gx = x0 + col0, gy = y0 + row;
    if (gx >= w || gy >= h) continue;
    float st[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) ssim_across(wt, &hs[(s * 3 + c) * kSsimPlane + row * kSsimPitch + col0], st[s]);
    float dA[4], dB[4], dC[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float ex = st[0][q], ey = st[1][q], e2 = st[2][q], exy = st[3][q];
      // shifted moments -> sum of variances, covariance; means of the unshifted images
      const float v = __builtin_fmaf(-ey, ey, __builtin_fmaf(-ex, ex, e2)), cxy = __builtin_fmaf(-ex, ey, exy);
      const float mx = ex + kSsimShift, my = ey + kSsimShift;
      const float n1 = __builtin_fmaf(2.f * mx, my, kSsimC1), n2 = __builtin_fmaf(2.f, cxy, kSsimC2);
      const float d1 = __builtin_fmaf(mx, mx, __builtin_fmaf(my, my, kSsimC1)), d2 = v + kSsimC2;
      const float inv = 1.f / (d1 * d2);
      const float a1 = n1 * inv, a2 = n2 * inv, s = n1 * a2;
      const float s1 = s * (d2 * inv), s2 = s * (d1 * inv);   // s / d1, s / d2
      if (gx + q < w) ssum += s;
      // derivatives with respect to the shifted statistics (the shift moves the mean term only)
      dA[q] = 2.f * (my * a2 - mx * s1 + ex * s2 - ey * a1);
      dB[q] = -s2;
      dC[q] = 2.f * a1;
    }
    float* o = maps + c * plane + (size_t)gy * pitch + gx;   // columns up to the pitch are written and never used
    *reinterpret_cast<float4*>(o) = make_float4(dA[0], dA[1], dA[2], dA[3]);
    *reinterpret_cast<float4*>(o + 3 * plane) = make_float4(dB[0], dB[1], dB[2], dB[3]);
    *reinterpret_cast<float4*>(o + 6 * plane) = make_float4(dC[0], dC[1], dC[2], dC[3]);
  }
  double d = (double)ssum;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) d += __shfl_xor(d, off, 64);
  if ((t & 63) == 0) red[t >> 6] = d;
  __syncthreads();
  if (t == 0) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kSsimThreads / 64; ++k) s += red[k];
    partial[tile] = s;
  }
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
    double total = 0.0;
    for (int k = 0; k < kSsimThreads / 64; ++k) total += red[k];
    *loss = (float)((double)*loss + (double)lam * (1.0 - total / count));
  }
}

__global__ void __launch_bounds__(kSsimThreads) ssim_bwd_kernel(const float* __restrict__ img,
                                                                const float* __restrict__ tgt, int w, int h,
                                                                const SsimWeights wt, const float* __restrict__ maps,
                                                                int pitch, float scale, float* __restrict__ dL,
                                                                int tiles_x, int ntiles,
                                                                const double* __restrict__ partial, double count,
                                                                float lam, float* __restrict__ loss) {
  __shared__ __align__(16) float hs[3 * 3 * kSsimPlane];
  if (blockIdx.x == gridDim.x - 1) {
    ssim_final(partial, ntiles, count, lam, loss, reinterpret_cast<double*>(hs));
    return;
  }
  const int tile = ssim_tile(blockIdx.x, ntiles);
  if (tile < 0) return;
  const int t = threadIdx.x;
  const int x0 = (tile % tiles_x) * kSsimT, y0 = (tile / tiles_x) * kSsimRows;
  const size_t plane = (size_t)pitch * h;
  if (t < 3 * kSsimCols) {   // down: the maps are zero outside the image
    const int c = t / kSsimCols, col = t - c * kSsimCols;
    const int gx = x0 - kSsimR + col;
    const bool in_x = gx >= 0 && gx < w;
    const float* p = maps + c * plane + (in_x ? gx : 0);
    float mv[3][kSsimIn];
#pragma unroll
    for (int k = 0; k < kSsimIn; ++k) {
      const size_t o = (size_t)min(max(y0 - kSsimR + k, 0), h - 1) * pitch;
#pragma unroll
      for (int m = 0; m < 3; ++m) mv[m][k] = p[o + 3 * m * plane];
    }
    float acc[3][kSsimRows] = {};
    SsimRow<kSsimIn - 1>::each([&](auto K) {
      constexpr int k = decltype(K)::value;
      const int gy = y0 - kSsimR + k;
      const bool in = in_x && gy >= 0 && gy < h;
      const float v[3] = {in ? mv[0][k] : 0.f, in ? mv[1][k] : 0.f, in ? mv[2][k] : 0.f};
      ssim_tap<k>(wt, v, acc);
    });
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
      for (int q = 0; q < kSsimRows; ++q) hs[(m * 3 + c) * kSsimPlane + q * kSsimPitch + col] = acc[m][q];
  }
  __syncthreads();
  for (int i = t; i < kSsimTasks; i += kSsimThreads) {   // across; channels in neighbouring lanes share their lines
    const int c = i % 3, col0 = 4 * (i / 3 % kSsimQuads), row = i / (3 * kSsimQuads);
    const int gx = x0 + col0, gy = y0 + row;
    if (gx >= w || gy >= h) continue;
    const size_t o = 3 * ((size_t)gy * w + gx) + c;
    float x[4], y[4], g[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const size_t oq = gx + q < w ? o + 3 * q : o;
      x[q] = img[oq] - kSsimShift;
      y[q] = tgt[oq] - kSsimShift;
      g[q] = dL[oq];
    }
    float f[3][4];
#pragma unroll
    for (int m = 0; m < 3; ++m) ssim_across(wt, &hs[(m * 3 + c) * kSsimPlane + row * kSsimPitch + col0], f[m]);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (gx + q < w)
        dL[o + 3 * q] = g[q] - scale * __builtin_fmaf(y[q], f[2][q], __builtin_fmaf(2.f * x[q], f[1][q], f[0][q]));
  }
}

static size_t ssim_blocks(int w, int h) {
  return (size_t)((w + kSsimT - 1) / kSsimT) * (size_t)((h + kSsimRows - 1) / kSsimRows);
}

// The maps' rows are padded to 16 bytes and start at the first such address of the caller's scratch.
static size_t ssim_map_bytes(int w, int h) {
  const size_t pitch = ((size_t)w + 3) / 4 * 4;
  return (9 * pitch * h * sizeof(float) + 255) / 256 * 256;
}

size_t ssim_scratch_bytes(int w, int h) {
  return ssim_map_bytes(w, h) + ssim_blocks(w, h) * sizeof(double) + 16;
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
  float* maps = reinterpret_cast<float*>((reinterpret_cast<uintptr_t>(scratch) + 15) & ~(uintptr_t)15);
  double* partial = reinterpret_cast<double*>(reinterpret_cast<char*>(maps) + ssim_map_bytes(w, h));
  const int pitch = (w + 3) / 4 * 4;
  const int tiles_x = (w + kSsimT - 1) / kSsimT;
  const int ntiles = (int)ssim_blocks(w, h);
  const unsigned blocks = 8 * ((ntiles + 7) / 8);
  const double count = 3.0 * (double)w * (double)h;
  hipLaunchKernelGGL(ssim_fwd_kernel, dim3(blocks), dim3(kSsimThreads), 0, stream, img, target, w, h, wt, maps, pitch,
                     partial, tiles_x, ntiles);
  hipLaunchKernelGGL(ssim_bwd_kernel, dim3(blocks + 1), dim3(kSsimThreads), 0, stream, img, target, w, h, wt,
                     (const float*)maps, pitch, (float)((double)lam / count), dL, tiles_x, ntiles,
                     (const double*)partial, count, lam, loss);
  return hipGetLastError();
}

}  // namespace ges
