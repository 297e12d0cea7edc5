// loss.hip -- frequency-modulated L1 loss of GES (Sec. 4.3) and its gradient.
//
// Mask (made per target and omega; the training step remakes it every iteration as omega grows):
//   grey = (r + g + b) / 3, area-down-sampled by 5 (image Laplacian scale 0.2, App. B.2);
//   DoG = G(grey, sigma1) - G(grey, sigma2), sigma2 = 0.1 + 10 omega, sigma1 = 2 sigma2 (Eq. mask),
//   separable normalised Gaussians of radius ceil(3 sigma) with replicated borders;
//   M = |DoG| / max|DoG| > 0.5 (an all-zero mask when max|DoG| <= 1e-5), up-sampled by nearest lookup;
//   for omega <= 0.5, M = 1 - M_(omega+0.5), M_(omega+0.5) taken directly (omega = 0 as the limit from above).
// Loss: L = lam_l1 mean|I - T| + lam_w mean(|I - T| M) (Eq. laplace, Eq. final without the SSIM term),
//   dL/dI = (lam_l1 + lam_w M) sign(I - T) / (3 h w).  The per-block partial sums are added in a
//   fixed order by one block, so the loss is deterministic.
// Memory: the loss reads I, T (12 B/px each) and M (1 B/px) and writes dL/dI (12 B/px): HBM-bound.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "ges_internal.h"

namespace ges {

constexpr int kScale = 5;
constexpr int kMaxTaps = 2 * 64 + 1;   // supports sigma up to 21 (omega <= 1)

// Blur weights of both Gaussians, made on the host and passed by value (they land in the kernel-argument
// segment and are read with scalar loads).
struct MaskWeights {
  float w1[kMaxTaps];
  float w2[kMaxTaps];
  int r1, r2;
};

size_t freq_mask_scratch_bytes(int w, int h) {
  const size_t wl = (size_t)(w + kScale - 1) / kScale, hl = (size_t)(h + kScale - 1) / kScale;
  return 768 + 4 * wl * hl * sizeof(float);
}

static void mask_weights(MaskWeights& mw, float s1, float s2) {
  for (int which = 0; which < 2; ++which) {
    const double s = which == 0 ? s1 : s2;
    const int R = (int)std::ceil(3.0 * (double)(which == 0 ? s1 : s2));
    float* w = which == 0 ? mw.w1 : mw.w2;
    double sum = 0.0;
    for (int k = -R; k <= R; ++k) sum += std::exp(-(double)(k * k) / (2.0 * s * s));
    for (int k = -R; k <= R; ++k) w[k + R] = (float)(std::exp(-(double)(k * k) / (2.0 * s * s)) / sum);
    if (which == 0) mw.r1 = R; else mw.r2 = R;
  }
}

// The mask is three launches (four where it has more than kMaxInline tiles), each a few microseconds of latency more than
// of work: a kernel asks for all it reads at once, stages it in LDS and walks the up to 129 taps there.  1080p, omega
// 0.75: 41 -> 21 us; 512 x 512: 29 -> 17.  The four kernels before took the taps from memory, 8 in flight, and the
// maximum by 648 atomics on one address.  Every sum runs in the order of the pixels or taps.
constexpr int kRowThreads = 1024;
constexpr int kRowSegment = 1024;                          // low pixels of a row per block: images up to 5,120 wide in one
constexpr int kRowChunk = 512;                             // low pixels averaged at a time
constexpr int kRowAhead = 2;                               // x 5 rows: pixels a thread has in flight

// The weights to LDS, all at once: read where they are used, from the kernel's arguments, each line of 16 is a wait of its
// own for memory.
__device__ __forceinline__ void stage_weights(const MaskWeights& mw, float (&ws)[2][kMaxTaps + 3]) {
  for (int k = threadIdx.x; k < 2 * kMaxTaps; k += blockDim.x) {
    const int which = k >= kMaxTaps ? 1 : 0, e = k - which * kMaxTaps;
    ws[which][e] = (which ? mw.w2 : mw.w1)[e];
  }
}

// Grey, down-sampled row and the horizontal pass of both blurs.
__global__ void __launch_bounds__(kRowThreads) mask_rows_kernel(const MaskWeights mw, const float* __restrict__ img, int w,
                                                                int h, int wl, float* __restrict__ h1,
                                                                float* __restrict__ h2) {
  __shared__ float grey[kScale][kRowChunk * kScale];
  __shared__ float low[kRowSegment + kMaxTaps - 1];
  __shared__ __align__(16) float ws[2][kMaxTaps + 3];
  const int t = threadIdx.x, y = blockIdx.y;
  stage_weights(mw, ws);
  const int xs = blockIdx.x * kRowSegment, xe = min(xs + kRowSegment, wl);
  const int R = max(mw.r1, mw.r2);
  const int a = max(xs - R, 0), b = min(xe + R, wl);       // low pixels this block needs
  const int rows = min(kScale, h - y * kScale);
  for (int c0 = a; c0 < b; c0 += kRowChunk) {
    const int nlow = min(kRowChunk, b - c0), px0 = c0 * kScale, npx = min(nlow * kScale, w - px0);
    const float* base = img + 3 * ((size_t)(y * kScale) * w + px0);
    for (int p0 = 0; p0 < npx; p0 += kRowThreads * kRowAhead) {
      float v[kRowAhead][kScale];
#pragma unroll
      for (int j = 0; j < kRowAhead; ++j)
#pragma unroll
        for (int r = 0; r < kScale; ++r) {
          const float* q = base + 3 * ((size_t)min(r, rows - 1) * w + min(p0 + j * kRowThreads + t, npx - 1));
          v[j][r] = (q[0] + q[1] + q[2]) * (1.f / 3.f);
        }
#pragma unroll
      for (int j = 0; j < kRowAhead; ++j) {
        const int p = p0 + j * kRowThreads + t;
        if (p < npx)
#pragma unroll
          for (int r = 0; r < kScale; ++r) grey[r][p] = v[j][r];
      }
    }
    __syncthreads();
    if (t < nlow) {
      const int cols = min(kScale, npx - t * kScale);
      float acc = 0.f;
      if (rows == kScale && cols == kScale) {
#pragma unroll
        for (int e = 0; e < kScale * kScale; ++e) acc += grey[e / kScale][t * kScale + e % kScale];
      } else {
        for (int dy = 0; dy < rows; ++dy)
          for (int dx = 0; dx < cols; ++dx) acc += grey[dy][t * kScale + dx];
      }
      low[c0 - a + t] = acc / (float)(rows * cols);
    }
    __syncthreads();
  }
  for (int x = xs + t; x < xe; x += kRowThreads) {
    float a1 = 0.f, a2 = 0.f;
#pragma unroll 8
    for (int k = 0; k <= 2 * mw.r1; ++k) a1 += ws[0][k] * low[min(max(x - mw.r1 + k, 0), wl - 1) - a];
#pragma unroll 8
    for (int k = 0; k <= 2 * mw.r2; ++k) a2 += ws[1][k] * low[min(max(x - mw.r2 + k, 0), wl - 1) - a];
    h1[(size_t)y * wl + x] = a1;
    h2[(size_t)y * wl + x] = a2;
  }
}

constexpr int kColTileX = 32, kColTileY = 16;
constexpr int kColThreads = kColTileX * kColTileY;
constexpr int kColSpan = kColTileY + kMaxTaps - 1;         // rows a tile reads
constexpr int kMaxInline = 512;                            // tile maxima that mask_up_kernel's waves take themselves

// The largest of non-negative floats: they order like their bits.
__device__ __forceinline__ unsigned wave_max_bits(unsigned m) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, off, 64));
  return m;
}

// Vertical pass, |DoG| and the tile's largest, over the responses that are numbers: one NaN in the target would otherwise
// take the mask of the whole image (its bits are above all).
__global__ void __launch_bounds__(kColThreads) mask_cols_kernel(const MaskWeights mw, const float* __restrict__ h1,
                                                                const float* __restrict__ h2, int wl, int hl,
                                                                float* __restrict__ dog, unsigned* __restrict__ tile_max) {
  __shared__ float s1[kColSpan][kColTileX];
  __shared__ float s2[kColSpan][kColTileX];
  __shared__ unsigned wmax[kColThreads / 64];
  __shared__ __align__(16) float ws[2][kMaxTaps + 3];
  const int t = threadIdx.x, tx = t % kColTileX, ty = t / kColTileX;
  const int x = blockIdx.x * kColTileX + tx, y0 = blockIdx.y * kColTileY;
  const int n1 = kColTileY + 2 * mw.r1, n2 = kColTileY + 2 * mw.r2;
  stage_weights(mw, ws);
  {
    constexpr int kPer = (kColSpan + kColTileY - 1) / kColTileY;
    float v1[kPer], v2[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {   // rows outside the image repeat its edge
      const int r = ty + j * kColTileY;
      const size_t xc = min(x, wl - 1);
      v1[j] = r < n1 ? h1[(size_t)min(max(y0 - mw.r1 + r, 0), hl - 1) * wl + xc] : 0.f;
      v2[j] = r < n2 ? h2[(size_t)min(max(y0 - mw.r2 + r, 0), hl - 1) * wl + xc] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int r = ty + j * kColTileY;
      if (r < n1) s1[r][tx] = v1[j];
      if (r < n2) s2[r][tx] = v2[j];
    }
  }
  __syncthreads();
  float d = 0.f;
  if (x < wl && y0 + ty < hl) {
    float a1 = 0.f, a2 = 0.f;
#pragma unroll 8
    for (int k = 0; k <= 2 * mw.r1; ++k) a1 += ws[0][k] * s1[ty + k][tx];
#pragma unroll 8
    for (int k = 0; k <= 2 * mw.r2; ++k) a2 += ws[1][k] * s2[ty + k][tx];
    d = fabsf(a1 - a2);
    dog[(size_t)(y0 + ty) * wl + x] = d;
  }
  const unsigned m = wave_max_bits(d == d ? __float_as_uint(d) : 0u);
  if ((t & 63) == 0) wmax[t >> 6] = m;
  __syncthreads();
  if (t == 0) {
    unsigned b = wmax[0];
    for (int k = 1; k < kColThreads / 64; ++k) b = max(b, wmax[k]);
    tile_max[blockIdx.y * gridDim.x + blockIdx.x] = b;
  }
}

__global__ void __launch_bounds__(1024) mask_max_kernel(unsigned* __restrict__ tile_max, int n) {
  __shared__ unsigned wmax[16];
  unsigned m = 0;
  for (int k = threadIdx.x; k < n; k += 1024) m = max(m, tile_max[k]);
  m = wave_max_bits(m);
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 0; k < 16; ++k) m = max(m, wmax[k]);
    tile_max[0] = m;
  }
}

// Four neighbouring pixels of a row per thread; they lie over at most two low pixels.  words: a row's bytes can be stored
// four at a time (the mask and its rows start at multiples of 4).
__global__ void __launch_bounds__(256) mask_up_kernel(const unsigned* __restrict__ tile_max, int ntiles,
                                                      const float* __restrict__ dog, int wl, int w, int invert, int words,
                                                      uint8_t* __restrict__ mask) {
  const int x = 4 * (blockIdx.x * 256 + threadIdx.x), y = blockIdx.y;
  unsigned bits = 0;
  for (int k = threadIdx.x & 63; k < ntiles; k += 64) bits = max(bits, tile_max[k]);
  const float m = __uint_as_float(wave_max_bits(bits));
  if (x >= w) return;
  const float* row = dog + (size_t)(y / kScale) * wl;
  const int l0 = x / kScale, l1 = min(l0 + 1, wl - 1);
  unsigned b0 = 0, b1 = 0;
  if (m > 1e-5f) {
    b0 = row[l0] / m > 0.5f ? 1 : 0;
    b1 = row[l1] / m > 0.5f ? 1 : 0;
  }
  if (invert) {
    b0 ^= 1;
    b1 ^= 1;
  }
  const int split = (l0 + 1) * kScale - x;   // pixels of the first
  unsigned v = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) v |= (q < split ? b0 : b1) << (8 * q);
  uint8_t* o = mask + (size_t)y * w + x;
  if (words) {
    *reinterpret_cast<unsigned*>(o) = v;
  } else {
    for (int q = 0; q < 4 && x + q < w; ++q) o[q] = (uint8_t)(v >> (8 * q));
  }
}

hipError_t launch_freq_mask(const float* target, int w, int h, float omega, void* scratch, uint8_t* mask,
                            hipStream_t stream) {
  const bool invert = omega <= 0.5f;
  const float om = invert ? omega + 0.5f : omega;
  const float s2 = 0.1f + 10.f * om, s1 = 2.f * s2;
  const int wl = (w + kScale - 1) / kScale, hl = (h + kScale - 1) / kScale;
  float* h1 = reinterpret_cast<float*>(reinterpret_cast<char*>(scratch) + 256);
  float* h2 = h1 + (size_t)wl * hl;
  float* dog = h2 + (size_t)wl * hl;
  unsigned* tile_max = reinterpret_cast<unsigned*>(dog + (size_t)wl * hl);   // at most one a low pixel
  MaskWeights mw;
  mask_weights(mw, s1, s2);
  const dim3 tiles((wl + kColTileX - 1) / kColTileX, (hl + kColTileY - 1) / kColTileY);
  int ntiles = (int)(tiles.x * tiles.y);
  hipLaunchKernelGGL(mask_rows_kernel, dim3((wl + kRowSegment - 1) / kRowSegment, hl), dim3(kRowThreads), 0, stream, mw,
                     target, w, h, wl, h1, h2);
  hipLaunchKernelGGL(mask_cols_kernel, tiles, dim3(kColThreads), 0, stream, mw, h1, h2, wl, hl, dog, tile_max);
  if (ntiles > kMaxInline) {
    hipLaunchKernelGGL(mask_max_kernel, dim3(1), dim3(1024), 0, stream, tile_max, ntiles);
    ntiles = 1;
  }
  const int words = (w % 4 == 0 && reinterpret_cast<uintptr_t>(mask) % 4 == 0) ? 1 : 0;
  hipLaunchKernelGGL(mask_up_kernel, dim3((w + 1023) / 1024, h), dim3(256), 0, stream, tile_max, ntiles, dog, wl, w,
                     invert ? 1 : 0, words, mask);
  return hipGetLastError();
}

// ---- the mask with library-held scratch (no scratch argument, no allocation) -------------------
// One fixed array per device; its device address is looked up once per device, with that device
// current, and kept.  Host code never passes the array's own name to a kernel (on the host that name is a
// stand-in, not a device address): every use goes through the looked-up pointer.
constexpr size_t kMaskStaticBytes = GES_MASK_STATIC_SCRATCH_BYTES;
constexpr int kMaxStaticDevices = 64;
static __device__ __align__(256) unsigned char mask_static_scratch[kMaskStaticBytes];

namespace {
std::mutex g_static_mu;
void* g_static_ptr[kMaxStaticDevices] = {};
}  // namespace

size_t freq_mask_static_capacity() { return kMaskStaticBytes; }

hipError_t launch_freq_mask_static(const float* target, int w, int h, float omega, uint8_t* mask,
                                   hipStream_t stream) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxStaticDevices) return hipErrorInvalidDevice;
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_static_mu);
    if (!g_static_ptr[dev]) {
      e = hipGetSymbolAddress(&g_static_ptr[dev], HIP_SYMBOL(mask_static_scratch));
      if (e != hipSuccess) {
        g_static_ptr[dev] = nullptr;
        return e;
      }
    }
    ptr = g_static_ptr[dev];
  }
  // the mask's kernels write whatever they read of the scratch, so nothing has to start at zero
  return launch_freq_mask(target, w, h, omega, ptr, mask, stream);
}

constexpr int kLossThreads = 256;
constexpr int kLossBlocks = 1024;

__global__ void __launch_bounds__(kLossThreads) loss_kernel(const float* __restrict__ img,
                                                            const float* __restrict__ tgt,
                                                            const uint8_t* __restrict__ mask, int64_t npix,
                                                            float lam_l1, float lam_w, float* __restrict__ dL,
                                                            float* __restrict__ partial) {
  __shared__ float red[kLossThreads / 64];
  const float inv_n = 1.f / (3.f * (float)npix);
  float acc = 0.f;
  for (int64_t p = (int64_t)blockIdx.x * kLossThreads + threadIdx.x; p < npix; p += (int64_t)gridDim.x * kLossThreads) {
    const float wgt = lam_l1 + (mask ? lam_w * (float)mask[p] : 0.f);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float d = img[3 * p + c] - tgt[3 * p + c];
      acc = __builtin_fmaf(wgt, fabsf(d), acc);
      const float sg = d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f);
      dL[3 * p + c] = wgt * sg * inv_n;
    }
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float s = 0.f;
    for (int k = 0; k < kLossThreads / 64; ++k) s += red[k];
    partial[blockIdx.x] = s;
  }
}

// Sum of the block partials in binary64, in a fixed order: 256 strided partial sums, then a fixed
// butterfly within each wave and the four wave sums in order.
__global__ void __launch_bounds__(256) loss_final_kernel(const float* __restrict__ partial, int nb, float scale,
                                                         float* __restrict__ out) {
  __shared__ double wsum[4];
  double s = 0.0;
  for (int k = threadIdx.x; k < nb; k += 256) s += (double)partial[k];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *out = (float)((((wsum[0] + wsum[1]) + wsum[2]) + wsum[3]) * (double)scale);
}

size_t loss_scratch_bytes() { return kLossBlocks * sizeof(float); }

hipError_t launch_loss(const float* img, const float* target, const uint8_t* mask, int w, int h, float lam_l1,
                       float lam_w, void* scratch, float* loss_out, float* dL_dimg, hipStream_t stream) {
  const int64_t npix = (int64_t)w * h;
  float* partial = reinterpret_cast<float*>(scratch);
  const int nb = (int)std::min<int64_t>(kLossBlocks, (npix + kLossThreads - 1) / kLossThreads);
  hipLaunchKernelGGL(loss_kernel, dim3(nb), dim3(kLossThreads), 0, stream, img, target, mask, npix, lam_l1, lam_w,
                     dL_dimg, partial);
  hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(256), 0, stream, partial, nb, 1.f / (3.f * (float)npix), loss_out);
  return hipGetLastError();
}

}  // namespace ges
