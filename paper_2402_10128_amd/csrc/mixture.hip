// mixture.hip -- the paper's 1-D mixture simulation as one batched kernel (Sec. 3.2; App. A.3).
//
// Each problem fits a mixture of n components -- Gaussian (GMM), difference of Gaussians with variance
// ratio 4 (DoG), Laplacian of Gaussian (LoG) or generalized exponential (GEF, per-component beta) -- to a
// 1-D signal sampled on m points of a linspace, by Adam on the mean squared error, for a number of epochs.
// Component i has parameters (w_raw, mu, s, beta); w = w_raw, or softplus(w_raw) for positive weights.
//
// One workgroup of 256 threads runs one problem through all its epochs: the signal, the residuals, the
// parameters, their Adam moments and gradients stay in LDS.  Per epoch:
//   1. per component, its constants (MixComp);
//   2. residuals r_j = model(x_j) - y_j, threads over points, four points per thread for one read of a component;
//   3. gradients sum_j (2/m) r_j dc_i/dtheta(x_j): the four waves take components in turn, the 64 lanes split the
//      points.  A chunk of 1,024 points and residuals stays in registers for all of a wave's components, and a
//      component's constant factors multiply its sums, not their terms;
//   4. Adam on every parameter (the update shared with the splat optimiser).
// What bounds it is VALU issue: of the 6.9 M cycles of the paper's sweep (7,680 problems x 1,000 points, 20 epochs)
// a SIMD issues VALU instructions in 6.8 M.  The sweep took 13.1 ms when each term carried its factors, the
// exponentials and powers were the library's, a reduction was 24 shuffles and the arrays for the largest m left room for
// 3 blocks per CU; it takes 2.92 ms.  The exponentials and logarithms are the hardware's base-2 ones on constants that
// are rounded once from binary64; gradients and losses are as close to binary64 as before (7e-8 to 1e-6 in the 2-norm,
// by model and parameter).  An exponential below 2^-126 is 0.
// A component that would read past the LDS arrays (n outside 1..128), an unknown model or target row, or
// m outside 1..4096 is not run: its loss is set to NaN.
#include <cmath>

#include "ges_internal.h"

namespace ges {

constexpr int kMixThreads = 256;
constexpr int kMixMaxN = GES_MIX_MAX_COMPONENTS;
constexpr int kMixMaxM = GES_MIX_MAX_POINTS;
constexpr float kMixEps = 1e-8f;
constexpr float kMixNu = 4.f;

struct MixArgs {
  const ges_mix_problem* problems;
  const float* targets;
  int32_t ntargets, m;
  float x0, dx;
  float* params;          // [P][kMixMaxN][4]
  float* grad_out;        // [P][kMixMaxN][4] gradient at the initial parameters, or NULL
  float* final_loss;      // [P]
  const int32_t* order;   // [P] problem index per block (a permutation), or NULL for the identity
  int32_t nproblems;
  int32_t epochs;
  float lr, b1, b2, eps;
};

// Per-component constants of one epoch, computed in binary64 and rounded once.  With inv = 1/(2 s^2 + eps) the component
// is w E, E = exp2(k q): q = d^2 = (x - mu)^2, or |d|^beta for GEF.  Step 3 sums, over the factors f:
//   GMM  r E,             r E d,                    r E d^2
//   DoG  r (E - E2),      r (E - k_mu E2) d,        r (E - k_s E2) d^2     E2 = exp2(k2 q), the subtracted Gaussian
//   LoG  r P E,           r (P + k_mu) E d,         r (P + k_s) E d^2      P = 1 - q/s^2
//   GEF  r E,             r E q / d,                r E q,                 r E q log2|d|
struct __attribute__((aligned(16))) MixComp {
  float w, mu, k;
  float beta_k2_is2;      // GEF, DoG, LoG
  float at0;              // GEF: q at d = 0
  float k_mu, k_s;
  float f[4];             // of w_raw, mu, s, beta; 2/m included
};

__device__ __forceinline__ MixComp mix_prepare(const float* th, int model, int positive, double scale) {
  MixComp c{};
  const float w_raw = th[0], beta = th[3];
  const double s = (double)th[2], eps = (double)kMixEps, nu = (double)kMixNu;
  const double log2e = 1.44269504088896340736, ln2 = 0.693147180559945309417;
  float dw = 1.f;
  c.mu = th[1];
  c.w = w_raw;
  if (positive) {
    c.w = w_raw > 30.f ? w_raw : log1pf(expf(fminf(w_raw, 30.f)));
    dw = 1.f / (1.f + expf(-w_raw));
  }
  const double inv = 1.0 / (2.0 * s * s + eps), w = (double)c.w * scale * inv;
  c.k = (float)(-inv * log2e);
  c.f[0] = (float)(dw * scale);
  c.f[1] = (float)(2.0 * w);
  c.f[2] = (float)(4.0 * w * s * inv);
  if (model == GES_MIX_GEF) {
    c.beta_k2_is2 = beta;
    c.at0 = powf(0.f, beta);
    c.f[1] = (float)(w * beta);
    c.f[3] = (float)(-w * ln2);
  } else if (model == GES_MIX_DOG) {
    const double inv2 = 1.0 / (2.0 * s * s / nu + eps), ratio = inv2 / inv;
    c.beta_k2_is2 = (float)(-inv2 * log2e);
    c.k_mu = (float)ratio;
    c.k_s = (float)(ratio * ratio / nu);
  } else if (model == GES_MIX_LOG) {
    const double is2 = 1.0 / (s * s), ratio = is2 / inv;
    c.beta_k2_is2 = (float)is2;
    c.k_mu = (float)ratio;
    c.k_s = (float)(0.5 * ratio * ratio);
  }
  return c;
}

// |d|^beta for a normal |d|, by the hardware's base-2 logarithm and exponential; beta log2|d| is carried in two parts.
__device__ __forceinline__ float mix_pow(float l, float beta) {
  const float h = beta * l;
  const float e = fminf(__builtin_amdgcn_exp2f(h), 3.402823466e38f);   // finite: the second part may be negative
  return __builtin_fmaf(e, __builtin_fmaf(beta, l, -h) * 0.693147180559945309417f, e);
}

// Component c at x, over w.
template <int MODEL>
__device__ __forceinline__ float mix_value(const MixComp& c, float x) {
  const float d = x - c.mu;
  if (MODEL == GES_MIX_GEF) {
    const float ad = fabsf(d);
    const float a = ad < 1.17549435e-38f ? c.at0 : mix_pow(__builtin_amdgcn_logf(ad), c.beta_k2_is2);
    return __builtin_amdgcn_exp2f(a * c.k);
  }
  const float q = d * d, E = __builtin_amdgcn_exp2f(q * c.k);
  if (MODEL == GES_MIX_DOG) return E - __builtin_amdgcn_exp2f(q * c.beta_k2_is2);
  if (MODEL == GES_MIX_LOG) return __builtin_fmaf(-q, c.beta_k2_is2, 1.f) * E;
  return E;
}

// Adds the terms of one point with residual r (table above MixComp).
template <int MODEL>
__device__ __forceinline__ void mix_grad(const MixComp& c, float x, float r, float (&acc)[4]) {
  const float d = x - c.mu;
  if (MODEL == GES_MIX_GEF) {
    const float ad = fabsf(d);
    const bool at = ad < 1.17549435e-38f;   // at the centre (or a denormal off it) the derivatives but w's are 0
    const float l = __builtin_amdgcn_logf(ad);
    const float a = at ? c.at0 : mix_pow(l, c.beta_k2_is2);
    const float rE = r * __builtin_amdgcn_exp2f(a * c.k), ra = rE * a;
    acc[0] += rE;
    acc[1] = __builtin_fmaf(ra, at ? 0.f : __builtin_amdgcn_rcpf(d), acc[1]);
    acc[2] += ra;
    acc[3] = __builtin_fmaf(ra, at ? 0.f : l, acc[3]);
    return;
  }
  const float q = d * d, rE = r * __builtin_amdgcn_exp2f(q * c.k);
  if (MODEL == GES_MIX_GMM) {
    acc[0] += rE;
    acc[1] = __builtin_fmaf(rE, d, acc[1]);
    acc[2] = __builtin_fmaf(rE, q, acc[2]);
  } else if (MODEL == GES_MIX_DOG) {
    const float rE2 = r * __builtin_amdgcn_exp2f(q * c.beta_k2_is2);
    acc[0] += rE - rE2;
    acc[1] = __builtin_fmaf(__builtin_fmaf(-c.k_mu, rE2, rE), d, acc[1]);
    acc[2] = __builtin_fmaf(__builtin_fmaf(-c.k_s, rE2, rE), q, acc[2]);
  } else {
    const float P = __builtin_fmaf(-q, c.beta_k2_is2, 1.f);
    acc[0] = __builtin_fmaf(rE, P, acc[0]);
    acc[1] = __builtin_fmaf(rE * d, P + c.k_mu, acc[1]);
    acc[2] = __builtin_fmaf(rE * q, P + c.k_s, acc[2]);
  }
}

// The wave's sums of four values: row k of 16 lanes returns that of v[k], in each of its lanes.  The two swaps halve the
// values and the lanes that hold them at once, so 3 swaps and 7 adds do what 24 shuffles would.
__device__ __forceinline__ float mix_sum_rows(const float (&v)[4]) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[2]), false, false);
  u2 q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[1]), __float_as_uint(v[3]), false, false);
  const float even = __uint_as_float(p.x) + __uint_as_float(p.y);   // lanes 0-31: value 0, 32-63: value 2
  const float odd = __uint_as_float(q.x) + __uint_as_float(q.y);
  p = __builtin_amdgcn_permlane16_swap(__float_as_uint(even), __float_as_uint(odd), false, false);
  float s = __uint_as_float(p.x) + __uint_as_float(p.y);
#define GES_ROW_ROR(n) s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x120 + (n), 0xf, 0xf, true))
  GES_ROW_ROR(8);
  GES_ROW_ROR(4);
  GES_ROW_ROR(2);
  GES_ROW_ROR(1);
#undef GES_ROW_ROR
  return s;
}

constexpr int kMixAhead = 4;    // points per thread that share a component's constants in step 2 ...
constexpr int kMixChunk = 16;   // ... and in step 3, where they stay in registers for all of a wave's components

// Residuals of NE points j0, j0 + kMixThreads, ... of a thread; l2 += their squares.
template <int MODEL, int NE>
__device__ __forceinline__ void mix_residuals(const MixArgs& a, int n, int j0, const MixComp* comp, const float* sy,
                                              float* sr, float& l2) {
  float v[NE], x[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    v[e] = 0.f;
    x[e] = a.x0 + (float)(j0 + e * kMixThreads) * a.dx;
  }
#pragma unroll 2
  for (int i = 0; i < n; ++i) {
    const MixComp c = comp[i];
#pragma unroll
    for (int e = 0; e < NE; ++e) v[e] = __builtin_fmaf(c.w, mix_value<MODEL>(c, x[e]), v[e]);
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int j = j0 + e * kMixThreads;
    if (j < a.m) {
      const float r = v[e] - sy[j];
      sr[j] = r;
      l2 = __builtin_fmaf(r, r, l2);
    }
  }
}

struct MixLds {
  float th[kMixMaxN][4], mo[kMixMaxN][4], ve[kMixMaxN][4], gr[kMixMaxN][4];
  MixComp comp[kMixMaxN];
  float lsum[kMixThreads / 64];
};

// All epochs of one problem.  sy, sr: [m] signal and residuals.
template <int MODEL>
__device__ __forceinline__ void mix_fit(const MixArgs& a, int p, int n, int positive, MixLds& L, const float* sy,
                                        float* sr) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int M = a.m;
  double pow1 = 1.0, pow2 = 1.0;   // b1^step, b2^step
  for (int ep = 0; ep <= a.epochs; ++ep) {
    // 1. per-component constants
    for (int i = t; i < n; i += kMixThreads) L.comp[i] = mix_prepare(L.th[i], MODEL, positive, 2.0 / (double)M);
    __syncthreads();
    // 2. residuals (and, after the last update, the loss)
    float l2 = 0.f;
    for (int c0 = 0; c0 < M; c0 += kMixThreads * kMixAhead) {
      static_assert(kMixAhead == 4, "one case each");
      switch (min((M - c0 + kMixThreads - 1) / kMixThreads, kMixAhead)) {   // uniform
        case 1: mix_residuals<MODEL, 1>(a, n, c0 + t, L.comp, sy, sr, l2); break;
        case 2: mix_residuals<MODEL, 2>(a, n, c0 + t, L.comp, sy, sr, l2); break;
        case 3: mix_residuals<MODEL, 3>(a, n, c0 + t, L.comp, sy, sr, l2); break;
        default: mix_residuals<MODEL, 4>(a, n, c0 + t, L.comp, sy, sr, l2); break;
      }
    }
    if (ep == a.epochs) {   // final loss: mean r^2 over the points, lanes then waves in a fixed order
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) l2 += __shfl_xor(l2, off, 64);
      if (lane == 0) L.lsum[wave] = l2;
      __syncthreads();
      if (t == 0) a.final_loss[p] = (((L.lsum[0] + L.lsum[1]) + L.lsum[2]) + L.lsum[3]) / (float)M;
      break;
    }
    __syncthreads();
    // 3. gradients: a chunk of points in registers, the wave's components over it
    for (int c0 = 0; c0 < M; c0 += 64 * kMixChunk) {
      float r[kMixChunk], x[kMixChunk];
#pragma unroll
      for (int e = 0; e < kMixChunk; ++e) {
        const int j = c0 + e * 64 + lane, jc = min(j, M - 1);   // lanes past the end: the last point, with no weight
        r[e] = j < M ? sr[jc] : 0.f;
        x[e] = a.x0 + (float)jc * a.dx;
      }
      for (int i = wave; i < n; i += kMixThreads / 64) {
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        const MixComp c = L.comp[i];
#pragma unroll
        for (int e = 0; e < kMixChunk; ++e) {
          if (e % 4 == 0 && c0 + e * 64 >= M) break;   // uniform
          mix_grad<MODEL>(c, x[e], r[e], acc);
        }
        const float sum = mix_sum_rows(acc);
        const int k = lane >> 4;
        if ((lane & 15) == 0) L.gr[i][k] = (c0 ? L.gr[i][k] : 0.f) + sum * L.comp[i].f[k];
      }
    }
    __syncthreads();
    if (ep == 0 && a.grad_out) {
      float* G = a.grad_out + (size_t)p * kMixMaxN * 4;
      for (int q = t; q < n * 4; q += kMixThreads) G[q] = L.gr[q >> 2][q & 3];
    }
    // 4. Adam (bias corrections of step ep + 1)
    if (t < n * 4) {
      pow1 *= (double)a.b1;
      pow2 *= (double)a.b2;
      const float step_size = (float)((double)a.lr / (1.0 - pow1)), inv_sqrt_bc2 = (float)(1.0 / sqrt(1.0 - pow2));
      for (int q = t; q < n * 4; q += kMixThreads)
        adam_update(L.th[q >> 2][q & 3], L.gr[q >> 2][q & 3], L.mo[q >> 2][q & 3], L.ve[q >> 2][q & 3], a.b1, a.b2,
                    a.eps, step_size, inv_sqrt_bc2);
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kMixThreads) mix_fit_kernel(const MixArgs a) {
  __shared__ MixLds L;
  extern __shared__ float points[];   // [2][m]
  // blocks take problems from the largest n down (a problem's time grows with n), so the longest ones do
  // not start last; results go to the problem's own rows
  const int p = a.order ? a.order[blockIdx.x] : (int)blockIdx.x;
  if (p < 0 || p >= a.nproblems) return;   // not a problem of this batch: nothing to do
  const int t = threadIdx.x;
  const ges_mix_problem pr = a.problems[p];
  const int n = pr.n, M = a.m;
  if (n < 1 || n > kMixMaxN || pr.model < 0 || pr.model > GES_MIX_GEF || pr.target < 0 || pr.target >= a.ntargets ||
      M < 1 || M > kMixMaxM) {
    if (t == 0) a.final_loss[p] = __int_as_float(0x7fc00000);
    return;
  }
  float* P = a.params + (size_t)p * kMixMaxN * 4;
  const float* y = a.targets + (size_t)pr.target * M;
  float* sy = points;
  float* sr = points + M;
  for (int j = t; j < M; j += kMixThreads) sy[j] = y[j];
  for (int q = t; q < n * 4; q += kMixThreads) {
    L.th[q >> 2][q & 3] = P[q];
    L.mo[q >> 2][q & 3] = 0.f;
    L.ve[q >> 2][q & 3] = 0.f;
  }
  __syncthreads();
  switch (pr.model) {   // uniform per block
    case GES_MIX_GMM: mix_fit<GES_MIX_GMM>(a, p, n, pr.positive, L, sy, sr); break;
    case GES_MIX_DOG: mix_fit<GES_MIX_DOG>(a, p, n, pr.positive, L, sy, sr); break;
    case GES_MIX_LOG: mix_fit<GES_MIX_LOG>(a, p, n, pr.positive, L, sy, sr); break;
    default: mix_fit<GES_MIX_GEF>(a, p, n, pr.positive, L, sy, sr); break;
  }
  for (int q = t; q < n * 4; q += kMixThreads) P[q] = L.th[q >> 2][q & 3];
}

hipError_t launch_mix_fit(const ges_mix_problem* problems, int nproblems, const float* targets, int ntargets, int m,
                          float x0, float dx, float* params, float* grad_out, float* final_loss, const int32_t* order,
                          int epochs, float lr, float b1, float b2, float eps, hipStream_t stream) {
  if (nproblems == 0) return hipSuccess;
  MixArgs a{problems, targets, ntargets, m, x0, dx, params, grad_out, final_loss, order, nproblems, epochs, lr, b1,
            b2, eps};
  hipLaunchKernelGGL(mix_fit_kernel, dim3((unsigned)nproblems), dim3(kMixThreads),
                     m >= 1 && m <= kMixMaxM ? 2 * (size_t)m * sizeof(float) : 0, stream, a);
  return hipGetLastError();
}

}  // namespace ges
