// mixture.hip -- the paper's 1-D mixture simulation as one batched kernel (Sec. 3.2; App. A.3).
//
// Each problem fits a mixture of n components -- Gaussian (GMM), difference of Gaussians with variance
// ratio 4 (DoG), Laplacian of Gaussian (LoG) or generalized exponential (GEF, per-component beta) -- to a
// 1-D signal sampled on m points of a linspace, by Adam on the mean squared error, for a number of epochs.
// Component i has parameters (w_raw, mu, s, beta); w = w_raw, or softplus(w_raw) for positive weights.
//
// One workgroup of 256 threads runs one problem through all its epochs: the signal, the residuals, the
// parameters, their Adam moments and gradients stay in LDS.  Per epoch:
//   1. per component, the quantities every point needs (MixComp);
//   2. residuals r_j = model(x_j) - y_j, threads over points, four points per thread for one read of a component;
//   3. gradients sum_j (2/m) r_j dc_i/dtheta(x_j): the four waves take components in turn, the 64 lanes split the
//      points and a butterfly adds the lanes.  A chunk of 1,024 points and residuals stays in registers for all of a
//      wave's components;
//   4. Adam on every parameter (the update shared with the splat optimiser), the bias corrections of 256 steps at a time
//      from a table.
// What bounds it is VALU issue: an exponential is 14 instructions, a component's term of the residual 21 and of the
// gradients 31 to 75.  The paper's sweep (7,680 problems x 1,000 points, 20 epochs) took 13.1 ms with the model looked up per
// term, its arrays sized for the largest m (3 blocks per CU), 24 shuffles per reduction and two binary64 powers per
// thread and epoch; it takes 7.0, of which 1.2 are four waves per SIMD (128 registers) instead of three.
// Taking the constant factors out of the sums and the exponentials from the hardware's base-2 one takes 2.9 ms, no further
// from binary64 -- but Adam's first steps are the sign of a gradient over its size, and where that is near zero other
// roundings move a parameter by up to 6e-3 of its scale; so every term keeps its roundings, and only factors that
// are powers of two are moved, to where they cost no bit of a subnormal result either.
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

// Per-component constants of one epoch.
struct __attribute__((aligned(16))) MixComp {
  float w, mu, inv1;     // inv1 = 1/(2 s^2 + eps)
  float beta_inv2_is2;   // GEF: beta; DoG: inv2 = 1/(2 s^2/nu + eps); LoG: is2 = 1/s^2
  float at0;             // GEF: |x - mu|^beta at x = mu
  float dw, s, rs;       // dw/dw_raw; LoG: 1/s
};

__device__ __forceinline__ MixComp mix_prepare(const float* th, int model, int positive) {
  MixComp c{};
  const float w_raw = th[0];
  c.mu = th[1];
  c.s = th[2];
  if (positive) {
    c.w = w_raw > 30.f ? w_raw : log1pf(expf(fminf(w_raw, 30.f)));
    c.dw = 1.f / (1.f + expf(-w_raw));
  } else {
    c.w = w_raw;
    c.dw = 1.f;
  }
  c.inv1 = 1.f / (2.f * c.s * c.s + kMixEps);
  if (model == GES_MIX_GEF) {
    c.beta_inv2_is2 = th[3];
    c.at0 = powf(0.f, th[3]);
  } else if (model == GES_MIX_DOG) {
    c.beta_inv2_is2 = 1.f / (2.f * c.s * c.s / kMixNu + kMixEps);
  } else if (model == GES_MIX_LOG) {
    c.beta_inv2_is2 = 1.f / (c.s * c.s);
    c.rs = 1.f / c.s;
  }
  return c;
}

// Component c at x, over w.
template <int MODEL>
__device__ __forceinline__ float mix_value(const MixComp& c, float x) {
  const float d = x - c.mu, d2 = d * d;
  if (MODEL == GES_MIX_GEF) {
    const float ad = fabsf(d);
    const float a = ad == 0.f ? c.at0 : expf(c.beta_inv2_is2 * logf(ad));
    return expf(-a * c.inv1);
  }
  const float E1 = expf(-d2 * c.inv1);
  if (MODEL == GES_MIX_DOG) return E1 - expf(-d2 * c.beta_inv2_is2);
  if (MODEL == GES_MIX_LOG) return (1.f - d2 * c.beta_inv2_is2) * E1;
  return E1;
}

// Adds r times the derivatives of a component by (w_raw, mu, s, beta) at x; but for GEF, x2 = 2 x.
template <int MODEL>
__device__ __forceinline__ void mix_grad(const MixComp& c, float x2, float r, float (&acc)[4]) {
  float base, db_mu, db_s;
  if (MODEL == GES_MIX_GEF) {
    const float d = x2 - c.mu, s4 = 4.f * c.s;
    const float beta = c.beta_inv2_is2, ad = fabsf(d);
    const bool off = ad != 0.f;
    const float l = logf(ad);
    const float a = off ? expf(beta * l) : c.at0;
    base = expf(-a * c.inv1);
    const float da_mu = off ? -beta * expf((beta - 1.f) * l) * (d > 0.f ? 1.f : -1.f) : 0.f;
    const float da_b = off ? a * l : 0.f;
    db_mu = -base * da_mu * c.inv1;
    db_s = base * a * s4 * c.inv1 * c.inv1;
    acc[3] = __builtin_fmaf(r, c.w * (-base * da_b * c.inv1), acc[3]);
  } else {
    // twice the distance, dd, and four times its square: the factors of two and four that the derivatives have come with
    // them.  Powers of two change no rounding but below the normal numbers, where taking them here keeps a bit that a
    // factor left for the sum would lose (d4 overflows from a distance of 9e18 on)
    const float dd = x2 - 2.f * c.mu, d4 = dd * dd;
    const float E1 = expf(-d4 * (0.25f * c.inv1));
    if (MODEL == GES_MIX_GMM) {
      base = E1;
      db_mu = E1 * dd * c.inv1;
      db_s = E1 * d4 * c.s * c.inv1 * c.inv1;
    } else if (MODEL == GES_MIX_DOG) {
      const float inv2 = c.beta_inv2_is2, E2 = expf(-d4 * (0.25f * inv2));
      base = E1 - E2;
      db_mu = E1 * dd * c.inv1 - E2 * dd * inv2;
      static_assert(kMixNu == 4.f, "the variance ratio is the factor of d4");
      db_s = E1 * d4 * c.s * c.inv1 * c.inv1 - E2 * d4 * (c.s / kMixNu) * inv2 * inv2;
    } else {
      const float is2 = c.beta_inv2_is2, P = 1.f - d4 * (0.25f * is2);
      base = P * E1;
      db_mu = dd * is2 * E1 + base * dd * c.inv1;
      // 2 d2 is2 / s by the reciprocal rounded to nearest: the remainder step rounds it as the division would (Markstein,
      // 1990), the last instruction of a division sees to zeros, infinities and NaN.  No scaling: where s is so large or
      // small that it would matter, is2 is 0 or infinite
      const float n = d4 * (0.5f * is2), q = n * c.rs;
      const float over_s = __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-q, c.s, n), c.rs, q), c.s, n);
      db_s = over_s * E1 + base * d4 * c.s * c.inv1 * c.inv1;
    }
  }
  acc[0] = __builtin_fmaf(r, c.dw * base, acc[0]);
  acc[1] = __builtin_fmaf(r, c.w * db_mu, acc[1]);
  acc[2] = __builtin_fmaf(r, c.w * db_s, acc[2]);
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
    for (int e = 0; e < NE; ++e) v[e] += c.w * mix_value<MODEL>(c, x[e]);
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
  float2 bias[kMixThreads];   // (step size, 1/sqrt(bias correction 2)) of the next steps
};

// All epochs of one problem.  sy, sr: [m] signal and residuals.
template <int MODEL>
__device__ __forceinline__ void mix_fit(const MixArgs& a, int p, int n, int positive, MixLds& L, const float* sy,
                                        float* sr) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int M = a.m;
  const float scale = 2.f / (float)M;
  for (int ep = 0; ep <= a.epochs; ++ep) {
    // 1. per-component constants
    for (int i = t; i < n; i += kMixThreads) L.comp[i] = mix_prepare(L.th[i], MODEL, positive);
    if (ep % kMixThreads == 0 && ep + t < a.epochs) {
      const int step = ep + t + 1;
      const double bc1 = 1.0 - pow((double)a.b1, (double)step), bc2 = 1.0 - pow((double)a.b2, (double)step);
      L.bias[t] = make_float2((float)((double)a.lr / bc1), (float)(1.0 / sqrt(bc2)));
    }
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
    // 3. gradients: up to 1,024 points in registers, the wave's components over them
    float r[kMixChunk], x[kMixChunk];
    auto load = [&](int c0) {
#pragma unroll
      for (int e = 0; e < kMixChunk; ++e) {
        const int j = c0 + e * 64 + lane, jc = min(j, M - 1);   // lanes past the end: the last point, with no weight
        r[e] = j < M ? sr[jc] : 0.f;
        x[e] = (MODEL == GES_MIX_GEF ? 1.f : 2.f) * (a.x0 + (float)jc * a.dx);
      }
    };
    const bool one = M <= 64 * kMixChunk;
    if (one) load(0);
    for (int i = wave; i < n; i += kMixThreads / 64) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      const MixComp c = L.comp[i];
      for (int c0 = 0; c0 < M; c0 += 64 * kMixChunk) {
        if (!one) load(c0);
#pragma unroll
        for (int e = 0; e < kMixChunk; ++e) {
          if (e % 4 == 0 && c0 + e * 64 >= M) break;   // uniform
          mix_grad<MODEL>(c, x[e], r[e], acc);
        }
      }
      const float sum = mix_sum_rows(acc);
      if ((lane & 15) == 0) L.gr[i][lane >> 4] = sum * scale;
    }
    __syncthreads();
    if (ep == 0 && a.grad_out) {
      float* G = a.grad_out + (size_t)p * kMixMaxN * 4;
      for (int q = t; q < n * 4; q += kMixThreads) G[q] = L.gr[q >> 2][q & 3];
    }
    // 4. Adam (bias corrections of step ep + 1)
    const float2 bias = L.bias[ep % kMixThreads];
    for (int q = t; q < n * 4; q += kMixThreads)
      adam_update(L.th[q >> 2][q & 3], L.gr[q >> 2][q & 3], L.mo[q >> 2][q & 3], L.ve[q >> 2][q & 3], a.b1, a.b2, a.eps,
                  bias.x, bias.y);
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kMixThreads, 4) mix_fit_kernel(const MixArgs a) {
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
