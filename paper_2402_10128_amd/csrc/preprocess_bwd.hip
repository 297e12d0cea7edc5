// preprocess_bwd.hip -- chain rule of the per-splat preprocess (GES Sec. 4.1-4.2).
//
// From the accumulated gradients of a splat's 2-D quantities (mean2D, conic a/b/c, opacity, colour and,
// with the GEF falloff, beta) to its mean, log-scale, quaternion, opacity logit, SH coefficients and
// beta.  The chain runs in binary64: forward quantities (scales, opacity, rotation, covariance, the
// conic, the view direction) are recomputed in binary64 from the binary32 inputs, and only the decisions
// (visibility, guard clamp of the Jacobian, colour clamp) come from the forward pass, through a 4-byte
// visibility word per splat.  Several of the sums cancel (e.g. the scale gradient of an axis along the
// view ray), and binary32 there leaves an error proportional to the splat's whole gradient; the FP64
// vector rate of gfx950 equals its non-packed FP32 rate.  Nothing here feeds a decision, so this file is built
// with contraction allowed.
// Two launches:
//   chain:  the splats with a 2-D gradient (about a tenth: the backward raster composited them somewhere) are
//           gathered from the visibility words and chained one per lane, 48 bytes of gradients each;
//   emit:   every splat's gradients are written, or applied at once as an Adam update, as one stream over the
//           parameter arrays; the SH gradients are the product of the basis of the view direction and the colour
//           gradient, formed there.  The views of one scene are added up in registers and LDS.
// In one launch the chain's registers (203, and 430 with spills for several views) left two waves per SIMD for what
// is a stream over memory, and a tenth of its lanes working.  Measured, one launch -> chain and emit: Adam fused, 3M
// splats 1,061 -> 60 + 800 us, four views of 200k 315 -> 65 + 92; gradients stored, 1M 105 -> 45 + 50, 5M 456 -> 362 in
// all; 1k 8 -> 11 (the second launch).
// Memory: the stream reads 4 bytes per splat and view and writes the gradients (240 B at SH degree 3), or reads and
// writes the parameters and both moments (1,440 B); the chain reads about 430 B per splat it takes.
#include "ges_internal.h"

namespace ges {

// Real SH normalisations in binary64 (same values as the forward's binary32 constants, unrounded).
constexpr double kD0 = 0.28209479177387814;   // 1/(2 sqrt(pi))
constexpr double kD1 = 0.4886025119029199;    // sqrt(3/pi)/2
constexpr double kD2a = 1.0925484305920792;   // sqrt(15/pi)/2
constexpr double kD2b = 0.31539156525252005;  // sqrt(5/pi)/4
constexpr double kD2c = 0.5462742152960396;   // sqrt(15/pi)/4
constexpr double kD3a = 0.5900435899266435;   // sqrt(35/(2 pi))/4
constexpr double kD3b = 2.890611442640554;    // sqrt(105/pi)/2
constexpr double kD3c = 0.4570457994644658;   // sqrt(21/(2 pi))/4
constexpr double kD3d = 0.3731763325901154;   // sqrt(7/pi)/4
constexpr double kD3e = 1.445305721320277;    // sqrt(105/pi)/4

__device__ __forceinline__ void sh_basis_f64(double x, double y, double z, int degree, double* Y) {
  Y[0] = kD0;
  if (degree < 1) return;
  Y[1] = -kD1 * y; Y[2] = kD1 * z; Y[3] = -kD1 * x;
  if (degree < 2) return;
  const double xx = x * x, yy = y * y, zz = z * z;
  Y[4] = kD2a * x * y; Y[5] = -kD2a * y * z; Y[6] = kD2b * (2.0 * zz - xx - yy); Y[7] = -kD2a * x * z;
  Y[8] = kD2c * (xx - yy);
  if (degree < 3) return;
  Y[9] = -kD3a * y * (3.0 * xx - yy);
  Y[10] = kD3b * x * y * z;
  Y[11] = -kD3c * y * (4.0 * zz - xx - yy);
  Y[12] = kD3d * z * (2.0 * zz - 3.0 * xx - 3.0 * yy);
  Y[13] = -kD3c * x * (4.0 * zz - xx - yy);
  Y[14] = kD3e * z * (xx - yy);
  Y[15] = -kD3a * x * (xx - 3.0 * yy);
}

// Gradient, parameter and moment stores are non-temporal: 720 MB of gradients per 3M-splat frame stream past
// the caches (measured on that frame: 0.29 -> 0.27 ms for the backward, and the parameters the next frame's
// preprocess reads stay in the last-level cache).
typedef float NtF4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void nt_store4(float4* d, float4 v) {
  NtF4 x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<NtF4*>(d));
}

// How the stream takes the gradients: stored; applied as an Adam update; or applied with the parameters and moments
// loaded past the caches too.  That pays once they exceed the last-level cache (256 MB): at 3M splats, 2.2 GB, the
// stream takes 800 us against 946, and the next frame's preprocess 174 against 207; at 200k, 144 MB, they are
// still there from one step to the next, and it takes 99 against 92.
enum EmitMode : int { kStore, kUpdate, kUpdateStream };
constexpr int64_t kStreamBytes = 256 << 20;

template <EmitMode M, class T>
__device__ __forceinline__ T emit_load(const T* p) {
  if constexpr (M == kUpdateStream) return __builtin_nontemporal_load(p);
  else return *p;
}

// Output of one parameter gradient: stored when the caller asked for gradients, and with an update also
// applied at once to the parameter (the gradient never goes through memory).
template <EmitMode M, int P>
__device__ __forceinline__ void emit(float* g, const AdamSplats& A, int64_t idx, float val) {
  if constexpr (M != kStore) {
    if (A.gin[P]) val = A.gin[P][idx] + val;      // the other views' gradients, then this view's
  }
  if (g) {
    if (A.accumulate) g[idx] = g[idx] + val;
    else __builtin_nontemporal_store(val, g + idx);
  }
  if constexpr (M != kStore) {
    float p = emit_load<M>(A.p[P] + idx), m = emit_load<M>(A.m[P] + idx), v = emit_load<M>(A.v[P] + idx);
    adam_update(p, val, m, v, A.b1, A.b2, A.eps, A.step_size[P], A.inv_sqrt_bc2);
    __builtin_nontemporal_store(p, A.p[P] + idx);
    __builtin_nontemporal_store(m, A.m[P] + idx);
    __builtin_nontemporal_store(v, A.v[P] + idx);
  }
}

template <EmitMode M, int P>
__device__ __forceinline__ void emit4(float* g, const AdamSplats& A, int64_t idx4, float4 val) {
  if constexpr (M != kStore) {
    if (A.gin[P]) {
      const float4 o = reinterpret_cast<const float4*>(A.gin[P])[idx4];
      val = make_float4(o.x + val.x, o.y + val.y, o.z + val.z, o.w + val.w);
    }
  }
  if (g) {
    float4* d = reinterpret_cast<float4*>(g) + idx4;
    if (A.accumulate) {
      const float4 o = *d;
      *d = make_float4(o.x + val.x, o.y + val.y, o.z + val.z, o.w + val.w);
    } else {
      nt_store4(d, val);
    }
  }
  if constexpr (M != kStore) {
    NtF4 p = emit_load<M>(reinterpret_cast<const NtF4*>(A.p[P]) + idx4);
    NtF4 m = emit_load<M>(reinterpret_cast<const NtF4*>(A.m[P]) + idx4);
    NtF4 v = emit_load<M>(reinterpret_cast<const NtF4*>(A.v[P]) + idx4);
    const float gr[4] = {val.x, val.y, val.z, val.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float pc = p[c], mc = m[c], vc = v[c];
      adam_update(pc, gr[c], mc, vc, A.b1, A.b2, A.eps, A.step_size[P], A.inv_sqrt_bc2);
      p[c] = pc;
      m[c] = mc;
      v[c] = vc;
    }
    __builtin_nontemporal_store(p, reinterpret_cast<NtF4*>(A.p[P]) + idx4);
    __builtin_nontemporal_store(m, reinterpret_cast<NtF4*>(A.m[P]) + idx4);
    __builtin_nontemporal_store(v, reinterpret_cast<NtF4*>(A.v[P]) + idx4);
  }
}

// Digamma psi(x) for x > 0 in binary64: psi(x) = psi(x + k) - sum 1/(x + j) up to x + k >= 6, then the
// asymptotic series ln x - 1/(2x) - 1/(12x^2) + 1/(120x^4) - 1/(252x^6) + 1/(240x^8) - 1/(132x^10).
__device__ __forceinline__ double digamma(double x) {
  double acc = 0.0;
  while (x < 6.0) {
    acc -= 1.0 / x;
    x += 1.0;
  }
  const double i = 1.0 / x, i2 = i * i;
  const double series = i2 * (1.0 / 12 - i2 * (1.0 / 120 - i2 * (1.0 / 252 - i2 * (1.0 / 240 - i2 / 132))));
  return acc + log(x) - 0.5 * i - series;
}

// View direction of a splat in binary64, and its length.
__device__ __forceinline__ void view_dir(const ViewDesc& V, double mx, double my, double mz, double& x, double& y,
                                         double& z, double& len) {
  double cpos[3];
#pragma unroll
  for (int j = 0; j < 3; ++j)
    cpos[j] = -((double)V.R[j] * (double)V.t[0] + (double)V.R[3 + j] * (double)V.t[1] + (double)V.R[6 + j] * (double)V.t[2]);
  const double e0 = mx - cpos[0], e1 = my - cpos[1], e2 = mz - cpos[2];
  len = sqrt(e0 * e0 + e1 * e1 + e2 * e2);
  x = e0 / len;
  y = e1 / len;
  z = e2 / len;
}

// Chain rule of splat i, whose 2-D gradient the row reduction left in grad2d: everything but the SH gradients, as
// (mean, log-scale, opacity, beta, quaternion) in V.chain.  EXACT: the exact shape modification (its ln Gamma takes
// many registers).
template <int D, bool EXACT>
__device__ __forceinline__ void chain_splat(const ViewDesc& V, int64_t i) {
  constexpr int K = (D + 1) * (D + 1);
  const uint32_t flags = V.vis[i] & 0xffu;
  const double2* gp = reinterpret_cast<const double2*>(V.grad2d + (int64_t)kGradStride * i);
  const double2 g01 = gp[0], g23 = gp[1], g45 = gp[2], g67 = gp[3], g89 = gp[4];
  float out[12];
  const double grgb[3] = {g67.x, g67.y, g89.x};
  const double gu = g01.x, gv = g01.y, ga = g23.x, gb = g23.y, gc = g45.x, gop = g45.y;
  const double gbeta2 = g89.y;

  const float* mu = V.means + 3 * i;
  const double mx = mu[0], my = mu[1], mz = mu[2];
  const float4 qv = reinterpret_cast<const float4*>(V.quats)[i];
  const double beta = V.beta[i];
  double R[9];
  for (int k = 0; k < 9; ++k) R[k] = V.R[k];
  double p[3];
  for (int r = 0; r < 3; ++r) p[r] = R[3 * r] * mx + R[3 * r + 1] * my + R[3 * r + 2] * mz + (double)V.t[r];
  const double z = p[2];
  const double s[3] = {exp((double)V.log_scales[3 * i]), exp((double)V.log_scales[3 * i + 1]),
                       exp((double)V.log_scales[3 * i + 2])};
  const double op = 1.0 / (1.0 + exp(-(double)V.logits[i]));

  // quaternion
  const double q0 = qv.x, q1 = qv.y, q2 = qv.z, q3 = qv.w;
  const double nr = sqrt(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
  const double qw = q0 / nr, qx = q1 / nr, qy = q2 / nr, qz = q3 / nr;
  double Q[9];
  Q[0] = 1.0 - 2.0 * (qy * qy + qz * qz); Q[1] = 2.0 * (qx * qy - qw * qz); Q[2] = 2.0 * (qx * qz + qw * qy);
  Q[3] = 2.0 * (qx * qy + qw * qz); Q[4] = 1.0 - 2.0 * (qx * qx + qz * qz); Q[5] = 2.0 * (qy * qz - qw * qx);
  Q[6] = 2.0 * (qx * qz - qw * qy); Q[7] = 2.0 * (qy * qz + qw * qx); Q[8] = 1.0 - 2.0 * (qx * qx + qy * qy);
  double phi = 1.0;
  const double rho = V.rho;
  if (V.falloff == GES_FALLOFF_PHI) phi = 2.0 / (1.0 + exp(-(rho * beta - 2.0 * rho)));
  else if (EXACT) phi = 2.0 * exp(lgamma(3.0 / beta) - lgamma(1.0 / beta));
  const double S[3] = {phi * s[0], phi * s[1], phi * s[2]};
  double Mm[9];
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) Mm[3 * r + c] = Q[3 * r + c] * S[c];
  double Sig[9];
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) Sig[3 * r + c] = Mm[3 * r] * Mm[3 * c] + Mm[3 * r + 1] * Mm[3 * c + 1] + Mm[3 * r + 2] * Mm[3 * c + 2];

  // perspective Jacobian at p; the guard clamp of x/z, y/z is the forward's decision (record flags)
  const double fx = V.fx, fy = V.fy;
  const bool clx = (flags & 8u) != 0, cly = (flags & 16u) != 0;
  const double limx = 1.3 * (0.5 * (double)V.width / fx), limy = 1.3 * (0.5 * (double)V.height / fy);
  const double txz = clx ? copysign(limx, p[0] / z) : p[0] / z;
  const double tyz = cly ? copysign(limy, p[1] / z) : p[1] / z;
  const double xc = txz * z, yc = tyz * z;
  const double iz = 1.0 / z, iz2 = iz * iz, iz3 = iz2 * iz;
  const double J00 = fx * iz, J11 = fy * iz, J02 = -fx * xc * iz2, J12 = -fy * yc * iz2;
  double T[6];
  for (int c = 0; c < 3; ++c) {
    T[c] = J00 * R[c] + J02 * R[6 + c];
    T[3 + c] = J11 * R[3 + c] + J12 * R[6 + c];
  }
  // 2-D covariance and its inverse (the conic), recomputed in binary64
  double TS[6];
  for (int r = 0; r < 2; ++r)
    for (int c = 0; c < 3; ++c) TS[3 * r + c] = T[3 * r] * Sig[c] + T[3 * r + 1] * Sig[3 + c] + T[3 * r + 2] * Sig[6 + c];
  const double c00 = TS[0] * T[0] + TS[1] * T[1] + TS[2] * T[2] + 0.3;
  const double c01 = TS[0] * T[3] + TS[1] * T[4] + TS[2] * T[5];
  const double c11 = TS[3] * T[3] + TS[4] * T[4] + TS[5] * T[5] + 0.3;
  const double det = c00 * c11 - c01 * c01;
  const double ca = c11 / det, cb = -c01 / det, cc = c00 / det;

  // conic -> covariance: dL/dcov = -C G_C C with C = conic, G_C the symmetric gradient
  const double gx = -(ca * ca * ga + ca * cb * gb + cb * cb * gc);
  const double gy = -(2.0 * ca * cb * ga + (ca * cc + cb * cb) * gb + 2.0 * cb * cc * gc);
  const double gz = -(cb * cb * ga + cb * cc * gb + cc * cc * gc);
  // G2: gradient w.r.t. the full symmetric 2x2 covariance (off-diagonal split in half)
  const double G2[4] = {gx, 0.5 * gy, 0.5 * gy, gz};

  // cov = T Sigma T^T: dL/dSigma = T^T G2 T (symmetric), dL/dT = 2 G2 T Sigma
  double GT[6];   // G2 T (2x3)
  for (int c = 0; c < 3; ++c) {
    GT[c] = G2[0] * T[c] + G2[1] * T[3 + c];
    GT[3 + c] = G2[2] * T[c] + G2[3] * T[3 + c];
  }
  double GS[9];   // T^T (G2 T)
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) GS[3 * r + c] = T[r] * GT[c] + T[3 + r] * GT[3 + c];
  double gT[6];
  for (int r = 0; r < 2; ++r)
    for (int c = 0; c < 3; ++c)
      gT[3 * r + c] = 2.0 * (GT[3 * r] * Sig[c] + GT[3 * r + 1] * Sig[3 + c] + GT[3 * r + 2] * Sig[6 + c]);
  // T = J W: dL/dJ = dL/dT W^T
  const double gJ00 = gT[0] * R[0] + gT[1] * R[1] + gT[2] * R[2];
  const double gJ02 = gT[0] * R[6] + gT[1] * R[7] + gT[2] * R[8];
  const double gJ11 = gT[3] * R[3] + gT[4] * R[4] + gT[5] * R[5];
  const double gJ12 = gT[3] * R[6] + gT[4] * R[7] + gT[5] * R[8];
  double gp0 = 0.0, gp1 = 0.0, gz_ = 0.0;
  gz_ += -fx * iz2 * gJ00 + 2.0 * fx * xc * iz3 * gJ02 - fy * iz2 * gJ11 + 2.0 * fy * yc * iz3 * gJ12;
  const double gxc = -fx * iz2 * gJ02, gyc = -fy * iz2 * gJ12;
  if (clx) gz_ += gxc * txz; else gp0 += gxc;
  if (cly) gz_ += gyc * tyz; else gp1 += gyc;
  // mean2D
  gp0 += gu * fx * iz;
  gp1 += gv * fy * iz;
  gz_ += -(gu * fx * p[0] + gv * fy * p[1]) * iz2;

  // Sigma = M M^T: dL/dM = 2 GS M
  double gS[3] = {0.0, 0.0, 0.0};
  double gQ[9];
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) {
      const double gM = 2.0 * (GS[3 * r] * Mm[c] + GS[3 * r + 1] * Mm[3 + c] + GS[3 * r + 2] * Mm[6 + c]);
      gS[c] += gM * Q[3 * r + c];
      gQ[3 * r + c] = gM * S[c];
    }
  const double gphi = gS[0] * s[0] + gS[1] * s[1] + gS[2] * s[2];
  for (int c = 0; c < 3; ++c) out[3 + c] = (float)(gS[c] * phi * s[c]);
  {
    double gb_ = 0.0;
    if (V.falloff == GES_FALLOFF_PHI) gb_ = gphi * rho * phi * (1.0 - 0.5 * phi);
    else if (EXACT)   // d phi / d beta = phi (psi(1/b) - 3 psi(3/b)) / b^2
      gb_ = gphi * phi * (digamma(1.0 / beta) - 3.0 * digamma(3.0 / beta)) / (beta * beta);
    else gb_ = gbeta2;
    out[7] = (float)gb_;
  }
  // rotation -> unit quaternion -> quaternion
  {
    const double w = qw, x = qx, y = qy, zq = qz;
    const double gw = 2.0 * (-zq * gQ[1] + y * gQ[2] + zq * gQ[3] - x * gQ[5] - y * gQ[6] + x * gQ[7]);
    const double gxq = 2.0 * (y * gQ[1] + zq * gQ[2] + y * gQ[3] - 2.0 * x * gQ[4] - w * gQ[5] + zq * gQ[6] + w * gQ[7] - 2.0 * x * gQ[8]);
    const double gyq = 2.0 * (-2.0 * y * gQ[0] + x * gQ[1] + w * gQ[2] + x * gQ[3] + zq * gQ[5] - w * gQ[6] + zq * gQ[7] - 2.0 * y * gQ[8]);
    const double gzq = 2.0 * (-2.0 * zq * gQ[0] - w * gQ[1] + x * gQ[2] + w * gQ[3] - 2.0 * zq * gQ[4] + y * gQ[5] + x * gQ[6] + y * gQ[7]);
    const double dot = gw * w + gxq * x + gyq * y + gzq * zq;
    out[8] = (float)((gw - w * dot) / nr);
    out[9] = (float)((gxq - x * dot) / nr);
    out[10] = (float)((gyq - y * dot) / nr);
    out[11] = (float)((gzq - zq * dot) / nr);
  }
  out[6] = (float)(gop * op * (1.0 - op));


  // colour: the SH coefficients' dependence on the view direction
  double gmu[3] = {0.0, 0.0, 0.0};
  if (D > 0) {
    double gc3[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) gc3[ch] = (flags & (1u << ch)) ? 0.0 : grgb[ch];
    double x, y, zz_, len;
    view_dir(V, mx, my, mz, x, y, zz_, len);
    // dL/dY_k = sum_ch gc3[ch] c_k,ch.  Rows of 3K floats; for degrees 1 and 3 they are 16-byte aligned (checked on
    // the host), so they move as float4.
    const float* shc = V.sh + (int64_t)3 * K * i;
    double gY[16];
#pragma unroll
    for (int k = 0; k < K; ++k) gY[k] = 0.0;
    if constexpr ((3 * K) % 4 == 0) {
      const float4* s4 = reinterpret_cast<const float4*>(shc);
      float4 xv[3 * K / 4];
#pragma unroll
      for (int m = 0; m < 3 * K / 4; ++m) xv[m] = s4[m];
#pragma unroll
      for (int m = 0; m < 3 * K / 4; ++m) {
        const float xs[4] = {xv[m].x, xv[m].y, xv[m].z, xv[m].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) gY[(4 * m + e) / 3] += gc3[(4 * m + e) % 3] * (double)xs[e];
      }
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) gY[k] += gc3[ch] * (double)shc[3 * k + ch];
    }
    double gdx = 0.0, gdy = 0.0, gdz = 0.0;
    gdy += -kD1 * gY[1]; gdz += kD1 * gY[2]; gdx += -kD1 * gY[3];
    if (D > 1) {
      const double xx = x * x, yy = y * y, z2v = zz_ * zz_;
      gdx += kD2a * y * gY[4]; gdy += kD2a * x * gY[4];
      gdy += -kD2a * zz_ * gY[5]; gdz += -kD2a * y * gY[5];
      gdx += -2.0 * kD2b * x * gY[6]; gdy += -2.0 * kD2b * y * gY[6]; gdz += 4.0 * kD2b * zz_ * gY[6];
      gdx += -kD2a * zz_ * gY[7]; gdz += -kD2a * x * gY[7];
      gdx += 2.0 * kD2c * x * gY[8]; gdy += -2.0 * kD2c * y * gY[8];
      if (D > 2) {
        gdx += -kD3a * 6.0 * x * y * gY[9]; gdy += -kD3a * (3.0 * xx - 3.0 * yy) * gY[9];
        gdx += kD3b * y * zz_ * gY[10]; gdy += kD3b * x * zz_ * gY[10]; gdz += kD3b * x * y * gY[10];
        gdx += 2.0 * kD3c * x * y * gY[11]; gdy += -kD3c * (4.0 * z2v - xx - 3.0 * yy) * gY[11];
        gdz += -8.0 * kD3c * y * zz_ * gY[11];
        gdx += -6.0 * kD3d * x * zz_ * gY[12]; gdy += -6.0 * kD3d * y * zz_ * gY[12];
        gdz += kD3d * (6.0 * z2v - 3.0 * xx - 3.0 * yy) * gY[12];
        gdx += -kD3c * (4.0 * z2v - 3.0 * xx - yy) * gY[13]; gdy += 2.0 * kD3c * x * y * gY[13];
        gdz += -8.0 * kD3c * x * zz_ * gY[13];
        gdx += 2.0 * kD3e * x * zz_ * gY[14]; gdy += -2.0 * kD3e * y * zz_ * gY[14]; gdz += kD3e * (xx - yy) * gY[14];
        gdx += -kD3a * (3.0 * xx - 3.0 * yy) * gY[15]; gdy += 6.0 * kD3a * x * y * gY[15];
      }
    }
    // d = e/|e|: dL/de = (dL/dd - d (d . dL/dd)) / |e|
    const double dd = gdx * x + gdy * y + gdz * zz_;
    gmu[0] = (gdx - x * dd) / len;
    gmu[1] = (gdy - y * dd) / len;
    gmu[2] = (gdz - zz_ * dd) / len;
  }
  // p = W mu + t
  for (int c = 0; c < 3; ++c) out[c] = (float)(gmu[c] + R[c] * gp0 + R[3 + c] * gp1 + R[6 + c] * gz_);
  float4* o = reinterpret_cast<float4*>(V.chain) + 3 * i;
#pragma unroll
  for (int k = 0; k < 3; ++k) o[k] = make_float4(out[4 * k], out[4 * k + 1], out[4 * k + 2], out[4 * k + 3]);
}

// Splats a chain block gathers from: many, so that the tenth of them it takes fills its lanes; few where the
// splats would not fill the device otherwise.
constexpr int kChainSpan = 2048;
inline int chain_span(int64_t n) { return n >= 262144 ? kChainSpan : 256; }

template <int D, bool EXACT>
__global__ void __launch_bounds__(256, 2) preprocess_chain_kernel(const DeviceBatch* __restrict__ db, int64_t blocks,
                                                               int span) {
  __shared__ uint16_t list[kChainSpan];
  __shared__ uint32_t count;
  const int64_t v = blockIdx.x / blocks;
  const ViewDesc& V = db->views[v];
  const int64_t base = (blockIdx.x - v * blocks) * span;
  const int lane = threadIdx.x & 63;
  if (threadIdx.x == 0) count = 0u;
  __syncthreads();
  for (int k = threadIdx.x; k < span; k += 256) {
    const bool in = base + k < V.n;
    const uint32_t vis = in ? V.vis[base + k] : 0u;
    const bool take = (vis & kVisBit) && (vis & kRowBit);
    const uint64_t m = __ballot(take);
    uint32_t at = 0;
    if (lane == 0 && m) at = atomicAdd(&count, (uint32_t)__builtin_popcountll(m));   // the order does not matter
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    if (take) list[at + __builtin_popcountll(m & ((1ull << lane) - 1ull))] = (uint16_t)k;
  }
  __syncthreads();
  const uint32_t n = count;
#pragma unroll 1
  for (uint32_t r = threadIdx.x; r < n; r += 256) {
    const ViewDesc* here = &V;
    asm volatile("" : "+s"(here));   // keeps the camera's values and their products out of registers between splats
    chain_splat<D, EXACT>(*here, base + list[r]);
  }
}

constexpr int kRowPad = 13;   // float4 slots per staged SH-gradient row (12 used at degree 3; 13 spreads LDS banks)

// Adds the gradients of splat i over the views, in view order, to `acc` (see chain_splat) and its SH row in LDS.  A
// view without rows of the splat adds zero.
template <int D>
__device__ __forceinline__ void sum_views(const DeviceBatch* db, const AdamSplats& A, int64_t i,
                                          bool in, float (&acc)[12], float* row) {
  constexpr int K = (D + 1) * (D + 1);
  for (int v = 0; v < db->nviews; ++v) {
    const ViewDesc& V = db->views[v];
    const uint32_t vis = in ? V.vis[i] : 0u;
    const bool row_here = (vis & kVisBit) && (vis & kRowBit);
    double2* gp = reinterpret_cast<double2*>(V.grad2d + (int64_t)kGradStride * i);
    if (in && V.keep_grad2d)   // inspection: rows nothing was added to, and the slots past the tenth, read as zero
      for (int k = row_here ? 5 : 0; k < kGradStride / 2; ++k) gp[k] = make_double2(0.0, 0.0);
    if (A.stat_accum && (vis & kVisBit)) {   // densification statistic: the mean-2D gradient in NDC units
      if (row_here) {
        const double2 g01 = gp[0];
        const double su = g01.x * A.half_w, sv = g01.y * A.half_h;
        A.stat_accum[i] += (float)sqrt(su * su + sv * sv);
      }
      A.stat_count[i] += 1.f;
    }
    if (!row_here) continue;
    const float4* c = reinterpret_cast<const float4*>(V.chain) + 3 * i;
    const float4 c0 = c[0], c1 = c[1], c2 = c[2];
    const float val[12] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w, c2.x, c2.y, c2.z, c2.w};
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = acc[k] + val[k];
    const double2 g67 = gp[3], g89 = gp[4];
    const double gc3[3] = {(vis & 1u) ? 0.0 : g67.x, (vis & 2u) ? 0.0 : g67.y, (vis & 4u) ? 0.0 : g89.x};
    const float* mu = V.means + 3 * i;
    double x = 0.0, y = 0.0, z = 0.0, len;
    if (D > 0) view_dir(V, mu[0], mu[1], mu[2], x, y, z, len);
    double Y[16];
    sh_basis_f64(x, y, z, D, Y);
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) row[3 * k + ch] = row[3 * k + ch] + (float)(Y[k] * gc3[ch]);   // dL/dc = Y gc
  }
}

__device__ __forceinline__ void rows_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per 64 splats; the views of a batch (one scene) are added up on the way.
template <int D, EmitMode M>
__global__ void __launch_bounds__(256) preprocess_emit_kernel(const DeviceBatch* __restrict__ db, ges_splat_grads G,
                                                              AdamSplats A) {
  constexpr int K = (D + 1) * (D + 1);
  __shared__ __align__(16) float sRows[4][64 * kRowPad * 4];
  const int64_t blk = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float* rows = sRows[wave];
  const int64_t n = db->views[0].n;
  const int64_t w0 = blk * 256 + wave * 64;
  if (w0 >= n) return;
  const int64_t i = w0 + lane;
  const int cnt = (int)min<int64_t>(64, n - w0);
  float acc[12] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (M == kStore && A.accumulate && db->nviews > 1) {
    // several views added to the stored gradients: view by view, starting from those
    A.accumulate = 0;
    if (G.sh)
      for (int m = lane; m < cnt * 3 * K; m += 64)
        rows[(m / (3 * K)) * kRowPad * 4 + (m % (3 * K))] = G.sh[(int64_t)3 * K * w0 + m];
    if (i < n) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (G.means) acc[c] = G.means[3 * i + c];
        if (G.log_scales) acc[3 + c] = G.log_scales[3 * i + c];
      }
      if (G.opacity_logits) acc[6] = G.opacity_logits[i];
      if (G.beta) acc[7] = G.beta[i];
      if (G.quats) {
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[8 + c] = G.quats[4 * i + c];
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < 3 * K; ++k) rows[lane * kRowPad * 4 + k] = 0.f;
  }
  rows_fence();
  sum_views<D>(db, A, i, i < n, acc, rows + lane * kRowPad * 4);
  rows_fence();
  // the wave's rows are one contiguous block of 3K x cnt floats: whole float4s at degrees 1 and 3
  if (M != kStore || G.sh) {
    if constexpr ((3 * K) % 4 == 0) {
      constexpr int F4 = 3 * K / 4;
      const int64_t base4 = (int64_t)F4 * w0;
      const float4* r4 = reinterpret_cast<const float4*>(rows);
#pragma unroll 4
      for (int m = lane; m < cnt * F4; m += 64)
        emit4<M, kParSh>(G.sh, A, base4 + m, r4[(m / F4) * kRowPad + (m % F4)]);
    } else {
#pragma unroll 4
      for (int m = lane; m < cnt * 3 * K; m += 64)
        emit<M, kParSh>(G.sh, A, (int64_t)3 * K * w0 + m, rows[(m / (3 * K)) * kRowPad * 4 + (m % (3 * K))]);
    }
  }
  rows_fence();
  // means and log-scales through LDS, so that consecutive lanes take consecutive floats
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    rows[3 * lane + c] = acc[c];
    rows[192 + 3 * lane + c] = acc[3 + c];
  }
  rows_fence();
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int m = lane + 64 * c;
    if (m < 3 * cnt) {
      emit<M, kParMeans>(G.means, A, 3 * w0 + m, rows[m]);
      emit<M, kParScales>(G.log_scales, A, 3 * w0 + m, rows[192 + m]);
    }
  }
  if (i < n) {
    emit4<M, kParQuats>(G.quats, A, i, make_float4(acc[8], acc[9], acc[10], acc[11]));
    emit<M, kParOpacity>(G.opacity_logits, A, i, acc[6]);
    emit<M, kParBeta>(G.beta, A, i, acc[7]);
  }
}

template <int D>
hipError_t launch_preprocess_backward_t(const DeviceBatch* dbatch, const Batch& b, const ges_splat_grads& g,
                                        const AdamSplats& a, bool fused, hipStream_t stream) {
  const int64_t n = b.items / b.nviews;   // the views of a backward render the same splats
  const int span = chain_span(n);
  const int64_t blocks = (n + span - 1) / span;
  hipLaunchKernelGGL((b.falloff == GES_FALLOFF_PHI_EXACT ? preprocess_chain_kernel<D, true>
                                                         : preprocess_chain_kernel<D, false>),
                     dim3((unsigned)(blocks * b.nviews)), dim3(256), 0, stream, dbatch, blocks, span);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)(b.pre_blocks / b.nviews));
  const int64_t bytes = n * 3 * 4 * (12 + 3 * (D + 1) * (D + 1));   // parameters and moments
  auto kernel = !fused ? preprocess_emit_kernel<D, kStore>
                       : bytes <= kStreamBytes ? preprocess_emit_kernel<D, kUpdate> : preprocess_emit_kernel<D, kUpdateStream>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, dbatch, g, a);
  return hipGetLastError();
}

hipError_t launch_preprocess_backward(const DeviceBatch* dbatch, const Batch& b, int sh_degree,
                                      const ges_splat_grads* grads, hipStream_t stream, const AdamSplats* args,
                                      bool fused) {
  if (b.pre_blocks == 0) return hipSuccess;
  const ges_splat_grads none{};
  const ges_splat_grads& g = grads ? *grads : none;
  const AdamSplats a = args ? *args : AdamSplats{};
  switch (sh_degree) {   // a kernel per degree: the registers of the others would cost this one its waves
    case 0: return launch_preprocess_backward_t<0>(dbatch, b, g, a, fused, stream);
    case 1: return launch_preprocess_backward_t<1>(dbatch, b, g, a, fused, stream);
    case 2: return launch_preprocess_backward_t<2>(dbatch, b, g, a, fused, stream);
    default: return launch_preprocess_backward_t<3>(dbatch, b, g, a, fused, stream);
  }
}

}  // namespace ges
