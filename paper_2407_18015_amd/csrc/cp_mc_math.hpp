// cp_mc_math.hpp -- per-sample math of the Gaussian Monte Carlo estimators
// (normal deviates from uniforms, the normal CDF and density), on the
// hardware transcendental instructions of gfx950; upper_tail also serves the
// FP32 independent-Gaussian quadrature.
//
// Measured against FP64 on the generator's uniforms: v_sin_f32 / v_cos_f32
// (argument in revolutions) 1.3e-7 absolute, v_sqrt_f32 9e-8, v_exp_f32
// 8e-8 and v_rcp_f32 9e-8 relative; v_log_f32 within one ulp of log2.
// The Monte Carlo normal CDF uses the complementary error function of Numerical Recipes
// (Press et al., 2nd ed., Sec. 6.2, routine erfcc: a Chebyshev fit of
// log(erfc) with fractional error below 1.2e-7 everywhere), so one CDF costs
// a reciprocal, nine fused multiply-adds and one exponential.
//
// The quadrature's tail is exp(-z^2/2) times a polynomial: erfcx(x)/2 =
// t p8(t), t = 1 / (1 + 0.37 x), x = |z| / sqrt 2, p8 of degree 8 fitted here
// to the smallest largest relative error on x <= 9 (1.3e-8; a linear program
// over 2000 Chebyshev points in t).  Working on zs = z sqrt(log2(e) / 2)
// makes the exponential one multiply and one v_exp_f32, which the density
// shares.  In FP32 the tail is within 4.7e-7 (rms 1.2e-7) of the exact one
// for |z| < 2 and within 1.0e-6 (3.0e-7) for |z| < 4, unbiased.  erfcc has
// 6.5e-7 (1.4e-7) and 2.0e-6 (4.8e-7, of which 2.8e-7 of one sign), and takes
// four more instructions and a second exponential where the density is needed
// as well.
#pragma once

#include <hip/hip_runtime.h>

namespace cp {

// Box-Muller: (u0, u1) in (0, 1] -> two independent N(0, 1) deviates
__device__ __forceinline__ void box_muller(float u0, float u1, float& z0, float& z1) {
  constexpr float kMinus2Ln2 = -1.3862943611198906f;  // -2 ln 2 (log2 -> ln)
  const float rad = __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(u0));
  z0 = rad * __builtin_amdgcn_cosf(u1);  // cos(2 pi u1)
  z1 = rad * __builtin_amdgcn_sinf(u1);  // sin(2 pi u1)
}

// 2^y and e^y for y <= 0 (the arguments here)
__host__ __device__ __forceinline__ float exp2_neg(float y) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_exp2f(y);
#else
  return exp2f(y);
#endif
}
__device__ __forceinline__ float exp_neg(float y) { return __builtin_amdgcn_exp2f(y * 1.4426950408889634f); }

constexpr float kTailScale = 0.84932180028801904f;  // sqrt(log2(e) / 2)

// From zs = kTailScale z: e = exp(-z^2 / 2), q = Pr(N(0, 1) > |z|) = t p8(t) e
__host__ __device__ __forceinline__ void upper_tail(float zs, float& q, float& e) {
  const float u = __builtin_fmaf(0.30804520612834824f, __builtin_fabsf(zs), 1.0f);
#if defined(__HIP_DEVICE_COMPILE__)
  const float t = __builtin_amdgcn_rcpf(u);
#else
  const float t = 1.0f / u;
#endif
  e = exp2_neg(-zs * zs);
  float p = 0.03130626671814147f;
  p = __builtin_fmaf(p, t, -0.1533205317712483f);
  p = __builtin_fmaf(p, t, 0.24692474439337447f);
  p = __builtin_fmaf(p, t, -0.14670328476729463f);
  p = __builtin_fmaf(p, t, 0.15823428115939212f);
  p = __builtin_fmaf(p, t, 0.0520316513544866f);
  p = __builtin_fmaf(p, t, 0.10344868697324719f);
  p = __builtin_fmaf(p, t, 0.10366847941107675f);
  p = __builtin_fmaf(p, t, 0.10440969988813159f);
  q = p * t * e;
}

// erfc(x), x >= 0
__device__ __forceinline__ float erfc_pos(float x) {
  const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, x, 1.0f));
  float p = 0.17087277f;
  p = fmaf(p, t, -0.82215223f);
  p = fmaf(p, t, 1.48851587f);
  p = fmaf(p, t, -1.13520398f);
  p = fmaf(p, t, 0.27886807f);
  p = fmaf(p, t, -0.18628806f);
  p = fmaf(p, t, 0.09678418f);
  p = fmaf(p, t, 0.37409196f);
  p = fmaf(p, t, 1.00002368f);
  p = fmaf(p, t, -1.26551223f);
  return t * exp_neg(fmaf(-x, x, p));
}

// standard normal CDF and density
__device__ __forceinline__ float phi_cdf(float r) {
  const float h = 0.5f * erfc_pos(fabsf(r) * 0.70710678118654752f);  // upper tail of |r|
  return r < 0.0f ? h : 1.0f - h;
}
__device__ __forceinline__ float phi_pdf(float r) { return 0.39894228040143268f * exp_neg(-0.5f * r * r); }

}  // namespace cp
