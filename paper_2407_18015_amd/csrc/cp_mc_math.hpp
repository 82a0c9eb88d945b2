// cp_mc_math.hpp -- per-sample math of the Gaussian Monte Carlo estimators
// (normal deviates from uniforms, the normal CDF and density), on the
// hardware transcendental instructions of gfx950; upper_tail also serves the
// FP32 independent-Gaussian quadrature.
//
// Measured against FP64 on the generator's uniforms: v_sin_f32 / v_cos_f32
// (argument in revolutions) 1.3e-7 absolute, v_sqrt_f32 9e-8, v_exp_f32
// 8e-8 and v_rcp_f32 9e-8 relative; v_log_f32 within one ulp of log2.
// Upper tails of the normal distribution are exp(-z^2/2) times a polynomial in a
// reciprocal, so one costs a reciprocal, seven or eight fused multiply-adds and
// one exponential.  (The complementary error function of Numerical Recipes,
// Press et al., 2nd ed., Sec. 6.2, routine erfcc, a Chebyshev fit of log(erfc)
// to 1.2e-7, is the alternative: four more instructions, and less exact.)
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

// the same over kDeviateScale = sqrt(2 ln 2), which the caller's factors take
constexpr float kDeviateScale = 1.1774100225154747f;
__device__ __forceinline__ void box_muller_scaled(float u0, float u1, float& z0, float& z1) {
  const float rad = __builtin_amdgcn_sqrtf(-__builtin_amdgcn_logf(u0));
  z0 = rad * __builtin_amdgcn_cosf(u1);
  z1 = rad * __builtin_amdgcn_sinf(u1);
}

// 2^y for y <= 0 (the arguments here)
__host__ __device__ __forceinline__ float exp2_neg(float y) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_exp2f(y);
#else
  return exp2f(y);
#endif
}

constexpr double kTailScale = 0.84932180028801904272;  // sqrt(log2(e) / 2)

// From zs = kTailScale z: e = exp(-z^2 / 2), q = Pr(N(0, 1) > |z|) = t p8(t) e;
// slope = kTailSlope (in a vector register it issues at full rate)
constexpr float kTailSlope = 0.30804520612834824f;
__host__ __device__ __forceinline__ void upper_tail(float zs, float slope, float& q, float& e) {
  const float u = __builtin_fmaf(slope, __builtin_fabsf(zs), 1.0f);
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

// FP64: 2^y for -1e4 < y <= 0 (or NaN).  y = n + f with |f| <= 1/2, 2^f = 1 +
// f p10(f) (interpolated at Chebyshev points, 2e-17).
__host__ __device__ __forceinline__ double exp2_neg(double y) {
  const double n = __builtin_rint(y), f = y - n;
  double p = 4.4549605981865186e-10;
  p = __builtin_fma(p, f, 7.072585949269223e-09);
  p = __builtin_fma(p, f, 1.0178062445845774e-07);
  p = __builtin_fma(p, f, 1.321544258792169e-06);
  p = __builtin_fma(p, f, 1.525273382983612e-05);
  p = __builtin_fma(p, f, 0.0001540353044173605);
  p = __builtin_fma(p, f, 0.0013333558146416936);
  p = __builtin_fma(p, f, 0.009618129107606888);
  p = __builtin_fma(p, f, 0.0555041086648216);
  p = __builtin_fma(p, f, 0.24022650695910097);
  p = __builtin_fma(p, f, 0.6931471805599453);
  return __builtin_ldexp(__builtin_fma(f, p, 1.0), (int)n);
}

// FP64, from the same zs: q = e p9(x) / p10(x) with x = |zs|, the ratio
// interpolating exp(z^2 / 2) Pr(N(0, 1) > z) at Chebyshev points of (z - 4) /
// (z + 4) over z <= 30 (9e-17 there, 6e-15 at 38, where q vanishes; one degree
// less reaches 3e-17 up to 9.9, but 1e-10 at 28).  All coefficients are
// positive, so both polynomials lose no digits.  Half the work of erfc and exp,
// which evaluate every range of z that a wave holds and the exponential twice.
__host__ __device__ __forceinline__ void upper_tail(double zs, double, double& q, double& e) {
  double x = __builtin_fabs(zs);
  x = x > 33.0 ? 33.0 : x;  // 2^-x^2 is 0 from here on
  e = exp2_neg(-x * x);
  double n = 5.4831700515742165e-06;
  n = __builtin_fma(n, x, 0.00012723838728142183);
  n = __builtin_fma(n, x, 0.0014414748868951692);
  n = __builtin_fma(n, x, 0.010325276039219889);
  n = __builtin_fma(n, x, 0.051173036386345586);
  n = __builtin_fma(n, x, 0.18141961556916425);
  n = __builtin_fma(n, x, 0.4602520793420452);
  n = __builtin_fma(n, x, 0.8092325515282937);
  n = __builtin_fma(n, x, 0.9039577837722884);
  n = __builtin_fma(n, x, 0.5);
  double d = 1.6182640174000773e-05;
  d = __builtin_fma(d, x, 0.00037552237450265343);
  d = __builtin_fma(d, x, 0.004265940310335866);
  d = __builtin_fma(d, x, 0.03074417129493282);
  d = __builtin_fma(d, x, 0.15408044501589319);
  d = __builtin_fma(d, x, 0.5570200103834194);
  d = __builtin_fma(d, x, 1.4629334901909385);
  d = __builtin_fma(d, x, 2.7442300072908297);
  d = __builtin_fma(d, x, 3.506283604000219);
  d = __builtin_fma(d, x, 2.7473528462442243);
  d = __builtin_fma(d, x, 1.0);
#if defined(__HIP_DEVICE_COMPILE__)
  // reciprocal to 2^-24, one Newton step, and the quotient corrected by its remainder
  double r = __builtin_amdgcn_rcp(d);
  r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
  const double a = n * r;
  q = __builtin_fma(__builtin_fma(-d, a, n), r, a) * e;
#else
  q = n / d * e;
#endif
}

// The tail alone for the Monte Carlo estimators, e kept to itself: p7 fitted
// the same way (8.2e-8, against 1.2e-7 of erfcc) with t = 1 / (1 + 0.33 x); in
// FP32 within 5.0e-7 (rms 1.3e-7) of the exact tail for |z| < 2.
__device__ __forceinline__ float upper_tail7(float zs) {
  const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.2747430216820403f, __builtin_fabsf(zs), 1.0f));
  float p = -0.06796436939967895f;
  p = __builtin_fmaf(p, t, 0.23134397803518358f);
  p = __builtin_fmaf(p, t, -0.17771920726259405f);
  p = __builtin_fmaf(p, t, 0.20627053501343956f);
  p = __builtin_fmaf(p, t, 0.022505477741305194f);
  p = __builtin_fmaf(p, t, 0.10096186106928375f);
  p = __builtin_fmaf(p, t, 0.09141862964257003f);
  p = __builtin_fmaf(p, t, 0.09318305433040192f);
  return p * t * exp2_neg(-zs * zs);
}

// standard normal density
__device__ __forceinline__ float phi_pdf(float r) {
  return 0.39894228040143268f * __builtin_amdgcn_exp2f(-0.5f * r * r * 1.4426950408889634f);
}

}  // namespace cp
