// cp_fit.hpp -- per-vertex fitting arithmetic of the range and
// location-scale models, and the correctly rounded helpers of the fits.
//
// Rules (Sec. 5.1 and 5.2):
//   uniform       lo = min, hi = max of the members
//   Epanechnikov  m = mean, w = bw * std(ddof) * M^(-1/5)
//   Gaussian      mu = mean, sigma = std(ddof)  (the Epanechnikov arithmetic
//                 with another scale)
//   degenerate    all members equal: lo/hi = x -/+ eps*max(1,|x|), Epanechnikov
//                 w (Gaussian sigma) = eps*max(1,|m|)
// Statistics are accumulated in FP64 about the first member (shifted sums).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "cpcrit.h"

namespace cp {

// one operation, rounded once (no contraction with its neighbours)
#if defined(__HIP_DEVICE_COMPILE__)
#define CP_RN(NAME, OP, F32, F64)                                                              \
  __host__ __device__ __forceinline__ float rn_##NAME(float a, float b) { return F32(a, b); } \
  __host__ __device__ __forceinline__ double rn_##NAME(double a, double b) { return F64(a, b); }
#else
#define CP_RN(NAME, OP, F32, F64)                                                            \
  __host__ __device__ __forceinline__ float rn_##NAME(float a, float b) { return a OP b; } \
  __host__ __device__ __forceinline__ double rn_##NAME(double a, double b) { return a OP b; }
#endif
CP_RN(sub, -, __fsub_rn, __dsub_rn)
CP_RN(add, +, __fadd_rn, __dadd_rn)
CP_RN(mul, *, __fmul_rn, __dmul_rn)
CP_RN(div, /, __fdiv_rn, __ddiv_rn)
#undef CP_RN
__host__ __device__ __forceinline__ float rn_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__host__ __device__ __forceinline__ double rn_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// degenerate half-width of the range model: eps * max(1, |x|), rounded once
template <typename T>
__device__ __forceinline__ T degenerate_half(T eps, T x) {
  return rn_mul(eps, x < T(0) ? (-x > T(1) ? -x : T(1)) : (x > T(1) ? x : T(1)));
}

// a / M, correctly rounded, with iM = 1 / M rounded: the quotient corrected
// twice by its exact remainder (Markstein's scheme: the first correction leaves
// at most one unit in the last place, the second then rounds correctly).  Five
// operations against the fifteen of a division; values whose remainder could
// underflow or overflow are divided.
__device__ __forceinline__ double div_count(double a, double M, double iM) {
  const double s = fabs(a);
  if (!(s >= 1e-280 && s <= 1e300)) return a / M;
  double q = a * iM;
  q = fma(fma(-q, M, a), iM, q);
  return fma(fma(-q, M, a), iM, q);
}

// Bin of a member x of a vertex's range [lo, hi]: floor((x - lo) / (hi - lo) * nb),
// clamped.  All members share the divisor, so the quotient is its rounded
// reciprocal's product, corrected twice by the remainder (Markstein's scheme, as
// div_count), five operations.  It is the division's, correctly rounded, where
// the remainder is exact: its lowest bit is 2^-46 (FP64 2^-104) of range times
// quotient, at least 2^-149 (2^-1074) for a range from 1e-20 (1e-200) on and a
// quotient down to 2^-36, and a smaller one is bin 0 either way.  Ranges outside
// the limits, infinite and NaN ones divide.
template <typename T>
struct BinOf {
  T lo, range, inv, fnb;
  int nb;
  bool exact;
  __host__ __device__ __forceinline__ BinOf(T lo_, T hi, int nb_) : lo(lo_), range(rn_sub(hi, lo_)), fnb(T(nb_)), nb(nb_) {
    constexpr T kLo = sizeof(T) == 8 ? T(1e-200) : T(1e-20f), kHi = sizeof(T) == 8 ? T(1e200) : T(1e30f);
    exact = range >= kLo && range <= kHi;
    inv = rn_div(T(1), range);
  }
  // a / range
  __host__ __device__ __forceinline__ T quotient(T a) const {
    if (!exact) return rn_div(a, range);
    T t = rn_mul(a, inv);
    t = rn_fma(rn_fma(-t, range, a), inv, t);
    return rn_fma(rn_fma(-t, range, a), inv, t);
  }
  __host__ __device__ __forceinline__ int operator()(T x) const {
    const int j = (int)rn_mul(quotient(rn_sub(x, lo)), fnb);
    return j < 0 ? 0 : (j > nb - 1 ? nb - 1 : j);
  }
};

// Running statistics of one vertex's members, then its parameters.
// Uniform: (lo, hi) = (min, max); Epanechnikov / Gaussian: (m, w) with
// w = wscale * sqrt(sum of squared deviations).  Every fit kernel feeds the
// members of a vertex in order k = 0, 1, ..., M-1 through these operations,
// so all of them give the same parameters bit for bit.
//
// The Epanechnikov branch detects "all members equal" without a min / max:
// with x0 the first member and d = x - x0 in FP64, some member differs from
// x0 exactly when some |d| > 0 (the difference of two distinct values of the
// field's type is never 0 in FP64).  A NaN member gives a NaN d, which the
// test ignores, as the min / max comparisons ignore it; a NaN first member
// makes every d NaN: degenerate, as !(min < max) is then.  In FP32 no square of
// a d underflows, so the sum of squares tells as much (SQ) without a comparison
// per member; only where it is NaN are the members (member(k)) looked at again.
template <typename T, int MODEL, bool SQ = sizeof(T) == 4>
struct FitAcc {
  T mn, mx;
  double shift, s1, s2;
  bool spread;
  __device__ __forceinline__ void first(T x0) {
    if (MODEL == CP_UNIFORM) {
      mn = mx = x0;
    } else {
      shift = (double)x0;
      s1 = s2 = 0.0;
      spread = false;
    }
  }
  __device__ __forceinline__ void add(T xk) {
    if (MODEL == CP_UNIFORM) {
      mn = xk < mn ? xk : mn;
      mx = xk > mx ? xk : mx;
    } else {
      const double d = (double)xk - shift;
      if (!SQ) spread = spread || fabs(d) > 0.0;
      s1 += d;
      s2 = fma(d, d, s2);
    }
  }
  // iM = 1 / M
  template <typename Member>
  __device__ __forceinline__ void finish(int M, double iM, double wscale, double eps, T& p0, T& p1, Member member) {
    if (MODEL == CP_UNIFORM) {
      if (!(mn < mx)) {
        const T e = degenerate_half(T(eps), mn);
        p0 = rn_sub(mn, e);
        p1 = rn_add(mn, e);
      } else {
        p0 = mn;
        p1 = mx;
      }
      return;
    }
    if (SQ) {
      spread = s2 > 0.0;
      if (s2 != s2)
        for (int k = 1; k < M; ++k) spread = spread || fabs((double)member(k) - shift) > 0.0;
    }
    const double mean = shift + div_count(s1, (double)M, iM);
    double w;
    if (!spread) {
      w = eps * fmax(1.0, fabs(mean));
    } else {
      const double ss = fmax(s2 - div_count(s1 * s1, (double)M, iM), 0.0);
      w = wscale * sqrt(ss);
    }
    p0 = (T)mean;
    p1 = (T)w;
  }
};

// Parameters (p0, p1) of one vertex from its M members, member k at
// mem[at + k*ps].
template <typename T, int MODEL>
__device__ __forceinline__ void fit_ue_vertex(const T* __restrict__ mem, int M, int64_t ps, int64_t at, double iM,
                                              double wscale, double eps, T& p0, T& p1) {
  FitAcc<T, MODEL> acc;
  acc.first(mem[at]);
#pragma unroll 4
  for (int k = 1; k < M; ++k) acc.add(mem[(int64_t)k * ps + at]);
  acc.finish(M, iM, wscale, eps, p0, p1, [&](int k) { return mem[(int64_t)k * ps + at]; });
}

}  // namespace cp
