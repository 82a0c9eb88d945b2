// cp_device.hpp -- device-side building blocks of the closed-form kernels.
//
// Every routine works in a vertex-local coordinate frame: all breakpoints
// are differences of parameters of nearby vertices, so their magnitude is
// the distribution width rather than the data value.  The paper warns that
// its high-order templates become unstable for large or fractional data
// values (Sec. 4.3); in FP32 a node placed in global coordinates near 0.5
// already carries 3e-8 of rounding, which is 5e-6 of a 0.006-wide
// Epanechnikov kernel.  In the local frame the error is relative to the
// widths, and nothing is ever expanded into monomials.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

// Pure arithmetic is host+device so it can also be exercised on the CPU.
#define CP_HD __host__ __device__ __forceinline__

namespace cp {

// Fused multiply-add in the operand precision (FP32 stays FP32).
template <typename T>
CP_HD T cfma(T a, T b, T c);
template <>
CP_HD float cfma<float>(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}
template <>
CP_HD double cfma<double>(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}

// Reciprocal: the hardware v_rcp_f32 (1 ulp) in FP32 device code, exact
// division otherwise.  Parameters are reciprocated once per vertex.
template <typename T>
CP_HD T crcp(T x) {
  return T(1) / x;
}
template <>
CP_HD float crcp<float>(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.0f / x;
#endif
}

// ---------------------------------------------------------------------------
// Gauss-Legendre rules on [-1, 1]; an N-point rule integrates polynomials of
// degree <= 2N-1 exactly.
// ---------------------------------------------------------------------------
template <int N>
struct GL;
template <>
struct GL<1> {
  static constexpr double x[1] = {0.0};
  static constexpr double w[1] = {2.0};
};
template <>
struct GL<2> {
  static constexpr double x[2] = {-0.57735026918962576451, 0.57735026918962576451};
  static constexpr double w[2] = {1.0, 1.0};
};
template <>
struct GL<3> {
  static constexpr double x[3] = {-0.77459666924148337704, 0.0, 0.77459666924148337704};
  static constexpr double w[3] = {0.55555555555555555556, 0.88888888888888888889,
                                  0.55555555555555555556};
};
template <>
struct GL<4> {
  static constexpr double x[4] = {-0.86113631159405257522, -0.33998104358485626480, 0.33998104358485626480,
                                  0.86113631159405257522};
  static constexpr double w[4] = {0.34785484513745385737, 0.65214515486254614263, 0.65214515486254614263,
                                  0.34785484513745385737};
};
template <>
struct GL<5> {
  static constexpr double x[5] = {-0.90617984593866399280, -0.53846931010568309104, 0.0,
                                  0.53846931010568309104, 0.90617984593866399280};
  static constexpr double w[5] = {0.23692688505618908751, 0.47862867049936646804,
                                  0.56888888888888888889, 0.47862867049936646804,
                                  0.23692688505618908751};
};
template <>
struct GL<6> {
  static constexpr double x[6] = {-0.93246951420315202781, -0.66120938646626451366,
                                  -0.23861918608319690863, 0.23861918608319690863,
                                  0.66120938646626451366,  0.93246951420315202781};
  static constexpr double w[6] = {0.17132449237917034504, 0.36076157304813860757,
                                  0.46791393457269104739, 0.46791393457269104739,
                                  0.36076157304813860757, 0.17132449237917034504};
};
template <>
struct GL<7> {
  static constexpr double x[7] = {-0.94910791234275852453, -0.74153118559939443986, -0.40584515137739716691, 0.0,
                                  0.40584515137739716691,  0.74153118559939443986,  0.94910791234275852453};
  static constexpr double w[7] = {0.12948496616886969327, 0.27970539148927666790, 0.38183005050511894495,
                                  0.41795918367346938776, 0.38183005050511894495, 0.27970539148927666790,
                                  0.12948496616886969327};
};
template <>
struct GL<8> {
  static constexpr double x[8] = {-0.96028985649753623168, -0.79666647741362673959,
                                  -0.52553240991632898582, -0.18343464249564980494,
                                  0.18343464249564980494,  0.52553240991632898582,
                                  0.79666647741362673959,  0.96028985649753623168};
  static constexpr double w[8] = {0.10122853629037625915, 0.22238103445337447054,
                                  0.31370664587788728734, 0.36268378337836198297,
                                  0.36268378337836198297, 0.31370664587788728734,
                                  0.22238103445337447054, 0.10122853629037625915};
};
template <>
struct GL<10> {
  static constexpr double x[10] = {-0.97390652851717172008, -0.86506336668898451073, -0.67940956829902440623,
                                   -0.43339539412924719080, -0.14887433898163121088, 0.14887433898163121088,
                                   0.43339539412924719080,  0.67940956829902440623,  0.86506336668898451073,
                                   0.97390652851717172008};
  static constexpr double w[10] = {0.066671344308688137594, 0.14945134915058059315, 0.21908636251598204400,
                                   0.26926671930999635509,  0.29552422471475287017, 0.29552422471475287017,
                                   0.26926671930999635509,  0.21908636251598204400, 0.14945134915058059315,
                                   0.066671344308688137594};
};

// What the N-point rule misses on y^(2N) over [-1, 1],
// 2^(2N+1) (N!)^4 / ((2N+1) ((2N)!)^2): for a polynomial of degree <= 2N+1
// whose y^(2N) coefficient is c, the integral is the rule's sum plus e c (an
// odd top term integrates to zero under both).
template <int N>
struct GLRem;
template <>
struct GLRem<1> {
  static constexpr double e = 2.0 / 3.0;
};
template <>
struct GLRem<2> {
  static constexpr double e = 8.0 / 45.0;
};
template <>
struct GLRem<4> {
  static constexpr double e = 128.0 / 11025.0;
};
template <>
struct GLRem<7> {
  static constexpr double e = 512.0 / 2760615.0;
};

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
// A constant held in a vector register: an FP32 instruction with a modifier
// cannot carry a literal, and with a scalar register it issues at half rate.
// (FP64 issues at one rate, and registers are short: left to the compiler.)
CP_HD inline float vconst(float v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(v));
#endif
  return v;
}
CP_HD inline double vconst(double v) { return v; }
template <typename T>
CP_HD T tmin(T a, T b) {
  return b < a ? b : a;
}
template <typename T>
CP_HD T tmax(T a, T b) {
  return a < b ? b : a;
}
// minimum of two values known not to be NaN (one v_min instruction instead
// of a compare and a select)
CP_HD inline float fmin_nn(float a, float b) { return __builtin_fminf(a, b); }
CP_HD inline double fmin_nn(double a, double b) { return __builtin_fmin(a, b); }
CP_HD inline float fmax_nn(float a, float b) { return __builtin_fmaxf(a, b); }
CP_HD inline double fmax_nn(double a, double b) { return __builtin_fmax(a, b); }
// v clamped to lo <= hi, no NaN: one v_med3_f32 in FP32
CP_HD inline float clamp_nn(float v, float lo, float hi) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_fmed3f(v, lo, hi);
#else
  return fmin_nn(fmax_nn(v, lo), hi);
#endif
}
CP_HD inline double clamp_nn(double v, double lo, double hi) { return fmin_nn(fmax_nn(v, lo), hi); }
// v clamped to [0, 1]: a modifier of the instruction that produces v
CP_HD inline float clamp01(float v) { return fmin_nn(fmax_nn(v, 0.0f), 1.0f); }
CP_HD inline double clamp01(double v) { return fmin_nn(fmax_nn(v, 0.0), 1.0); }
template <typename T>
CP_HD T qnan() {
  return __builtin_nan("");
}

// Selection by a mask of ones or zeros: a < b as a subtraction and a shift,
// and m ? a : b as one v_bitop3_b32, issue in half the cycles of v_cmp and
// v_cndmask on gfx950.  Keys are not NaN; equal keys may give either mask.
CP_HD uint32_t sign_mask(float a) { return (uint32_t)(__builtin_bit_cast(int32_t, a) >> 31); }
CP_HD uint32_t sign_mask(double a) { return (uint32_t)((int32_t)(__builtin_bit_cast(uint64_t, a) >> 32) >> 31); }
template <typename T>
CP_HD uint32_t less_mask(T a, T b) {
  return sign_mask(a - b);
}
CP_HD uint32_t sel_bits(uint32_t m, uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA);
#else
  return (m & a) | (~m & b);
#endif
}
CP_HD float sel(uint32_t m, float a, float b) {
  return __builtin_bit_cast(float, sel_bits(m, __builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b)));
}
CP_HD double sel(uint32_t m, double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  return __builtin_bit_cast(double, (uint64_t)sel_bits(m, (uint32_t)(x >> 32), (uint32_t)(y >> 32)) << 32 |
                                        sel_bits(m, (uint32_t)x, (uint32_t)y));
}

// Sorting network for four keys (5 comparators), payload follows its key; it
// records whether each comparator swapped, so that values computed in sorted
// order can be taken back to neighbour order by unsort4 (the comparators in
// reverse order, each its own inverse): ten selects per array instead of a
// select per (slot, neighbour) pair.
template <typename T, int P>
CP_HD void cswap_rec(T& ka, T& kb, T (&pa)[P], T (&pb)[P], uint32_t& m) {
  m = less_mask(kb, ka);
  const T t = sel(m, kb, ka);
  kb = sel(m, ka, kb);
  ka = t;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const T u = sel(m, pb[p], pa[p]);
    pb[p] = sel(m, pa[p], pb[p]);
    pa[p] = u;
  }
}

template <typename T, int P>
CP_HD void sort4_rec(T (&k)[4], T (&p)[4][P], uint32_t (&sw)[5]) {
  cswap_rec<T, P>(k[0], k[1], p[0], p[1], sw[0]);
  cswap_rec<T, P>(k[2], k[3], p[2], p[3], sw[1]);
  cswap_rec<T, P>(k[0], k[2], p[0], p[2], sw[2]);
  cswap_rec<T, P>(k[1], k[3], p[1], p[3], sw[3]);
  cswap_rec<T, P>(k[1], k[2], p[1], p[2], sw[4]);
}

template <typename T>
CP_HD void uswap(T& a, T& b, uint32_t m) {
  const T t = sel(m, b, a);
  b = sel(m, a, b);
  a = t;
}

template <typename T>
CP_HD void unsort4(T (&v)[4], const uint32_t (&sw)[5]) {
  uswap(v[1], v[2], sw[4]);
  uswap(v[1], v[3], sw[3]);
  uswap(v[0], v[2], sw[2]);
  uswap(v[2], v[3], sw[1]);
  uswap(v[0], v[1], sw[0]);
}

// ===========================================================================
// Uniform model (Sec. 4.3).  Local frame with origin at the vertex lower
// end: vertex support [0, Lv]; neighbour i support [a_i, b_i].
//
// Task 1 (Sec. 4.1.1): b_min = min(Lv, b_i); nothing if b_min <= 0.  Start
// points clamped to [0, b_min] and sorted give the pieces
// [0,c0], [c0,c1], [c1,c2], [c2,c3], [c3,b_min]; on piece k exactly the k
// neighbours sorted first have started (Tasks 2-3, Template k+1), so every
// lane runs the same five pieces (empty ones contribute zero).
// On piece k the integrand (1/Lv) prod_{i<k} (b_i - x)/L_i has degree k:
// Gauss-Legendre with 1 and 2 nodes is exact for k = 1 and 3; k = 2 and 4
// take 1 and 2 nodes plus the rule's remainder on the top-degree term (its
// coefficient the product of the factors' slopes).  k = 4 is the centre.
// ===========================================================================
template <typename T>
struct UniSide {
  T Lv, iLv;
  T c[4];      // sorted clamped start points
  T b[4];      // matching upper ends
  T iL[4];     // matching 1/(b - a)
  uint32_t sw[5];  // comparator swaps of the sort (unsort4 restores neighbour order)
  T bmin;
  bool empty;
};

// an absent neighbour is passed as a = 2 Lv, b = 3 Lv, iL = 1 / Lv: a factor
// that would start beyond b_min, never active on a non-empty piece
template <typename T>
CP_HD void uni_setup(UniSide<T>& s, T Lv, T iLv, const T (&a)[4], const T (&b)[4], const T (&iL)[4]) {
  s.Lv = Lv;
  s.iLv = iLv;
  s.bmin = fmin_nn(fmin_nn(fmin_nn(Lv, b[0]), fmin_nn(b[1], b[2])), b[3]);
  s.empty = !(s.bmin > T(0));
  T pay[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s.c[i] = clamp_nn(a[i], T(0), s.bmin);
    pay[i][0] = b[i];
    pay[i][1] = iL[i];
  }
  sort4_rec<T, 2>(s.c, pay, s.sw);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s.b[i] = pay[i][0];
    s.iL[i] = pay[i][1];
  }
}

// integral over [l, r] of prod_{i<K} (b_i - x) iL_i  (times nothing else);
// REM: K = 2N, and the y^K coefficient prod be_i gets the rule's remainder
template <typename T, int K, int N, bool REM = false>
CP_HD T uni_piece(const UniSide<T>& s, T l, T r) {
  static_assert(REM ? K == 2 * N : K <= 2 * N - 1, "rule too small for the piece");
  const T mid = (l + r) * T(0.5), hl = (r - l) * T(0.5);
  T al[K], be[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    al[i] = (s.b[i] - mid) * s.iL[i];
    be[i] = hl * s.iL[i];
  }
  T sum = T(0);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const T x = T(GL<N>::x[j]);
    T prod = T(1);
#pragma unroll
    for (int i = 0; i < K; ++i) prod *= cfma(-be[i], x, al[i]);
    sum = cfma(T(GL<N>::w[j]), prod, sum);
  }
  if constexpr (REM) {
    T c = be[0];
#pragma unroll
    for (int i = 1; i < K; ++i) c *= be[i];
    sum = cfma(T(GLRem<N>::e), c, sum);  // (-be_i) for each of an even number of factors
  }
  return sum * hl;
}

// the pieces up to three factors (the fourth is the centre's)
template <typename T>
CP_HD T uni_side_value(const UniSide<T>& s) {
  if (s.empty) return T(0);
  T acc = s.c[0];  // piece 0: no factor
  acc += uni_piece<T, 1, 1>(s, s.c[0], s.c[1]);
  acc += uni_piece<T, 2, 1, true>(s, s.c[1], s.c[2]);
  acc += uni_piece<T, 3, 2>(s, s.c[2], s.c[3]);
  return acc * s.iLv;
}

// The centre: the range [max(0, a_i), min(Lv, b_i)] on which all four
// neighbours vary (if there is one).  It is the last piece of the minimum's
// side, of the maximum's (reflected) and the middle one of both saddle terms,
// and S and F = 1 - S need the same nodes, so all of them are integrated here:
// out = (prod S, prod F, S_e F_n S_w F_s, F_e S_n F_w S_s), the last two with
// SAD.  Returns whether there is a centre.
//
// Measured at 2048^2 (20-member fit, FP32; with the mask selections above and
// v_med3 clamps, against one centre per side): Epanechnikov forward 92 -> 78 us,
// adjoint 159 -> 140, uniform forward 45 -> 40, adjoint 71 both; all are bound by
// vector issue, of which the selections took a fifth.
template <typename T, bool SAD>
CP_HD bool uni_centre(T Lv, T iLv, const T (&a)[4], const T (&b)[4], const T (&iL)[4], T (&out)[4]) {
  const T l = fmax_nn(fmax_nn(fmax_nn(T(0), a[0]), fmax_nn(a[1], a[2])), a[3]);
  const T r = fmin_nn(fmin_nn(fmin_nn(Lv, b[0]), fmin_nn(b[1], b[2])), b[3]);
#pragma unroll
  for (int q = 0; q < 4; ++q) out[q] = T(0);
  if (!(l < r)) return false;
  const T mid = (l + r) * T(0.5), hl = (r - l) * T(0.5);
  T al[4], af[4], be[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    al[i] = (b[i] - mid) * iL[i];
    af[i] = (mid - a[i]) * iL[i];
    be[i] = hl * iL[i];
  }
  T s[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
  for (int j = 0; j < 2; ++j) {  // both weights 1
    const T x = T(GL<2>::x[j]);
    T S[4], F[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      S[i] = cfma(-be[i], x, al[i]);
      F[i] = cfma(be[i], x, af[i]);
    }
    const T sa = S[0] * S[2], sb = S[1] * S[3], fa = F[0] * F[2], fb = F[1] * F[3];
    s[0] = cfma(sa, sb, s[0]);
    s[1] = cfma(fa, fb, s[1]);
    if (SAD) {
      s[2] = cfma(sa, fb, s[2]);
      s[3] = cfma(fa, sb, s[3]);
    }
  }
  // degree 4: the rule's remainder, the same for all (an even number of
  // factors of either slope)
  const T c = be[0] * be[1] * (be[2] * be[3]), k = hl * iLv;
#pragma unroll
  for (int q = 0; q < (SAD ? 4 : 2); ++q) out[q] = k * cfma(T(GLRem<2>::e), c, s[q]);
  return true;
}

// Local derivatives of one side:  f(Lv, a_i, b_i) = (1/Lv) int_0^{b_min} prod S_i
//   df/da_i = (1/L_i) int_{i active} p_v prod_k S_k
//   df/db_i = (1/L_i) int_{i active} p_v (prod_{k!=i} S_k - prod_k S_k)
//   df/dLv  = (-f + prod_i S_i(Lv)) / Lv
template <typename T>
struct UniGrad {
  T f, dLv;
  T da[4], db[4];  // by neighbour index 0..3
};

// REM: K = 2N; the leave-one-out sums (degree K - 1) are exact, the full
// product (degree K) gets the rule's remainder on prod be_i
template <typename T, int K, int N, bool REM = false>
CP_HD void uni_piece_grad(const UniSide<T>& s, T l, T r, T& full, T (&loo)[4]) {
  static_assert(REM ? K == 2 * N : K <= 2 * N - 1, "rule too small for the piece");
  const T mid = (l + r) * T(0.5), hl = (r - l) * T(0.5);
  T al[K], be[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    al[i] = (s.b[i] - mid) * s.iL[i];
    be[i] = hl * s.iL[i];
  }
  T sf = T(0), sl[K];
#pragma unroll
  for (int i = 0; i < K; ++i) sl[i] = T(0);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const T x = T(GL<N>::x[j]);
    const T wj = T(GL<N>::w[j]);
    T f[K], pre[K + 1], suf[K + 1];
#pragma unroll
    for (int i = 0; i < K; ++i) f[i] = cfma(-be[i], x, al[i]);
    pre[0] = T(1);
#pragma unroll
    for (int i = 0; i < K; ++i) pre[i + 1] = pre[i] * f[i];
    suf[K] = T(1);
#pragma unroll
    for (int i = K - 1; i >= 0; --i) suf[i] = suf[i + 1] * f[i];
    sf = cfma(wj, pre[K], sf);
#pragma unroll
    for (int i = 0; i < K; ++i) sl[i] = cfma(wj, pre[i] * suf[i + 1], sl[i]);
  }
  if constexpr (REM) {
    T c = be[0];
#pragma unroll
    for (int i = 1; i < K; ++i) c *= be[i];
    sf = cfma(T(GLRem<N>::e), c, sf);
  }
  full = sf * hl;
#pragma unroll
  for (int i = 0; i < K; ++i) loo[i] += sl[i] * hl;
}

template <typename T>
CP_HD void uni_side_grad(const UniSide<T>& s, UniGrad<T>& g) {
  g.f = T(0);
  g.dLv = T(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) g.da[i] = g.db[i] = T(0);
  if (s.empty) return;
  T I[5];
  T loo[4] = {T(0), T(0), T(0), T(0)};  // sorted slots; accumulated over pieces where active
  T act[4] = {T(0), T(0), T(0), T(0)};  // full integral over pieces where slot is active
  I[0] = s.c[0];
  uni_piece_grad<T, 1, 1>(s, s.c[0], s.c[1], I[1], loo);
  uni_piece_grad<T, 2, 1, true>(s, s.c[1], s.c[2], I[2], loo);
  uni_piece_grad<T, 3, 2>(s, s.c[2], s.c[3], I[3], loo);
  uni_piece_grad<T, 4, 2, true>(s, s.c[3], s.bmin, I[4], loo);
  // slot i is active on pieces i+1..4
  act[3] = I[4];
  act[2] = act[3] + I[3];
  act[1] = act[2] + I[2];
  act[0] = act[1] + I[1];
  const T iLv = s.iLv;
  const T f = (act[0] + I[0]) * iLv;
  g.f = f;
  // product of the survival factors at x = Lv (zero unless b_min = Lv)
  T gend = T(0);
  if (!(s.bmin < s.Lv)) {
    gend = T(1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // a factor that has not started at Lv is 1 (also an absent neighbour)
      T v = tmin(T(1), (s.b[i] - s.Lv) * s.iL[i]);
      gend *= (s.c[i] < s.Lv) ? tmax(v, T(0)) : T(1);
    }
  }
  g.dLv = (gend - f) * iLv;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    g.da[i] = act[i] * iLv * s.iL[i];
    g.db[i] = (loo[i] - act[i]) * iLv * s.iL[i];
  }
  // sorted slots -> neighbour index
  unsort4(g.da, s.sw);
  unsort4(g.db, s.sw);
}

// ===========================================================================
// Epanechnikov model (Sec. 4.3).  Local frame with origin at the vertex
// centre: vertex support [-wv, wv], neighbour i centre d_i, half-width w_i.
// pdf_v = 3/(4 wv) (1 - t^2), S_i = (1 - u)^2 (2 + u) / 4 with t = x/wv,
// u = (x - d_i)/w_i.  Piece k (k neighbours started) has degree 2 + 3k
// (the paper's order-15 remark, Sec. 4.3): Gauss-Legendre with 3 and 6
// nodes is exact for k = 1 and 3; k = 2 and 4 (degree 8 and 14) take 4 and 7
// nodes plus the rule's remainder on the top-degree term, whose coefficient
// is a product of the factors' leading coefficients; piece 0 is the vertex
// CDF in closed form.
// ===========================================================================
template <typename T>
struct EpaSide {
  T wv, iwv;
  T c[4], d[4], iw[4];
  uint32_t sw[5];  // comparator swaps of the sort (unsort4 restores neighbour order)
  T bmin;
  bool empty;
};

// an absent neighbour is passed as d = 4 wv, w = wv, iw = 1 / wv: a factor that
// would start beyond b_min, never active on a non-empty piece
template <typename T>
CP_HD void epa_setup(EpaSide<T>& s, T wv, T iwv, const T (&d)[4], const T (&w)[4], const T (&iw)[4]) {
  s.wv = wv;
  s.iwv = iwv;
  s.bmin = fmin_nn(fmin_nn(fmin_nn(wv, d[0] + w[0]), fmin_nn(d[1] + w[1], d[2] + w[2])), d[3] + w[3]);
  s.empty = !(s.bmin > -wv);
  T pay[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s.c[i] = clamp_nn(d[i] - w[i], -wv, s.bmin);
    pay[i][0] = d[i];
    pay[i][1] = iw[i];
  }
  sort4_rec<T, 2>(s.c, pay, s.sw);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s.d[i] = pay[i][0];
    s.iw[i] = pay[i][1];
  }
}

// 4 * vertex CDF at x: (1 + t)^2 (2 - t), t = x / wv
template <typename T>
CP_HD T epa_cdf4(const EpaSide<T>& s, T x) {
  const T t = x * s.iwv;
  const T o = T(1) + t;
  return o * o * (T(2) - t);
}

// 4 S(u) = u^3 - 3u + 2 in Horner form: three fused multiply-adds.  On a
// piece where the factor has started, u is in [-1, 1] and the rounding error
// is at most a few ulp of 3 in absolute terms.
template <typename T>
CP_HD T epa_s4(T u) {
  return cfma(cfma(u, u, T(-3)), u, T(2));
}

// integral over [l, r] of (1 - t^2) prod_{i<K} 4 S_i   (unscaled): the
// N-point rule, plus (REM) its remainder when the integrand's degree 2 + 3K
// is 2N: the y^(2N) coefficient is -bv^2 prod bu_i^3
template <typename T, int K, int N, bool REM = false>
CP_HD T epa_piece(const EpaSide<T>& s, T l, T r) {
  static_assert(REM ? 2 + 3 * K == 2 * N : 2 + 3 * K <= 2 * N - 1, "rule too small for the piece");
  const T mid = (l + r) * T(0.5), hl = (r - l) * T(0.5);
  const T av = mid * s.iwv, bv = hl * s.iwv;
  T au[K], bu[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    au[i] = (mid - s.d[i]) * s.iw[i];  // u = au + bu x
    bu[i] = hl * s.iw[i];
  }
  T sum = T(0);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const T x = T(GL<N>::x[j]);
    const T t = cfma(bv, x, av);
    T prod = cfma(-t, t, T(1));
#pragma unroll
    for (int i = 0; i < K; ++i) prod *= epa_s4(cfma(bu[i], x, au[i]));
    sum = cfma(T(GL<N>::w[j]), prod, sum);
  }
  if constexpr (REM) {
    T c = bv * bv;
#pragma unroll
    for (int i = 0; i < K; ++i) c *= bu[i] * bu[i] * bu[i];
    sum = cfma(T(-GLRem<N>::e), c, sum);
  }
  return sum * hl;
}

// the pieces up to three factors (the fourth is the centre's)
template <typename T>
CP_HD T epa_side_value(const EpaSide<T>& s) {
  if (s.empty) return T(0);
  const T kv = T(0.75) * s.iwv;  // pdf scale 3/(4 wv)
  const T acc = epa_cdf4(s, s.c[0]) * T(0.25);
  T p = epa_piece<T, 1, 3>(s, s.c[0], s.c[1]) * T(0.25);
  p = cfma(epa_piece<T, 2, 4, true>(s, s.c[1], s.c[2]), T(0.0625), p);
  p = cfma(epa_piece<T, 3, 6>(s, s.c[2], s.c[3]), T(0.015625), p);
  return cfma(kv, p, acc);
}

// Range and arguments of the centre (see uni_centre): u_i = au_i + bu_i y,
// t = av + bv y on y in [-1, 1].
template <typename T>
struct EpaCentre {
  T hl, av, bv, au[4], bu[4];
};
template <typename T>
CP_HD bool epa_centre_setup(EpaCentre<T>& c, T wv, T iwv, const T (&d)[4], const T (&w)[4], const T (&iw)[4]) {
  const T l = fmax_nn(fmax_nn(fmax_nn(-wv, d[0] - w[0]), fmax_nn(d[1] - w[1], d[2] - w[2])), d[3] - w[3]);
  const T r = fmin_nn(fmin_nn(fmin_nn(wv, d[0] + w[0]), fmin_nn(d[1] + w[1], d[2] + w[2])), d[3] + w[3]);
  const T mid = (l + r) * T(0.5);
  c.hl = (r - l) * T(0.5);
  c.av = mid * iwv;
  c.bv = c.hl * iwv;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    c.au[i] = (mid - d[i]) * iw[i];
    c.bu[i] = c.hl * iw[i];
  }
  return l < r;
}

// out as uni_centre; seven nodes and the remainder of the degree-14 term,
// -bv^2 prod bu_i^3 for all four products.  4 S and 4 F share u^2 - 3.
template <typename T, bool SAD>
CP_HD bool epa_centre(T wv, T iwv, const T (&d)[4], const T (&w)[4], const T (&iw)[4], T (&out)[4]) {
  EpaCentre<T> c;
#pragma unroll
  for (int q = 0; q < 4; ++q) out[q] = T(0);
  if (!epa_centre_setup(c, wv, iwv, d, w, iw)) return false;
  T s[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
  for (int j = 0; j < 7; ++j) {
    const T x = T(GL<7>::x[j]);
    const T t = cfma(c.bv, x, c.av);
    const T q = T(GL<7>::w[j]) * cfma(-t, t, T(1));
    T S[4], F[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const T u = cfma(c.bu[i], x, c.au[i]), o = cfma(u, u, T(-3));
      S[i] = cfma(o, u, T(2));
      F[i] = cfma(-o, u, T(2));
    }
    const T sa = q * (S[0] * S[2]), sb = S[1] * S[3], fa = q * (F[0] * F[2]), fb = F[1] * F[3];
    s[0] = cfma(sa, sb, s[0]);
    s[1] = cfma(fa, fb, s[1]);
    if (SAD) {
      s[2] = cfma(sa, fb, s[2]);
      s[3] = cfma(fa, sb, s[3]);
    }
  }
  T e = c.bv * c.bv;
#pragma unroll
  for (int i = 0; i < 4; ++i) e *= c.bu[i] * c.bu[i] * c.bu[i];
  const T k = T(0.75 / 256.0) * iwv * c.hl;
#pragma unroll
  for (int q = 0; q < (SAD ? 4 : 2); ++q) out[q] = k * cfma(T(-GLRem<7>::e), e, s[q]);
  return true;
}

// Local derivatives of one side, f(wv, d_i, w_i):
//   df/dd_i = int p_v p_i prod_{k!=i} S_k          (dS/dm = pdf)
//   df/dw_i = int p_v u_i p_i prod_{k!=i} S_k      (dS/dw = u pdf)
// and df/dwv = -(1/wv) sum_i (d_i df/dd_i + w_i df/dw_i), the scale
// invariance of P about the vertex centre (wv df/dwv + sum_i (d_i df/dd_i +
// w_i df/dw_i) = 0), which the caller forms in neighbour order (absent
// neighbours have zero derivatives): it equals -(1/wv) sum_i int x p_v p_i
// prod_{k!=i} S_k, since x = d_i + w_i u_i, and avoids integrating
// dpdf_v/dwv, whose integral over the support is 0 and cancels.  WF: also
// return f itself (the fused forward).
template <typename T>
struct EpaGrad {
  T f;
  T dd[4], dw[4];  // by neighbour index
};

// One piece with K started neighbours (sorted slots 0..K-1), N nodes.  The
// slot sums, times the piece's factor sc = 4^-(K-1) and its half-length, are
// added straight into the side's accumulators ad / aw (by sorted slot); WF:
// the piece's value, times fsc = 4^-K and the half-length, into `full`.
// The position sums have degree 3K + 1, the width sums and the value 3K + 2;
// REM: N = (3K + 2) / 2 nodes and the rule's remainder, from the y^(2N)
// coefficient, which is bv^2 prod_k bu_k^3 for every width sum (the leading
// coefficients -bv^2, -bu_i^2 and bu_i of its own factors, bu_k^3 of the
// others) and its negative for the value.
template <typename T, int K, int N, bool REM, bool WF>
CP_HD void epa_piece_grad(const EpaSide<T>& s, T l, T r, T sc, T fsc, T& full, T (&ad)[4], T (&aw)[4]) {
  static_assert(REM ? 3 * K + 2 == 2 * N : 3 * K + 2 <= 2 * N - 1, "rule too small for the piece");
  const T mid = (l + r) * T(0.5), hl = (r - l) * T(0.5);
  const T av = mid * s.iwv, bv = hl * s.iwv;
  T au[K], bu[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    au[i] = (mid - s.d[i]) * s.iw[i];  // u = au + bu x
    bu[i] = hl * s.iw[i];
  }
  T sf = T(0), sd[K], sww[K];
#pragma unroll
  for (int i = 0; i < K; ++i) sd[i] = sww[i] = T(0);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const T x = T(GL<N>::x[j]);
    const T t = cfma(bv, x, av);
    T u[K], S[K], pre[K + 1], suf[K + 1];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      u[i] = cfma(bu[i], x, au[i]);
      S[i] = epa_s4(u[i]);  // 4 S_i
    }
    // prefix products carry the node weight and the vertex pdf
    // (weight * 4 wv/3 * pdf_v = w_j (1 - t^2))
    pre[0] = T(GL<N>::w[j]) * cfma(-t, t, T(1));
#pragma unroll
    for (int i = 0; i < K; ++i) pre[i + 1] = pre[i] * S[i];
    suf[K] = T(1);
#pragma unroll
    for (int i = K - 1; i >= 0; --i) suf[i] = suf[i + 1] * S[i];
    if (WF) sf += pre[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      // (4 w_i / 3) p_i = 1 - u^2
      const T lw = cfma(-u[i], u[i], T(1)) * (pre[i] * suf[i + 1]);
      sd[i] += lw;
      sww[i] = cfma(lw, u[i], sww[i]);
    }
  }
  if constexpr (REM) {
    T c = bv * bv;
#pragma unroll
    for (int i = 0; i < K; ++i) c *= bu[i] * bu[i] * bu[i];
    const T ec = T(GLRem<N>::e) * c;
    if (WF) sf -= ec;
#pragma unroll
    for (int i = 0; i < K; ++i) sww[i] += ec;
  }
  const T ps = sc * hl;
  if (WF) full = cfma(sf, fsc * hl, full);
#pragma unroll
  for (int i = 0; i < K; ++i) {
    ad[i] = cfma(sd[i], ps, ad[i]);
    aw[i] = cfma(sww[i], ps, aw[i]);
  }
}

// the pieces up to three factors (the fourth is the centre's)
template <typename T, bool WF = true>
CP_HD void epa_side_grad(const EpaSide<T>& s, EpaGrad<T>& g) {
  g.f = T(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) g.dd[i] = g.dw[i] = T(0);
  if (s.empty) return;
  // neighbour slot i collects the pieces k > i, its factor p_i carrying
  // 3/(4 w_i) and the other started factors 4^-(k-1); the value of piece k
  // carries 4^-k
  T ad[4] = {T(0), T(0), T(0), T(0)}, aw[4] = {T(0), T(0), T(0), T(0)};
  T full = T(0);
  epa_piece_grad<T, 1, 3, false, WF>(s, s.c[0], s.c[1], T(1), T(0.25), full, ad, aw);
  epa_piece_grad<T, 2, 4, true, WF>(s, s.c[1], s.c[2], T(0.25), T(0.0625), full, ad, aw);
  epa_piece_grad<T, 3, 6, false, WF>(s, s.c[2], s.c[3], T(0.0625), T(0.015625), full, ad, aw);
  const T kv = T(0.75) * s.iwv;
  if (WF) g.f = cfma(kv, full, epa_cdf4(s, s.c[0]) * T(0.25));
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const T ki = T(0.75) * s.iw[i] * kv;
    g.dd[i] = ki * ad[i];
    g.dw[i] = ki * aw[i];
  }
  // sorted slots -> neighbour index (the last to start has no piece here)
  unsort4(g.dd, s.sw);
  unsort4(g.dw, s.sw);
}

// The centre's part of the weighted derivatives, g_min dP_min + g_max dP_max
// with respect to d_i and w_i (the minimum's coordinates), and with WF of both
// probabilities.  One leave-one-out sum for both sides: on the maximum's the
// density enters with the opposite sign and F in place of S.  The width sums
// have degree 14: remainder bv^2 prod bu_k^3 (g_min + g_max).
template <typename T, bool WF>
CP_HD void epa_centre_grad(T wv, T iwv, const T (&d)[4], const T (&w)[4], const T (&iw)[4], T gmin, T gmax,
                           T (&cd)[4], T (&cw)[4], T& pmin, T& pmax) {
  EpaCentre<T> c;
  T fs = T(0), ff = T(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) cd[i] = cw[i] = T(0);
  pmin = pmax = T(0);
  if (!epa_centre_setup(c, wv, iwv, d, w, iw)) return;
#pragma unroll
  for (int j = 0; j < 7; ++j) {
    const T x = T(GL<7>::x[j]);
    const T t = cfma(c.bv, x, c.av);
    const T q = T(GL<7>::w[j]) * cfma(-t, t, T(1)), qs = q * gmin, qf = -q * gmax;
    T u[4], p[4], S[4], F[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      u[i] = cfma(c.bu[i], x, c.au[i]);
      const T o = cfma(u[i], u[i], T(-3));
      p[i] = cfma(-u[i], u[i], T(1));
      S[i] = cfma(o, u[i], T(2));
      F[i] = cfma(-o, u[i], T(2));
    }
    const T s01 = S[0] * S[1], s23 = S[2] * S[3], f01 = F[0] * F[1], f23 = F[2] * F[3];
    if (WF) {
      fs = cfma(q * s01, s23, fs);
      ff = cfma(q * f01, f23, ff);
    }
    const T a23 = qs * s23, a01 = qs * s01, b23 = qf * f23, b01 = qf * f01;
    const T lo[4] = {cfma(S[1], a23, F[1] * b23), cfma(S[0], a23, F[0] * b23), cfma(S[3], a01, F[3] * b01),
                     cfma(S[2], a01, F[2] * b01)};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const T lw = p[i] * lo[i];
      cd[i] += lw;
      cw[i] = cfma(lw, u[i], cw[i]);
    }
  }
  T e = T(GLRem<7>::e) * c.bv * c.bv;
#pragma unroll
  for (int i = 0; i < 4; ++i) e *= c.bu[i] * c.bu[i] * c.bu[i];
  const T k = T(0.75) * iwv * c.hl, ew = e * (gmin + gmax);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const T ki = T(0.75 / 64.0) * iw[i] * k;
    cd[i] *= ki;
    cw[i] = ki * (cw[i] + ew);
  }
  if (WF) {
    pmin = T(1.0 / 256.0) * k * (fs - e);
    pmax = T(1.0 / 256.0) * k * (ff - e);
  }
}

}  // namespace cp
