// cp_saddle.hpp -- saddle probability on the 4-neighbour stencil (Eq. 2 in
// 1-D, Eq. 4 in 2-D).  Under independence (Sec. 3)
//   t1 = Pr[v < e, v > n, v < w, v > s] = int pdf_v S_e F_n S_w F_s dx
//   t2 = Pr[v > e, v < n, v > w, v < s] = int pdf_v F_e S_n F_w S_s dx
// and P_saddle = t1 + t2 (interior vertices; the alternating pattern needs
// all four neighbours).  Task 1 for a saddle term (Sec. 4.1.3): the range is
// [lo, hi] = [max(a_v, a of the F factors), min(b_v, b of the S factors)], cut
// at its events, the start points of the S factors and the end points of the F
// factors.  Sorted, they make five pieces, and which factors can vary on a
// piece follows from its place:
//   1st: both F (no S has started);
//   2nd: both F and the S that starts first;
//   3rd: all four, if both S started first: this is the centre, shared with
//        P_min and P_max (uni_centre); otherwise at most the S that starts
//        first and the F that ends last;
//   4th: both S and the F that ends last;
//   5th: both S (every F has ended).
// The factors that can vary are evaluated with their arguments clamped, the
// others are 1, so every piece is integrated exactly by the
// rule of its own degree: two to three factors instead of four, and for the
// Epanechnikov model 4, 6, 4, 6, 4 nodes beside the centre instead of 5 x 7.
//
// Measured (all four outputs of a 20-member fit, against five pieces with four
// clamped factors each): 2048^2 in FP32 Epanechnikov 273 -> 137 us, uniform
// 117 -> 60; 1024^2 in FP64 165 -> 77 and 70 -> 35.
#pragma once

#include "cp_device.hpp"
#include "cp_hist.hpp"
#include "cp_tiles.hpp"

namespace cp {

// A factor of a term by its argument v = (x - x0) i.  Uniform: v clamped to
// [0, 1], for S (x0, i) = (b, -1/L), for F (a, 1/L).  Epanechnikov: (v^3 - 3 v +
// 2) / 4 of v clamped to [-1, 1], for S (d, 1/w), for F (d, -1/w).  The origins
// are the parameters' own differences: a start point d - w rounds, which every
// factor of the pieces beside it would inherit.
template <typename T>
struct Ramp {
  T x0, i;
};
template <typename T>
CP_HD Ramp<T> sel(uint32_t m, const Ramp<T>& a, const Ramp<T>& b) {
  return {sel(m, a.x0, b.x0), sel(m, a.i, b.i)};
}

// The positive nodes of the rules below; the others are their negatives.
template <typename T>
struct MixedNodes {
  T n2[1], n4[2], n6[3];
  CP_HD MixedNodes()
      : n2{vconst(T(GL<2>::x[1]))}, n4{vconst(T(GL<4>::x[2])), vconst(T(GL<4>::x[3]))},
        n6{vconst(T(GL<6>::x[3])), vconst(T(GL<6>::x[4])), vconst(T(GL<6>::x[5]))} {}
  template <int N>
  CP_HD T at(int j) const {
    const int k = j < N / 2 ? N / 2 - 1 - j : j - N / 2;
    const T x = N == 1 ? T(0) : N == 2 ? n2[0] : N == 4 ? n4[k < 2 ? k : 0] : n6[k < 3 ? k : 0];
    return j < N / 2 ? -x : x;
  }
};

// acc plus the integral over [l, r] of the vertex kernel (uniform 1,
// Epanechnikov 1 - t^2) times K factors, by the N-point rule, REM: plus its
// remainder.  A factor's argument is clamped on the whole piece or nowhere
// inside it (its clamp points are events), so the midpoint decides whether it
// has a leading term.
//
// Epanechnikov: the Horner form of v^3 - 3 v + 2 with a clamp of its own (a half
// rate instruction).  From t = (v + 1) / 2, whose clamp is a modifier, as 1/2 -
// t^2 (3/2 - t), the terms' error is a quarter to a third larger (rms 6.1e-9
// against 4.8e-9 in FP32, widths within a factor of four).
template <typename T, int MODEL, int K, int N, bool REM>
CP_HD T mixed_piece(const MixedNodes<T>& nodes, T iwv, T l, T r, const Ramp<T> (&f)[K], T acc) {
  const T mid = (l + r) * T(0.5), hl = (r - l) * T(0.5);
  T am[K], bm[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    am[i] = (mid - f[i].x0) * f[i].i;
    bm[i] = hl * f[i].i;
  }
  const T av = mid * iwv, bv = hl * iwv;
  T sum = T(0);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const T x = nodes.template at<N>(j);
    T prod;
    if constexpr (MODEL == CP_UNIFORM) {
      prod = T(1);
    } else {
      const T t = cfma(bv, x, av);
      prod = cfma(-t, t, T(1));
    }
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const T v = cfma(bm[i], x, am[i]);
      prod *= MODEL == CP_UNIFORM ? clamp01(v) : epa_s4(clamp_nn(v, T(-1), T(1)));
    }
    sum = cfma(T(GL<N>::w[j]), prod, sum);
  }
  if constexpr (REM) {
    // leading coefficients: b (uniform), b^3, the vertex's kernel -bv^2
    T c = MODEL == CP_UNIFORM ? T(1) : -bv * bv;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const bool in = MODEL == CP_UNIFORM ? fabs(am[i] - T(0.5)) < T(0.5) : fabs(am[i]) < T(1);
      c *= in ? (MODEL == CP_UNIFORM ? bm[i] : bm[i] * bm[i] * bm[i]) : T(0);
    }
    sum = cfma(T(GLRem<N>::e), c, sum);
  }
  return cfma(sum, MODEL == CP_UNIFORM ? hl : T(1.0 / (1 << 2 * K)) * hl, acc);
}

// One saddle term without the centre, times the vertex's width (uniform Lv,
// Epanechnikov 4 wv / 3): [v0, v1] the vertex's range, S factors s (ends se),
// F factors f (ends fe).
template <typename T, int MODEL>
CP_HD T saddle_term(const MixedNodes<T>& nodes, T iwv, T v0, T v1, const Ramp<T> (&s)[2], const T (&ss)[2], const T (&se)[2],
                    const Ramp<T> (&f)[2], const T (&fs)[2], const T (&fe)[2], bool centre) {
  constexpr bool U = MODEL == CP_UNIFORM;
  const T lo = fmax_nn(v0, fmax_nn(fs[0], fs[1])), hi = fmin_nn(v1, fmin_nn(se[0], se[1]));
  if (!(lo < hi)) return T(0);
  const T s0 = clamp_nn(ss[0], lo, hi), s1 = clamp_nn(ss[1], lo, hi);
  const T f0 = clamp_nn(fe[0], lo, hi), f1 = clamp_nn(fe[1], lo, hi);
  const Ramp<T> first = sel(less_mask(ss[1], ss[0]), s[1], s[0]);
  const Ramp<T> last = sel(less_mask(fe[0], fe[1]), f[1], f[0]);
  const T sa = fmin_nn(s0, s1), sb = fmax_nn(s0, s1), fa = fmin_nn(f0, f1), fb = fmax_nn(f0, f1);
  const T p = fmax_nn(sa, fa), q = fmin_nn(sb, fb);
  const T c0 = fmin_nn(sa, fa), c1 = fmin_nn(p, q), c2 = fmax_nn(p, q), c3 = fmax_nn(sb, fb);
  const Ramp<T> sff[3] = {first, f[0], f[1]}, sf[2] = {first, last}, ssf[3] = {s[0], s[1], last};
  T acc = mixed_piece<T, MODEL, 2, U ? 1 : 4, true>(nodes, iwv, lo, c0, f, T(0));
  acc = mixed_piece<T, MODEL, 3, U ? 2 : 6, false>(nodes, iwv, c0, c1, sff, acc);
  if (!centre) acc = mixed_piece<T, MODEL, 2, U ? 1 : 4, true>(nodes, iwv, c1, c2, sf, acc);
  acc = mixed_piece<T, MODEL, 3, U ? 2 : 6, false>(nodes, iwv, c2, c3, ssf, acc);
  acc = mixed_piece<T, MODEL, 2, U ? 1 : 4, true>(nodes, iwv, c3, hi, s, acc);
  return acc;
}

// P_min, P_max (MM) and the saddle terms (of a vertex with all neighbours) of
// a valid stencil.
template <typename T, int MODEL, bool MM>
CP_HD void vertex_classes_ue(T p0, T p1, const T (&q0)[4], const T (&q1)[4], const bool (&pres)[4], T& pmin, T& pmax,
                             T& t1, T& t2) {
  Ramp<T> S[4], F[4];
  T st[4], en[4], o[4], v0, v1, k, iwv;
  bool centre;
  if constexpr (MODEL == CP_UNIFORM) {
    UniStencil<T> s;
    uni_stencil(s, p0, p1, q0, q1, pres);
    centre = uni_centre<T, true>(s.Lv, s.iLv, s.a, s.b, s.iL, o);
    if (MM) {
      UniSide<T> side;
      uni_min_side(side, s);
      pmin = o[0] + uni_side_value(side);
      uni_max_side(side, s, p1, q0, q1, pres);
      pmax = o[1] + uni_side_value(side);
    }
    v0 = T(0);
    v1 = s.Lv;
    k = iwv = s.iLv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      S[i] = {s.b[i], -s.iL[i]};
      F[i] = {s.a[i], s.iL[i]};
      st[i] = s.a[i];
      en[i] = s.b[i];
    }
  } else {
    EpaStencil<T> s;
    epa_stencil(s, p0, p1, q0, q1, pres);
    centre = epa_centre<T, true>(s.wv, s.iwv, s.d, s.w, s.iw, o);
    if (MM) {
      EpaSide<T> side;
      epa_min_side(side, s);
      pmin = o[0] + epa_side_value(side);
      epa_max_side(side, s, pres);
      pmax = o[1] + epa_side_value(side);
    }
    v0 = -s.wv;
    v1 = s.wv;
    iwv = s.iwv;
    k = T(0.75) * s.iwv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      st[i] = s.d[i] - s.w[i];
      en[i] = s.d[i] + s.w[i];
      S[i] = {s.d[i], s.iw[i]};
      F[i] = {s.d[i], -s.iw[i]};
    }
  }
  t1 = t2 = T(0);
  if (!(pres[0] && pres[1] && pres[2] && pres[3])) return;
  const MixedNodes<T> nodes;
  const Ramp<T> ewS[2] = {S[0], S[2]}, ewF[2] = {F[0], F[2]}, nsS[2] = {S[1], S[3]}, nsF[2] = {F[1], F[3]};
  const T ews[2] = {st[0], st[2]}, ewe[2] = {en[0], en[2]}, nss[2] = {st[1], st[3]}, nse[2] = {en[1], en[3]};
  t1 = cfma(k, saddle_term<T, MODEL>(nodes, iwv, v0, v1, ewS, ews, ewe, nsF, nss, nse, centre), o[2]);
  t2 = cfma(k, saddle_term<T, MODEL>(nodes, iwv, v0, v1, nsS, nss, nse, ewF, ews, ewe, centre), o[3]);
}

}  // namespace cp
