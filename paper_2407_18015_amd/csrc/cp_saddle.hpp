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
// The factors that can vary are evaluated clamped to [0, 1] (a modifier, no
// instruction), the others are 1, so every piece is integrated exactly by the
// rule of its own degree: two to three factors instead of four, and for the
// Epanechnikov model 4, 6, 4, 6, 4 nodes beside the centre instead of 5 x 7.
//
// Measured (all four outputs of a 20-member fit, against five pieces with four
// clamped factors each): 2048^2 in FP32 Epanechnikov 257 -> 129 us, uniform
// 109 -> 56; 1024^2 in FP64 141 -> 66 and 62 -> 32.
#pragma once

#include "cp_device.hpp"
#include "cp_hist.hpp"
#include "cp_tiles.hpp"

namespace cp {

// A factor by its argument: uniform F = (x - x0) i, S = 1 - that with
// (x0, i) = (a, 1/L); Epanechnikov v = (u + 1) / 2 = (x - x0) i with
// (x0, i) = (d - w, 1/(2 w)).  In both F rises from 0 to 1 on v in [0, 1].
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

// Integral over the half-length hl around mid of the vertex kernel (uniform 1,
// Epanechnikov 1 - t^2) times NS survival and NF distribution factors, by the
// N-point rule, REM: plus its remainder.  A factor's argument is clamped on the
// whole piece or nowhere inside it (its clamp points are events), so the
// midpoint decides whether it has a leading term.
template <typename T, int MODEL, int NS, int NF, int N, bool REM>
CP_HD T mixed_piece(const MixedNodes<T>& nodes, T iwv, T l, T r, const Ramp<T> (&s)[NS > 0 ? NS : 1], const Ramp<T> (&f)[NF > 0 ? NF : 1]) {
  const T mid = (l + r) * T(0.5), hl = (r - l) * T(0.5);
  T am[NS + NF], bm[NS + NF];
#pragma unroll
  for (int i = 0; i < NS + NF; ++i) {
    const Ramp<T>& q = i < NS ? s[i < NS ? i : 0] : f[i < NS ? 0 : i - NS];
    am[i] = (mid - q.x0) * q.i;
    bm[i] = hl * q.i;
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
    for (int i = 0; i < NS + NF; ++i) {
      const T v = clamp01(cfma(bm[i], x, am[i]));
      if constexpr (MODEL == CP_UNIFORM) {
        prod *= i < NS ? T(1) - v : v;
      } else {  // F = v^2 (3 - 2 v), halved: its constants are free operands
        const T v2 = v * v, g = T(1.5) - v;
        prod *= i < NS ? cfma(-v2, g, T(0.5)) : v2 * g;
      }
    }
    sum = cfma(T(GL<N>::w[j]), prod, sum);
  }
  if constexpr (REM) {
    // leading coefficients: S -b (uniform) or b^3 (halved), F the negative,
    // the vertex's kernel -bv^2 (Epanechnikov)
    T c = MODEL == CP_UNIFORM ? T(1) : -bv * bv;
#pragma unroll
    for (int i = 0; i < NS + NF; ++i) {
      const T b = MODEL == CP_UNIFORM ? -bm[i] : bm[i] * bm[i] * bm[i];
      const T m = fabs(am[i] - T(0.5)) < T(0.5) ? b : T(0);
      c *= i < NS ? m : -m;
    }
    sum = cfma(T(GLRem<N>::e), c, sum);
  }
  return sum * (MODEL == CP_UNIFORM ? hl : T(1 << (NS + NF)) * hl);
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
  const Ramp<T> first[1] = {sel(less_mask(ss[1], ss[0]), s[1], s[0])};
  const Ramp<T> last[1] = {sel(less_mask(fe[0], fe[1]), f[1], f[0])};
  const T sa = fmin_nn(s0, s1), sb = fmax_nn(s0, s1), fa = fmin_nn(f0, f1), fb = fmax_nn(f0, f1);
  const T p = fmax_nn(sa, fa), q = fmin_nn(sb, fb);
  const T c0 = fmin_nn(sa, fa), c1 = fmin_nn(p, q), c2 = fmax_nn(p, q), c3 = fmax_nn(sb, fb);
  const Ramp<T> none[1] = {first[0]};
  T acc = mixed_piece<T, MODEL, 0, 2, U ? 1 : 4, true>(nodes, iwv, lo, c0, none, f);
  acc += mixed_piece<T, MODEL, 1, 2, U ? 2 : 6, false>(nodes, iwv, c0, c1, first, f);
  if (!centre) acc += mixed_piece<T, MODEL, 1, 1, U ? 1 : 4, true>(nodes, iwv, c1, c2, first, last);
  acc += mixed_piece<T, MODEL, 2, 1, U ? 2 : 6, false>(nodes, iwv, c2, c3, s, last);
  acc += mixed_piece<T, MODEL, 2, 0, U ? 1 : 4, true>(nodes, iwv, c3, hi, s, none);
  return acc;
}

// P_min, P_max (MM) and the saddle terms (of a vertex with all neighbours) of
// a valid stencil.
template <typename T, int MODEL, bool MM>
CP_HD void vertex_classes_ue(T p0, T p1, const T (&q0)[4], const T (&q1)[4], const bool (&pres)[4], T& pmin, T& pmax,
                             T& t1, T& t2) {
  Ramp<T> r[4];
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
      r[i] = {s.a[i], s.iL[i]};
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
      r[i] = {st[i], T(0.5) * s.iw[i]};
    }
  }
  t1 = t2 = T(0);
  if (!(pres[0] && pres[1] && pres[2] && pres[3])) return;
  const MixedNodes<T> nodes;
  const Ramp<T> ew[2] = {r[0], r[2]}, ns[2] = {r[1], r[3]};
  const T ews[2] = {st[0], st[2]}, ewe[2] = {en[0], en[2]}, nss[2] = {st[1], st[3]}, nse[2] = {en[1], en[3]};
  t1 = cfma(k, saddle_term<T, MODEL>(nodes, iwv, v0, v1, ew, ews, ewe, ns, nss, nse, centre), o[2]);
  t2 = cfma(k, saddle_term<T, MODEL>(nodes, iwv, v0, v1, ns, nss, nse, ew, ews, ewe, centre), o[3]);
}

}  // namespace cp
