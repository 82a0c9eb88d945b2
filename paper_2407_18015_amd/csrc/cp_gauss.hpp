// cp_gauss.hpp -- independent Gaussian model (the parametric comparison
// model of Sec. 5.2: per-vertex N(mu, sigma^2) from the member mean and
// standard deviation).
//
// The paper notes that the Gaussian has no closed form (Sec. 4.3) and samples
// it by Monte Carlo.  Here the 1-D integrals of Eq. 3 / Eq. 4,
//   P_min = int phi_v S_e S_n S_w S_s,  P_max = int phi_v F_e F_n F_w F_s,
//   t1 = int phi_v S_e F_n S_w F_s,     t2 = int phi_v F_e S_n F_w S_s,
// are evaluated deterministically in one sweep.  Coordinates are in units of
// the vertex: t = (x - mu_v) / sigma_v, so phi_v dt is the standard normal
// and neighbour n enters through z_n = (t - d_n) r_n with
// d_n = (mu_n - mu_v) / sigma_v and r_n = sigma_v / sigma_n.
// The sweep covers t in [-C, C] (the rest of phi weighs 2e-9 for C = 6 and
// 1.3e-17 for C = 8.5).
//
// Nodes.  The integrand is an entire function that decays like a Gaussian, so
// the trapezoidal rule converges exponentially: its error is the integrand's
// Fourier transform at multiples of 2 pi / h, and the transform of a product
// of phi and the four Phi((t - d_n) r_n) (or of phi, a density of one
// neighbour and the other Phi) falls off like exp(-w^2 / (2 V)), V = 1 + sum
// of r_n^2 over the neighbours that vary inside the window.  With
// h = 2 pi / sqrt(2 Lam V) it leaves out at most 2 exp(-Lam) of a probability
// (of the density alone where no neighbour varies in the window, V = 1) and up
// to 2 Lam times that of a derivative's integrand.  Lam = 19.5 in FP32, 7e-9, and
// 37.5 in FP64, 1e-16 and 8e-15: over random stencils, narrow vertices beside
// wide and distant neighbours among them, below the rounding (with 17 and 32,
// 2e-14 and 8e-13 of FP64 probabilities and derivatives were left out).  Five
// equal sigmas take 27 nodes (FP64: 53); fitted fields of 20 members, whose
// sigmas differ by up to a factor of two or three, about 30 to 45.
// A neighbour much narrower than the vertex makes h small everywhere although
// the integrand is steep only near d_n.  There the rule is composite
// Gauss-Legendre instead: the window is cut at d_n + c_k / r_n of every
// neighbour and at c_k of the vertex, c_k running over K fixed multiples of
// the standard deviation in [-C, C] (FP32: 0, +-2, +-4, +-6, six nodes a
// panel; FP64: 0, +-1.5, +-3, +-4.5, +-6, +-8.5, ten nodes), so that a panel
// spans at most ~2 (1.5) deviations of every distribution that varies on it:
// ~1e-8 (~1e-14) absolute for any ratio, with 150 to 200 nodes (400 to 550)
// for overlapping supports.  Each vertex takes the rule with fewer nodes.
// Both kinds run through one node loop, so a wave that holds both pays the
// longer of the two, not their sum.
//
// Bound by vector issue.  A tail is one reciprocal, one exponential and nine
// fused multiply-adds in FP32; in FP64 a ratio of polynomials and the density's
// own exponential: two nodes take about 500 vector instructions (adjoint 550)
// against 753 (983) with the library's erfc and exp.  Measured on a 20-member fit
// of 1024^2, composite rule for every vertex (FP64: with erfc and exp) -> this:
// FP32 classification 543 -> 106 us, adjoint 1145 -> 159 us; FP64 8.4 -> 0.51 and
// 13.6 -> 0.74 ms.  Sigmas drawn over a factor of 300 (most waves then hold
// composite vertices), 512^2: FP32 181 -> 177 and 561 -> 278 us, FP64 2.13 -> 1.13
// and 3.81 -> 1.79 ms.
#pragma once

#include <cmath>

#include "cp_device.hpp"
#include "cp_mc_math.hpp"

namespace cp {

// hc: step of the trapezoidal rule at V = 1, 2 pi / sqrt(2 Lam)
template <typename T>
struct GaussRule;
template <>
struct GaussRule<float> {
  static constexpr int K = 7, N = 6;
  static constexpr float c[7] = {-6.f, -4.f, -2.f, 0.f, 2.f, 4.f, 6.f};
  static constexpr double hc = 1.00612;
};
template <>
struct GaussRule<double> {
  static constexpr int K = 11, N = 10;
  static constexpr double c[11] = {-8.5, -6.0, -4.5, -3.0, -1.5, 0.0, 1.5, 3.0, 4.5, 6.0, 8.5};
  static constexpr double hc = 0.72552;
};

// S = Pr(neighbour above) and F = 1 - S from z's sign and its tail q, by the
// sign's mask (an arithmetic shift and bit selections, which issue at twice the
// rate of a comparison and conditional moves)
template <typename T>
CP_HD void gauss_sides(T z, T q, T& S, T& F) {
  const uint32_t neg = sign_mask(z);
  const T c = T(1) - q;
  S = sel(neg, c, q);
  F = sel(neg, q, c);
}
// normal density factor exp(-t^2 / 2) (scaled after the square, whose rounding
// is then the only one that the exponential of all neighbours' terms inherits)
template <typename T>
CP_HD T gauss_density(T t) {
  return exp2_neg(t * t * T(-kTailScale * kTailScale));
}

// A stencil in vertex units and its rule; P: the type of z_n = (t - d) rs
// (rs = r times the rule's scale).  An absent neighbour has rs = 0, so it sits at its
// median (S = F = 1/2) everywhere and the caller multiplies by 2 for each; its
// d lies outside every window and s = 0 gives it no cuts.
template <typename T, typename P>
struct GaussPlan {
  P d[4], rs[4];
  T s[4];
  T h;          // step of the trapezoidal rule, nodes i h, |i| <= m
  int m;
  bool panels;  // composite rule instead
  // cut ck of neighbour n (any nearby point serves as well: held in T)
  CP_HD T cut(int n, T ck) const { return cfma(ck, s[n], T(d[n])); }
  // x in deviations of neighbour n
  CP_HD T dev(int n, T x) const { return (x - T(d[n])) * T(rs[n]) * T(1.0 / kTailScale); }

  // The smallest cut of neighbour n above x0, C if there is none.  FP32: the
  // cuts lie two deviations apart, so it is found from x0's own deviation, to
  // within one by rounding.
  CP_HD T next_cut(int n, T x0) const {
    using R = GaussRule<T>;
    constexpr T C = R::c[R::K - 1];
    T c = C;
    if constexpr (sizeof(T) == 4) {
      const T k = T(2) * floor(T(0.5) * dev(n, x0)) + T(2);
      const T k1 = tmax(k, -C), c1 = cut(n, k1), k2 = k1 + T(2), c2 = cut(n, k2);
      c = k2 <= C && c2 > x0 ? c2 : c;
      c = k1 <= C && c1 > x0 ? c1 : c;
    } else {
#pragma unroll
      for (int j = R::K - 1; j >= 0; --j) {
        const T v = cut(n, R::c[j]);
        c = v > x0 ? v : c;
      }
    }
    return c;
  }
  // cuts of neighbour n inside the window (FP32: to within one by rounding)
  CP_HD T cuts_inside(int n) const {
    using R = GaussRule<T>;
    constexpr T C = R::c[R::K - 1];
    T v = T(0);
    if constexpr (sizeof(T) == 4) {
      const T hi = floor(T(0.5) * tmin(dev(n, C), C)), lo = ceil(T(0.5) * tmax(dev(n, -C), -C));
      v = tmax(hi - lo + T(1), T(0));
    } else {
#pragma unroll
      for (int j = 0; j < R::K; ++j) v += cut(n, R::c[j]) > -C && cut(n, R::c[j]) < C ? T(1) : T(0);
    }
    return v;
  }
};

// FP32 steps keep 12 significant bits, so the nodes i h are exact
CP_HD float gauss_round_step(float h) {
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, h) & 0xfffff000u);
}
CP_HD double gauss_round_step(double h) { return h; }

template <typename T, typename P>
CP_HD void gauss_plan(GaussPlan<T, P>& g, T mv, T sv, const T (&mn)[4], const T (&sn)[4], const bool (&pres)[4]) {
  using R = GaussRule<T>;
  constexpr int K = R::K, N = R::N;
  constexpr T C = R::c[K - 1];
  const P isv = P(1) / P(sv);
  T V = T(1);
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const P r = pres[n] ? P(sv) / P(sn[n]) : P(0);
    g.d[n] = pres[n] ? (P(mn[n]) - P(mv)) * isv : P(4) * P(C);
    g.s[n] = pres[n] ? T(P(sn[n]) * isv) : T(0);
    g.rs[n] = r * P(kTailScale);
    // constant on the window: no bandwidth
    if (g.cut(n, -C) < C && g.cut(n, C) > -C) V = cfma(T(r), T(r), V);
  }
  g.h = gauss_round_step(T(R::hc) / sqrt(V));
  // nodes of both rules, the composite one's counted only where it can win
  const T nodes = T(2) * C / g.h + T(1);
  g.panels = false;
  if (nodes > T(N * (K - 1))) {
    T cuts = T(K - 1);
#pragma unroll
    for (int n = 0; n < 4; ++n) cuts += g.cuts_inside(n);
    g.panels = !(nodes <= T(N) * cuts);
  }
  // to the node nearest to C, whose cell reaches at least there
  g.m = g.panels ? 0 : (int)(C / g.h + T(0.5));
}

// Visit the nodes of the plan in order: node(position in P, position, weight)
// for each, flush(scale) after at most N of them and at the end: the sums since
// the last one, times a panel's half-length or the step.
template <typename T, typename P, typename Node, typename Flush>
CP_HD void gauss_nodes(const GaussPlan<T, P>& g, Node node, Flush flush) {
  using R = GaussRule<T>;
  constexpr int K = R::K, N = R::N;
  constexpr T C = R::c[K - 1];
  T x0 = -C, x1 = C;
  int i = -g.m;
  for (;;) {
    if (g.panels) {
      // the next cut after x0 (strictly: every panel makes progress)
      x1 = C;
#pragma unroll
      for (int k = 1; k < K - 1; ++k) x1 = T(R::c[k]) > x0 && T(R::c[k]) < x1 ? T(R::c[k]) : x1;
#pragma unroll
      for (int n = 0; n < 4; ++n) x1 = tmin(x1, g.next_cut(n, x0));
    }
    // two nodes at a time: independent work to issue while one waits on its
    // transcendentals.  No more than that: it would cost occupancy.
#pragma unroll 1
    for (int j = 0; j < N; j += 2) {
      if (!g.panels && i > g.m) break;
      P tp[2];
      T t[2], w[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (g.panels) {
          const P hl = (P(x1) - P(x0)) * P(0.5);
          tp[u] = cfma(hl, P(GL<N>::x[j + u]), (P(x0) + P(x1)) * P(0.5));
          t[u] = T(tp[u]);
          w[u] = T(GL<N>::w[j + u]);
        } else {
          t[u] = T(i + u) * g.h;
          tp[u] = P(t[u]);
          w[u] = i + u > g.m ? T(0) : T(1);
        }
      }
      i += 2;
      node(tp[0], t[0], w[0]);
      node(tp[1], t[1], w[1]);
    }
    flush(g.panels ? (P(x1) - P(x0)) * P(0.5) : P(g.h));
    x0 = x1;
    if (g.panels ? !(x1 < C) : i > g.m) break;
  }
}

// out = (P_min, P_max, t1, t2) of a vertex with valid parameters; neighbour
// order e, n, w, s; absent neighbours contribute 1; the saddle terms are 0
// unless all four are present.
template <typename T>
CP_HD void gauss_vertex(T mv, T sv, const T (&mn)[4], const T (&sn)[4], const bool (&pres)[4], T (&out)[4]) {
  GaussPlan<T, T> g;
  gauss_plan(g, mv, sv, mn, sn, pres);
  // sums of N nodes, and of those (one sum of 200 nodes in FP32 reached 9e-7 of
  // the 1e-6 that the probabilities may be off)
  T acc[4] = {T(0), T(0), T(0), T(0)}, sum[4] = {T(0), T(0), T(0), T(0)};
  const T slope = vconst(T(kTailSlope));
  const auto node = [&](T, T t, T w) {
    T S[4], F[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const T z = (t - g.d[n]) * g.rs[n];
      T q, e;
      upper_tail(z, slope, q, e);
      gauss_sides(z, q, S[n], F[n]);
    }
    // e, w (n = 0, 2) take S in t1 and F in t2; n, s the reverse
    const T phi = w * gauss_density(t);
    const T sa = phi * (S[0] * S[2]), fa = phi * (F[0] * F[2]), sb = S[1] * S[3], fb = F[1] * F[3];
    sum[0] = cfma(sa, sb, sum[0]);
    sum[1] = cfma(fa, fb, sum[1]);
    sum[2] = cfma(sa, fb, sum[2]);
    sum[3] = cfma(fa, sb, sum[3]);
  };
  gauss_nodes(g, node, [&](T scale) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc[q] = cfma(sum[q], scale, acc[q]);
      sum[q] = T(0);
    }
  });
  T scale = T(0.39894228040143267794);  // 1 / sqrt(2 pi)
#pragma unroll
  for (int n = 0; n < 4; ++n) scale *= pres[n] ? T(1) : T(2);
  const bool interior = pres[0] && pres[1] && pres[2] && pres[3];
  out[0] = acc[0] * scale;
  out[1] = acc[1] * scale;
  out[2] = interior ? acc[2] * scale : T(0);
  out[3] = interior ? acc[3] * scale : T(0);
}

// Weighted Jacobian of one stencil: jac[2 slot + q] = g_min dP_min/dtheta_q
// + g_max dP_max/dtheta_q, theta = (mu, sigma), slots v, e, n, w, s (absent
// neighbours: 0).  In vertex units, with p_n(x) = phi(z_n) / sigma_n the
// density of neighbour n:
//   dP_min/dmu_n    = int phi(t) p_n prod_{k!=n} S_k dt,
//   dP_min/dsigma_n = int phi(t) p_n z_n prod_{k!=n} S_k dt,
// and for P_max the same with F and the opposite sign (dF = -dS).  The
// vertex slot follows from translation invariance (dP/dmu_v = -sum_n
// dP/dmu_n) and scale invariance about mu_v (sigma_v dP/dsigma_v = -sum_n
// ((mu_n - mu_v) dP/dmu_n + sigma_n dP/dsigma_n)).  Same nodes as
// gauss_vertex; the density of a neighbour is the exponential its tail uses.
//
// Positions (nodes, z_n) in FP64 for both dtypes: in FP32 a panel node's t
// carries half an ulp of |t| <= 6 (2.4e-7), which z_n multiplies by
// sigma_v / sigma_n; the derivative integrands p_n z_n would inherit a
// relative error of that size for narrow neighbours.  The factors (tails,
// densities) and the sums over up to N nodes stay in T, the sums of those in
// FP64: dP/dsigma_n cancels between the nodes below and above the
// neighbour's mean.  The upstream weights enter at every node (g_min times
// the S integrand, -g_max times the F one, one sum per derivative).
template <typename T>
CP_HD void gauss_vertex_jac(T mv, T sv, const T (&mn)[4], const T (&sn)[4], const bool (&pres)[4], T gmin,
                            T gmax, T (&jac)[10]) {
  using P = double;
  GaussPlan<T, P> g;
  gauss_plan(g, mv, sv, mn, sn, pres);
  P a[4] = {P(0), P(0), P(0), P(0)}, b[4] = {P(0), P(0), P(0), P(0)};
  T qa[4] = {T(0), T(0), T(0), T(0)}, qb[4] = {T(0), T(0), T(0), T(0)};
  const T ngmax = -gmax;
  // FP32: z_n as one FP64 FMA (d_n rs_n rounds far below z_n's own FP32)
  const P nd[4] = {-g.d[0] * g.rs[0], -g.d[1] * g.rs[1], -g.d[2] * g.rs[2], -g.d[3] * g.rs[3]};
  const auto node = [&](P tp, T t, T w) {
    const T phi = w * gauss_density(t);
    T S[4], F[4], z[4], e[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      z[n] = sizeof(T) == 4 ? T(cfma(tp, g.rs[n], nd[n])) : T((tp - g.d[n]) * g.rs[n]);
      T q;
      upper_tail(z[n], T(kTailSlope), q, e[n]);
      gauss_sides(z[n], q, S[n], F[n]);
    }
    // the pair products carry the node weight, the vertex density and the
    // upstream weight
    const T pS = phi * gmin, pF = phi * ngmax;
    const T s01 = pS * (S[0] * S[1]), s23 = pS * (S[2] * S[3]), f01 = pF * (F[0] * F[1]), f23 = pF * (F[2] * F[3]);
    const T l[4] = {cfma(S[1], s23, F[1] * f23), cfma(S[0], s23, F[0] * f23), cfma(S[3], s01, F[3] * f01),
                    cfma(S[2], s01, F[2] * f01)};
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const T v = e[n] * l[n];
      qa[n] += v;
      qb[n] = cfma(v, z[n], qb[n]);
    }
  };
  const auto flush = [&](P scale) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      a[n] = cfma(P(qa[n]), scale, a[n]);
      b[n] = cfma(P(qb[n]), scale, b[n]);
      qa[n] = qb[n] = T(0);
    }
  };
  gauss_nodes(g, node, flush);
  // the vertex slot sums terms that cancel (the invariances): in FP64
  P smu = P(0), ssg = P(0), scale = P(0.15915494309189533577);  // 1 / (2 pi)
#pragma unroll
  for (int n = 0; n < 4; ++n) scale *= pres[n] ? P(1) : P(2);
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    jac[2 + 2 * n] = jac[3 + 2 * n] = T(0);
    if (!pres[n]) continue;
    const P c = scale / P(sn[n]);
    const P dmu = c * a[n];  // g-weighted dP/dmu_n
    const P dsg = c / P(kTailScale) * b[n];  // g-weighted dP/dsigma_n
    jac[2 + 2 * n] = T(dmu);
    jac[3 + 2 * n] = T(dsg);
    smu += dmu;
    ssg = cfma(g.d[n], dmu, cfma(P(sn[n]) / P(sv), dsg, ssg));
  }
  jac[0] = T(-smu);
  jac[1] = T(-ssg);
}

}  // namespace cp
