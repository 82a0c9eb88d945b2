// host_accuracy.cpp -- host-only build of the library's per-vertex routines for
// measurements of their rounding (test infrastructure; built by
// tests/test_host_accuracy.py with the HIP compiler's host pass only).
//
//   host_accuracy gauss <dtype> <in> <out>
//     in:  FP64 records: (mean, sigma) of v, e, n, w, s, then g_min, g_max
//     out: FP64 records: P_min, P_max, t1, t2 and the ten entries of the
//          weighted Jacobian by gauss_vertex and gauss_vertex_jac, then the same
//          fourteen in long double by 20-point panels of half a deviation of
//          every distribution.
//   host_accuracy tail <in> <out>
//     in:  FP64 z; out: FP64 relative error of upper_tail's FP64 tail at z.
//   host_accuracy epa <dtype> <in> <out>
//     in:  FP64 records: (centre, half-width) of v, e, n, w, s
//     out: FP64 records: t1, t2 by vertex_classes_ue, by five pieces of four
//          clamped cubic factors each in the same type, and by those in long
//          double.
//   host_accuracy hist <dtype> <nbins> <in> <out>
//     in:  FP64 records: lo, hi, masses of v, e, n, w, s
//     out: FP64 records: P_min, P_max by hist_vertex_minmax, by the end values
//          of every merged interval in Bernstein form in the same type, and by
//          those in long double.
//   dtype: 0 FP32, 1 FP64.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "cp_gauss.hpp"
#include "cp_hist.hpp"
#include "cp_internal.hpp"
#include "cp_saddle.hpp"
#include "cp_tiles.hpp"

namespace {

using Real = long double;
const Real kPi = acosl(-1.0L);

// n-point Gauss-Legendre rule
void legendre(int n, std::vector<Real>& x, std::vector<Real>& w) {
  x.resize(n);
  w.resize(n);
  for (int i = 0; i < n; ++i) {
    Real t = cosl(kPi * (i + 0.75L) / (n + 0.5L)), d = 0;
    for (int it = 0; it < 20; ++it) {
      Real a = 1, b = t;
      for (int k = 2; k <= n; ++k) {
        const Real c = ((2 * k - 1) * t * b - (k - 1) * a) / k;
        a = b;
        b = c;
      }
      d = n * (t * b - a) / (t * t - 1);
      t -= b / d;
    }
    x[i] = t;
    w[i] = 2 / ((1 - t * t) * d * d);
  }
}

// ---------------------------------------------------------------------------
// Gaussian
// ---------------------------------------------------------------------------
void gauss_exact(const double* p, double* out) {
  static std::vector<Real> X, W;
  if (X.empty()) legendre(20, X, W);
  const Real sv = p[1], C = 12 * sv, rs2 = 1 / sqrtl(2.0L), nrm = 1 / sqrtl(2 * kPi);
  Real m[4], s[4], o[4] = {0, 0, 0, 0}, dm[4] = {0, 0, 0, 0}, ds[4] = {0, 0, 0, 0};
  std::vector<Real> e;
  for (int i = 0; i < 4; ++i) {
    m[i] = (Real)p[2 + 2 * i] - p[0];
    s[i] = p[3 + 2 * i];
  }
  for (int k = -24; k <= 24; ++k) {
    e.push_back(k * 0.5L * sv);
    for (int i = 0; i < 4; ++i)
      if (fabsl(m[i] + k * 0.5L * s[i]) < C) e.push_back(m[i] + k * 0.5L * s[i]);
  }
  std::sort(e.begin(), e.end());
  for (size_t q = 0; q + 1 < e.size(); ++q) {
    const Real mid = (e[q] + e[q + 1]) / 2, hl = (e[q + 1] - e[q]) / 2;
    if (!(hl > 0)) continue;
    for (size_t j = 0; j < X.size(); ++j) {
      const Real t = mid + hl * X[j], w = W[j] * hl * expl(-t * t / (2 * sv * sv)) * nrm / sv;
      Real S[4], F[4], z[4];
      for (int i = 0; i < 4; ++i) {
        z[i] = (t - m[i]) / s[i];
        S[i] = 0.5L * erfcl(z[i] * rs2);
        F[i] = 0.5L * erfcl(-z[i] * rs2);
      }
      o[0] += w * S[0] * S[1] * S[2] * S[3];
      o[1] += w * F[0] * F[1] * F[2] * F[3];
      o[2] += w * S[0] * F[1] * S[2] * F[3];
      o[3] += w * F[0] * S[1] * F[2] * S[3];
      for (int i = 0; i < 4; ++i) {
        Real a = 1, b = 1;
        for (int k = 0; k < 4; ++k)
          if (k != i) {
            a *= S[k];
            b *= F[k];
          }
        const Real l = w * expl(-z[i] * z[i] / 2) * nrm / s[i] * ((Real)p[10] * a - (Real)p[11] * b);
        dm[i] += l;
        ds[i] += l * z[i];
      }
    }
  }
  Real smu = 0, ssg = 0;
  for (int i = 0; i < 4; ++i) {
    out[i] = (double)o[i];
    out[6 + 2 * i] = (double)dm[i];
    out[7 + 2 * i] = (double)ds[i];
    smu += dm[i];
    ssg += m[i] * dm[i] + s[i] * ds[i];
  }
  out[4] = (double)-smu;
  out[5] = (double)(-ssg / sv);
}

template <typename T>
void gauss(const double* p, double* out) {
  T m[4], s[4], o[4], j[10];
  const bool pres[4] = {true, true, true, true};
  for (int i = 0; i < 4; ++i) {
    m[i] = (T)p[2 + 2 * i];
    s[i] = (T)p[3 + 2 * i];
  }
  cp::gauss_vertex<T>((T)p[0], (T)p[1], m, s, pres, o);
  cp::gauss_vertex_jac<T>((T)p[0], (T)p[1], m, s, pres, (T)p[10], (T)p[11], j);
  for (int i = 0; i < 4; ++i) out[i] = (double)o[i];
  for (int i = 0; i < 10; ++i) out[4 + i] = (double)j[i];
  gauss_exact(p, out + 14);
}

double tail_error(double z) {
  double q, e;
  cp::upper_tail(z * cp::kTailScale, cp::kTailSlope, q, e);
  return (double)(q / (0.5L * erfcl(fabsl((Real)z) / sqrtl(2.0L))) - 1);
}

// ---------------------------------------------------------------------------
// Epanechnikov saddle terms: five pieces, all four factors clamped on each
// ---------------------------------------------------------------------------
template <typename T>
T epa_term_plain(int term, const double* p) {
  static std::vector<Real> X, W;
  if (X.empty()) legendre(8, X, W);
  const T wv = (T)p[1];
  T d[4], w[4], lo = -wv, hi = wv;
  bool F[4];
  for (int i = 0; i < 4; ++i) {
    d[i] = (T)p[2 + 2 * i] - (T)p[0];
    w[i] = (T)p[3 + 2 * i];
    F[i] = (i & 1) == (term == 0);
    if (F[i])
      lo = std::max(lo, (T)(d[i] - w[i]));
    else
      hi = std::min(hi, (T)(d[i] + w[i]));
  }
  if (!(lo < hi)) return 0;
  T e[6] = {lo, 0, 0, 0, 0, hi};
  for (int i = 0; i < 4; ++i) e[1 + i] = std::min(std::max((T)(F[i] ? d[i] + w[i] : d[i] - w[i]), lo), hi);
  std::sort(e + 1, e + 5);
  T acc = 0;
  for (int k = 0; k < 5; ++k) {
    const T mid = (e[k] + e[k + 1]) / 2, hl = (e[k + 1] - e[k]) / 2;
    T sum = 0;
    for (size_t j = 0; j < X.size(); ++j) {
      const T x = mid + hl * (T)X[j], t = x / wv;
      T prod = 1 - t * t;
      for (int i = 0; i < 4; ++i) {
        const T u = std::min(std::max((F[i] ? d[i] - x : x - d[i]) / w[i], (T)-1), (T)1);
        prod *= (u * u - 3) * u + 2;
      }
      sum += (T)W[j] * prod;
    }
    acc += sum * hl;
  }
  return acc * (T)0.75 / wv / 256;
}

template <typename T>
void epa(const double* p, double* out) {
  T q0[4], q1[4], a, b, t1, t2;
  const bool pres[4] = {true, true, true, true};
  for (int i = 0; i < 4; ++i) {
    q0[i] = (T)p[2 + 2 * i];
    q1[i] = (T)p[3 + 2 * i];
  }
  cp::vertex_classes_ue<T, CP_EPANECHNIKOV, true>((T)p[0], (T)p[1], q0, q1, pres, a, b, t1, t2);
  out[0] = (double)t1;
  out[1] = (double)t2;
  for (int k = 0; k < 2; ++k) {
    out[2 + k] = (double)epa_term_plain<T>(k, p);
    out[4 + k] = (double)epa_term_plain<Real>(k, p);
  }
}

// ---------------------------------------------------------------------------
// histogram probabilities: all merged intervals, end values, one running sum
// ---------------------------------------------------------------------------
template <typename T>
void hist_plain(int h, const double* p, double* out) {
  const int np = 2 + h;
  const T lov = (T)p[0], hv = (T)p[1] - lov;
  struct Hist {
    std::vector<T> U, e;  // survival at and position of the edges
  } q[5];
  for (int v = 0; v < 5; ++v) {
    const double* r = p + v * np;
    const T lo = (T)r[0] - lov, hi = (T)r[1] - lov, d = (hi - lo) / h;
    q[v].U.assign(h + 1, 0);
    q[v].e.assign(h + 1, lo);
    for (int k = h - 1; k >= 0; --k) q[v].U[k] = q[v].U[k + 1] + (T)r[2 + k];
    for (int k = 1; k <= h; ++k) q[v].e[k] = hi - (h - k) * d;
  }
  std::vector<T> x{0, hv};
  for (int v = 0; v < 5; ++v)
    for (const T e : q[v].e)
      if (e > 0 && e < hv) x.push_back(e);
  std::sort(x.begin(), x.end());
  // survival at x on the bin that holds c
  const auto S = [&](const Hist& s, T c, T at) -> T {
    if (!(c > s.e[0])) return s.U[0];
    for (int k = 0; k < h; ++k)
      if (c < s.e[k + 1]) {
        const T slope = (s.U[k] - s.U[k + 1]) * ((T)h / (s.e[h] - s.e[0]));
        return s.U[k + 1] + slope * (s.e[k + 1] - at);
      }
    return 0;
  };
  T amin = 0, amax = 0;
  for (size_t k = 0; k + 1 < x.size(); ++k) {
    const T mid = (x[k] + x[k + 1]) / 2;
    T pv = 0;
    for (int j = 0; j < h; ++j)
      if (mid < q[0].e[j + 1]) {
        pv = (q[0].U[j] - q[0].U[j + 1]) * ((T)h / hv);
        break;
      }
    T s[2][5] = {{1, 0, 0, 0, 0}, {1, 0, 0, 0, 0}};  // Bernstein coefficients, unscaled, of both products
    for (int i = 0; i < 4; ++i) {
      const T s0 = S(q[1 + i], mid, x[k]), s1 = S(q[1 + i], mid, x[k + 1]), tot = q[1 + i].U[0];
      for (int f = 0; f < 2; ++f) {
        const T a = f ? tot - s0 : s0, b = f ? tot - s1 : s1;
        for (int m = i + 1; m >= 0; --m) s[f][m] = (m <= i ? s[f][m] * a : 0) + (m > 0 ? s[f][m - 1] * b : 0);
      }
    }
    const T wgt = pv * (x[k + 1] - x[k]);
    for (int f = 0; f < 2; ++f)
      (f ? amax : amin) += wgt * ((s[f][0] + s[f][4]) / 5 + (s[f][1] + s[f][3]) / 20 + s[f][2] / 30);
  }
  out[0] = (double)amin;
  out[1] = (double)amax;
}

template <typename T>
void hist(int h, const double* p, double* out) {
  const int np = 2 + h;
  std::vector<T> L((size_t)(3 + h) * 5, T(0));
  for (int k = 0; k < np; ++k)
    for (int v = 0; v < 5; ++v) L[k * 5 + v] = (T)p[v * np + k];
  cp::hist_stage_validity<T, 1>(L.data(), 5, h, 0);
  cp::hist_stage_suffix<T, 1>(L.data(), 5, h, 0);
  const cp::HistSuf<T> U{L.data(), 5, h};
  const int en[4] = {1, 2, 3, 4};
  const bool pres[4] = {true, true, true, true};
  T lo[4], hi[4], pmin, pmax;
  for (int i = 0; i < 4; ++i) {
    lo[i] = L[1 + i] - L[0];
    hi[i] = L[6 + i] - L[0];
  }
  cp::hist_vertex_minmax(U, 0, en, pres, L[5] - L[0], lo, hi, pmin, pmax);
  out[0] = (double)pmin;
  out[1] = (double)pmax;
  hist_plain<T>(h, p, out + 2);
  hist_plain<Real>(h, p, out + 4);
}

template <typename Fn>
int records(const char* in, const char* outp, size_t ni, size_t no, Fn fn) {
  FILE* f = std::fopen(in, "rb");
  if (!f) return 2;
  std::vector<double> rec(ni), out(no), all;
  while (std::fread(rec.data(), sizeof(double), ni, f) == ni) {
    fn(rec.data(), out.data());
    all.insert(all.end(), out.begin(), out.end());
  }
  std::fclose(f);
  f = std::fopen(outp, "wb");
  if (!f) return 2;
  std::fwrite(all.data(), sizeof(double), all.size(), f);
  std::fclose(f);
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc == 5 && !std::strcmp(argv[1], "gauss"))
    return records(argv[3], argv[4], 12, 28, std::atoi(argv[2]) ? gauss<double> : gauss<float>);
  if (argc == 4 && !std::strcmp(argv[1], "tail"))
    return records(argv[2], argv[3], 1, 1, [](const double* p, double* o) { *o = tail_error(*p); });
  if (argc == 5 && !std::strcmp(argv[1], "epa"))
    return records(argv[3], argv[4], 10, 6, std::atoi(argv[2]) ? epa<double> : epa<float>);
  if (argc == 6 && !std::strcmp(argv[1], "hist")) {
    const int dt = std::atoi(argv[2]), h = std::atoi(argv[3]);
    return records(argv[4], argv[5], 5 * (2 + h), 6,
                   [=](const double* p, double* o) { dt ? hist<double>(h, p, o) : hist<float>(h, p, o); });
  }
  std::fprintf(stderr, "usage: see the head of this file\n");
  return 2;
}
