// cp_hist.hpp -- histogram model (Sec. 4.4.1): per-vertex sweep over the
// merged bin edges of the five stencil histograms.
//
// A histogram is a mixture of non-overlapping uniform kernels, so on every
// interval between consecutive edges of the five histograms the vertex pdf
// is constant and each neighbour's survival function is linear.  Eq. 5 sums
// the uniform-model probability over all h^5 kernel combinations; expanding
// that sum by linearity gives the same number as integrating
// pdf_v * prod S_n once over the merged edges, which costs O(5h) instead of
// O(h^5).  On each interval the product of four linear factors is integrated
// exactly, from the factors at the midpoint and their half-changes.
//
// Staged per vertex in LDS (planes of the extended tile, E vertices each):
//   0 lo, 1 hi, 2..h+1 masses, h+2 zero.  An invalid histogram (lo >= hi,
// non-finite, negative mass) is marked by lo = NaN while staging.  The
// sweeps then replace the masses by their suffix sums U_j = m_j + ... +
// m_{h-1} (FP64 sums rounded once; U_h = 0 is the zero plane), so the
// survival at an edge is one read.
#pragma once

#include "cp_device.hpp"

namespace cp {

// staged planes per vertex: lo, hi, h masses (then suffix sums), one zero plane
__host__ __device__ constexpr int hist_planes(int h) { return h + 3; }

template <typename T>
struct HistLds {
  const T* base;
  int E;  // vertices per plane (extended tile)
  int h;
  T ih;   // 1 / h
  // mass j of vertex e; `rev` reads the histogram of -X (bins reversed)
  CP_HD T mass(int e, int j, bool rev) const {
    const int p = rev ? (1 + h - j) : (2 + j);
    return base[p * E + e];
  }
  CP_HD bool valid(int e) const { return base[e] == base[e]; }
};

// Compute a here: without it the compiler moves an interval's integrals behind
// the cursor steps and copies the state they need (24 moves an interval).
template <typename T>
CP_HD void settle(T& a) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(a));
#endif
}

// Validity marking of every staged histogram (lo := NaN when invalid).
template <typename T, int NT>
CP_HD void hist_stage_validity(T* lds, int E, int h, int tid) {
  for (int e = tid; e < E; e += NT) {
    const T lo = lds[e], hi = lds[E + e];
    const T d = hi - lo;
    bool ok = d > T(0) && d < T(3.0e38) && (lo - lo) == T(0);
    for (int j = 0; j < h; ++j) {
      const T m = lds[(2 + j) * E + e];
      ok = ok && m >= T(0) && m < T(3.0e38);
    }
    if (!ok) lds[e] = __builtin_nan("");
  }
}

}  // namespace cp

// ---------------------------------------------------------------------------
// Forward in one sweep: P_min and P_max of a vertex share the merged edges
// of the five histograms over the vertex range [0, hv], with F = T - S for
// every neighbour.  The staged masses are first replaced, per staged vertex,
// by their suffix sums U_j = m_j + ... + m_{h-1} (FP64 sums rounded once), so
// a neighbour's survival at an edge is one LDS read and crossing an edge
// costs one read, whatever the number of bins.
// ---------------------------------------------------------------------------
namespace cp {

// masses (planes 2..h+1) -> suffix sums U_0 .. U_{h-1}; U_0 = total mass;
// plane h+2 := 0 (U_h)
template <typename T, int NT>
CP_HD void hist_stage_suffix(T* lds, int E, int h, int tid) {
  for (int e = tid; e < E; e += NT) {
    double acc = 0.0;
    for (int j = h - 1; j >= 0; --j) {
      acc += (double)lds[(2 + j) * E + e];
      lds[(2 + j) * E + e] = (T)acc;
    }
    lds[(2 + h) * E + e] = T(0);
  }
}

template <typename T>
struct HistSuf {
  const T* base;
  int E, h;
  // U_j of vertex e, 0 <= j <= h (plane 2 + h is the staged zero plane, U_h)
  CP_HD T U(int e, int j) const { return base[(2 + j) * E + e]; }
};

// One neighbour in the vertex frame: survival S(x) = snx + slope (nxt - x)
// on the current bin; F = tot - S.  Its edges above the first are counted
// down from the last, hi + k Delta with k = -(h - 1) .. 0 (k = 0: hi itself),
// so the cursor keeps hi and not lo, and its edge index is the float k: the
// next edge is one addition and one fused multiply-add, which issue in half
// the cycles of an integer's conversion.  p points to the suffix sum at the
// next edge and moves by one plane a step.
template <typename T>
struct SufCursor {
  const T* p;
  T k;  // next edge (-h: the first, lo); above 0: past the range
  T hi, d, id, nxt, snx, slope, tot;
};

template <typename T>
CP_HD void suf_cursor_init(SufCursor<T>& c, const HistSuf<T>& L, int e, T lo, T hi, bool present, T big) {
  const int h = L.h;
  const T* U0 = L.base + 2 * L.E + e;
  c.hi = hi;
  c.d = (hi - lo) * (T(1) / T(h));
  c.id = T(h) * crcp(hi - lo);
  // past the range, at the zero plane
  c.p = U0 + h * L.E;
  c.k = T(1);
  c.nxt = big;
  c.slope = T(0);
  if (!present) {  // constant factor 1 in both products
    c.snx = T(1);
    c.tot = T(2);
    return;
  }
  c.tot = *U0;
  c.snx = T(0);
  if (!(lo < T(0))) {  // range starts at or after x = 0
    c.p = U0;
    c.k = T(-h);
    c.nxt = lo;
    c.snx = c.tot;
    return;
  }
  if (!(hi > T(0))) return;  // the whole range lies below x = 0
  int j = (int)(-lo * c.id);
  j = j < 0 ? 0 : (j > h - 1 ? h - 1 : j);
  const auto edge = [&](int k) { return cfma(T(k - h), c.d, hi); };  // 1 <= k <= h
  if (j + 1 < h && !(edge(j + 1) > T(0))) ++j;
  if (j > 0 && edge(j) > T(0)) --j;
  c.k = T(j + 1 - h);
  c.nxt = edge(j + 1);
  c.p = U0 + (j + 1) * L.E;
  c.snx = *c.p;
  c.slope = (U0[j * L.E] - c.snx) * c.id;
}

// Cross the next edge (the callers' one branch; past the range the cursor stays
// at the zero plane, so survival and slope become 0 by themselves).
template <typename T>
CP_HD void suf_cursor_step(SufCursor<T>& c, int E, T big) {
  c.k += T(1);
  const bool past = c.k > T(0);
  c.p += past ? 0 : E;
  const T u = *c.p;
  c.slope = (c.snx - u) * c.id;
  c.snx = u;
  c.nxt = past ? big : cfma(c.k, c.d, c.hi);
}

// The vertex's own bins over [0, hv]: the upper edge nv = k dv of the current
// bin (k = 1 .. h; hv itself for the last: counted up, as P_min weighs the edges
// near 0 and there are at most h of them), U there (at p), the bin's density.
template <typename T>
struct VertexBins {
  const T* p;
  int left;  // bins above the current one
  T k, nv, pv, uv, dv, idv;
};

template <typename T>
CP_HD void vertex_bins_init(VertexBins<T>& b, const HistSuf<T>& L, int ev, T hv) {
  const int h = L.h;
  b.dv = hv * (T(1) / T(h));
  b.idv = T(h) * crcp(hv);
  b.p = L.base + 3 * L.E + ev;
  b.k = T(1);
  b.left = h - 1;
  b.nv = h > 1 ? b.dv : hv;
  b.uv = *b.p;
  b.pv = (L.U(ev, 0) - b.uv) * b.idv;
}

// (past the last bin the sweep has ended)
template <typename T>
CP_HD void vertex_bins_step(VertexBins<T>& b, int E, T hv) {
  b.p += b.left > 0 ? E : 0;
  b.left -= 1;
  b.k += T(1);
  const T u = *b.p;
  b.pv = (b.uv - u) * b.idv;
  b.uv = u;
  b.nv = b.left > 0 ? b.k * b.dv : hv;
}

// P_min and P_max of vertex ev; neighbour ranges [lo_i, hi_i] in the vertex
// frame (origin at the vertex lower end), vertex range [0, hv].  SAD: also
// the saddle terms t1 = int pdf_v S_e F_n S_w F_s and t2 = int pdf_v F_e S_n
// F_w S_s (Eq. 4) in the same sweep: on every merged sub-interval the four
// survival and distribution functions are the ones P_min and P_max use, so
// the two mixed products are two more exact integrals (the caller keeps them
// only for vertices with all four neighbours).
//
// Bound by vector issue: about 300 cycles per wave and interval, half of them
// the five cursor branches (a wave's lanes cross different edges, so all of
// them run).  P_min / P_max at 2048^2 x 10 bins: 0.506 -> 0.404 ms, of which the
// staging found every cell once instead of per plane gave 0.04.
template <typename T, bool SAD = false>
__host__ __device__ void hist_vertex_sweep(const HistSuf<T>& L, int ev, const int (&en)[4], const bool (&pres)[4],
                                           T hv, const T (&lo)[4], const T (&hi)[4], T& pmin, T& pmax, T& t1,
                                           T& t2) {
  const int h = L.h;
  const T big = hv + hv + T(1);
  VertexBins<T> vb;
  vertex_bins_init(vb, L, ev, hv);
  SufCursor<T> c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) suf_cursor_init(c[i], L, en[i], lo[i], hi[i], pres[i], big);
  T x0 = T(0), amin = T(0), amax = T(0), a1 = T(0), a2 = T(0);
  // integrals over the vertex's open bin, whose density they get when it ends
  T bmin = T(0), bmax = T(0), b1 = T(0), b2 = T(0);
  const auto fold = [&] {
    amin = cfma(vb.pv, bmin, amin);
    amax = cfma(vb.pv, bmax, amax);
    bmin = bmax = T(0);
    if constexpr (SAD) {
      a1 = cfma(vb.pv, b1, a1);
      a2 = cfma(vb.pv, b2, a2);
      b1 = b2 = T(0);
    }
  };
  const int maxit = 5 * (h + 1) + 2;  // every step crosses at least one edge
  for (int it = 0; it < maxit; ++it) {
    if (!(x0 < hv)) break;
    T x1 = vb.nv;
#pragma unroll
    for (int i = 0; i < 4; ++i) x1 = fmin_nn(x1, c[i].nxt);  // sweep edges: finite
    // The factors at the midpoint, S and F, and their half-change t >= 0: on
    // y in [-1, 1] S_i = S - t y, F_i = F + t y.  Opposite neighbours are
    // multiplied into quadratics p0 -/+ p1 y + p2 y^2 (p1 the magnitude for
    // S and F alike, p2 shared by them), and two quadratics integrate to
    //   2 [p0 q0 + (p0 q2 + p2 q0 +/- p1 q1) / 3 + p2 q2 / 5],
    // + where both are of S or both of F: then every term is non-negative and
    // nothing cancels.  In the saddle terms one of each, the magnitudes sum
    // to at most six times the result.  27 operations for P_min and P_max
    // (39 with the saddle terms) against 46 (92) from the end values in
    // Bernstein form.
    // The midpoint is reached from the interval's end, whose distance to the
    // cursor's edge is exact or small, and an interval's integrals get the
    // vertex's density with its whole bin: with a rounded midpoint and one sum
    // over all intervals the probabilities rounded worse than the end values'
    // (rms, FP32 and 4 bins 1.13 times, FP64 and 10 bins 1.1; so 1.04 and 0.9;
    // it costs the forward 2%).
    const T hl = (x1 - x0) * T(0.5);
    T S[4], F[4], t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      S[i] = cfma(c[i].slope, (c[i].nxt - x1) + hl, c[i].snx);
      F[i] = c[i].tot - S[i];
      t[i] = c[i].slope * hl;
    }
    T s0[2], s1[2], f0[2], f1[2], q2[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      s0[p] = S[p] * S[p + 2];
      s1[p] = cfma(S[p], t[p + 2], S[p + 2] * t[p]);
      f0[p] = F[p] * F[p + 2];
      f1[p] = cfma(F[p], t[p + 2], F[p + 2] * t[p]);
      q2[p] = t[p] * t[p + 2];
    }
    const T top = T(0.2) * (q2[0] * q2[1]), wgt = x1 - x0;
    const auto quartic = [&](T p0, T p1, T r0, T r1) {  // p1 r1 with the sign of its term
      const T m = cfma(p0, q2[1], cfma(q2[0], r0, p1 * r1));
      return cfma(T(1.0 / 3.0), m, cfma(p0, r0, top));
    };
    bmin = cfma(wgt, quartic(s0[0], s1[0], s0[1], s1[1]), bmin);
    bmax = cfma(wgt, quartic(f0[0], f1[0], f0[1], f1[1]), bmax);
    if constexpr (SAD) {
      b1 = cfma(wgt, quartic(s0[0], s1[0], f0[1], -f1[1]), b1);
      b2 = cfma(wgt, quartic(f0[0], f1[0], s0[1], -s1[1]), b2);
      settle(b1);
      settle(b2);
    }
    // the old state is dead from here on: the steps update it in place
    settle(bmin);
    settle(bmax);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (c[i].nxt == x1) suf_cursor_step(c[i], L.E, big);
    if (vb.nv == x1) {
      fold();
      vertex_bins_step(vb, L.E, hv);
    }
    x0 = x1;
  }
  fold();
  pmin = amin;
  pmax = amax;
  t1 = a1;
  t2 = a2;
}

template <typename T>
__host__ __device__ void hist_vertex_minmax(const HistSuf<T>& L, int ev, const int (&en)[4], const bool (&pres)[4],
                                            T hv, const T (&lo)[4], const T (&hi)[4], T& pmin, T& pmax) {
  T t1, t2;
  hist_vertex_sweep<T, false>(L, ev, en, pres, hv, lo, hi, pmin, pmax, t1, t2);
}

}  // namespace cp
