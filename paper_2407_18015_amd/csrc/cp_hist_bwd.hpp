// cp_hist_bwd.hpp -- adjoint of the histogram model with respect to the bin
// masses (free variables: P is multilinear in them, as in Eq. 5).
//
// One sweep over the vertex range integrates, for both P_min (prod S) and
// P_max (prod F = T - S), the leave-one-out products of every neighbour and
// their products with the survival function of the neighbour's current bin
// kernel, and emits each bin's weighted entry when the sweep leaves the bin.
// On every sub-interval all factors are linear, so the integrands are
// polynomials of degree <= 4: 2-point Gauss-Legendre plus the rule's
// remainder for the quartic terms, in closed form from the factors' slopes,
// integrates them exactly.  Entries of absent neighbours are not emitted.
//
// The sweep tile writes each stencil's entries to a workspace; a second
// kernel gathers every mass's five entries (no atomics).
#pragma once

#include "cp_hist.hpp"
#include "cp_internal.hpp"
#include "cp_tiles.hpp"

namespace cp {

// ---------------------------------------------------------------------------
// Both sides in one sweep over the vertex range [0, hv] (staged suffix sums):
//   dP_min/dm_j(v) = (1/Delta_v) int_{bin j of v} prod_n S_n
//   dP_max/dm_j(v) = (1/Delta_v) int_{bin j of v} prod_n F_n
//   dP_min/dm_j(n) = QS_n(e_j) + int_{bin j of n} pdf_v Kbar_j prod_{k!=n} S_k
//   dP_max/dm_j(n) = QF_n(hv) - QF_n(e_j) - int_{bin j of n} pdf_v Kbar_j prod_{k!=n} F_k
// with QS_n(y) = int_0^y pdf_v prod_{k!=n} S_k, QF_n likewise with F, and
// Kbar_j = (e_{j+1} - x)/Delta_n the survival function of bin j's kernel
// (dS_n/dm_j = Kbar_j, dF_n/dm_j = 1 - Kbar_j).  The upstream weights are
// folded into the accumulators (QS' = g_min QS, QF' = -g_max QF), so the
// entry of a neighbour bin is B + (1/Delta_n) int_{bin} (e_{j+1} - x)(lS + lF)
// with B = QS' + QF' at the bin's lower edge; it is emitted when the sweep
// leaves the bin, without the g_max QF_n(hv) term, which is known only at the
// end and belongs to every bin of the neighbour at or below the open one: it
// is stored once per neighbour (J.tail) and the gather adds it to all of the
// neighbour's bins, so the bins above the open one are emitted as
// QS_n(hv) - tail = B, those below the sweep as 0, and no entry is read back.  The node weights carry
// the vertex pdf and the half-length of the sub-interval, so the
// accumulators run over the whole sweep.
//
// Cursors as in the forward (SufCursor, VertexBins), staged layout of
// cp_hist.hpp.  A cursor's step and the emission of the bin it leaves are one
// branch with the state updated in place: selects cost four issue cycles each,
// and each interval ran the four of every cursor although it ends one or two
// bins.  Bound by vector issue, 535 cycles per wave and interval (760 before;
// both nodes unrolled, places as running pointers: 126 registers, four waves
// per SIMD, where rolled nodes and five waves took 2% longer), and beyond the
// caches by the entries' stores (JRow).  Adjoint with ten bins, 2048^2 1.29 ->
// 1.17 ms, 1024^2 0.335 -> 0.298.
//
// J.at(slot, k) is the place of an entry, J.step moves it to the next bin's,
// J.put emits there and J.tail(i, value) the tail of neighbour i; slot 0 is the
// vertex's own histogram, slot 1 + i neighbour i (e, n, w, s).
// ---------------------------------------------------------------------------
template <typename T, typename JOut>
__host__ __device__ void hist_jac_both(const HistSuf<T>& L, int ev, const int (&en)[4], const bool (&pres)[4],
                                       T hv, const T (&lo)[4], const T (&hi)[4], T gmin, T gmax, JOut& J, T& pmin,
                                       T& pmax) {
  const int h = L.h, E = L.E;
  const T big = hv + hv + T(1);
  VertexBins<T> vb;
  vertex_bins_init(vb, L, ev, hv);
  SufCursor<T> c[4];
  // where the open bin's entry goes (not read while the cursor is below its
  // range), and the first bin the sweep enters
  typename JOut::At jv = J.at(0, 0), jn[4];
  int first[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    suf_cursor_init(c[i], L, en[i], lo[i], hi[i], pres[i], big);
    const int j = (int)c[i].k + h - 1;  // the open bin (-1: below the range)
    jn[i] = J.at(1 + i, j);
    first[i] = j < 0 ? 0 : j;
  }
  const T below = T(-h);
  // B_n = QS'_n + QF'_n so far; Y_n = B_n Delta_n + (kernel-weighted integral over the open bin so far):
  // the entry of a bin left is Y_n / Delta_n
  T B[4], QF[4], Y[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) B[i] = QF[i] = Y[i] = T(0);
  T vS = T(0), vF = T(0), amin = T(0), amax = T(0);
  T x0 = T(0);
  const int maxit = 5 * (h + 1) + 2;
  for (int it = 0; it < maxit; ++it) {
    if (!(x0 < hv)) break;
    T x1 = vb.nv;
#pragma unroll
    for (int i = 0; i < 4; ++i) x1 = fmin_nn(x1, c[i].nxt);  // sweep edges: finite
    const T mid = (x0 + x1) * T(0.5), hl = (x1 - x0) * T(0.5);
    const T php = vb.pv * hl, wS = php * gmin, wF = -php * gmax;
    // two-point Gauss-Legendre: exact for the leave-one-out products (degree
    // 3); the degree-4 integrands (full products, leave-one-out products times
    // the bin kernel) get the rule's remainder in closed form below.
    const T dx = hl * T(GL<2>::x[1]);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const T x = q ? mid + dx : mid - dx;  // both weights 1
      T S[4], F[4], r[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        r[i] = c[i].nxt - x;
        S[i] = cfma(c[i].slope, r[i], c[i].snx);
        F[i] = c[i].tot - S[i];
      }
      const T s01 = S[0] * S[1], s23 = S[2] * S[3], f01 = F[0] * F[1], f23 = F[2] * F[3];
      vS = cfma(hl * s01, s23, vS);
      vF = cfma(hl * f01, f23, vF);
      const T ps01 = wS * s01, ps23 = wS * s23, pf01 = wF * f01, pf23 = wF * f23;
      const T lf[4] = {F[1] * pf23, F[0] * pf23, F[3] * pf01, F[2] * pf01};
      const T l[4] = {cfma(S[1], ps23, lf[0]), cfma(S[0], ps23, lf[1]), cfma(S[3], ps01, lf[2]),
                      cfma(S[2], ps01, lf[3])};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        B[i] += l[i];
        QF[i] += lf[i];
        Y[i] = cfma(l[i], r[i], Y[i]);
      }
    }
    // The rule misses (8/45) hl^5 c4 of a quartic with leading coefficient
    // c4.  S_k has slope -s_k and F_k slope +s_k (s_k the cursor's density),
    // so c4 is s0 s1 s2 s3 for both full products, and pdf_v (g_min + g_max)
    // times the other three densities for an entry's kernel-weighted
    // integrand; in t_k = hl s_k (a change of S_k, bounded) no power of hl
    // or of a density is formed.
    {
      T t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = hl * c[i].slope;
      const T t01 = t[0] * t[1], t23 = t[2] * t[3];
      const T k45 = T(GLRem<2>::e) * hl;
      const T kv = k45 * (t01 * t23), ke = k45 * (wS - wF);
      vS += kv;
      vF += kv;
      const T lt[4] = {t[1] * t23, t[0] * t23, t[3] * t01, t[2] * t01};
#pragma unroll
      for (int i = 0; i < 4; ++i) Y[i] = cfma(ke, lt[i], Y[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) settle(Y[i]);
    // bin boundaries, one branch each: inside it the state is updated in
    // place (nothing reads the old one any more), so no selects
    if (vb.nv == x1) {  // the vertex's entry is complete
      J.put(0, jv, (gmin * vS + gmax * vF) * vb.idv);
      J.step(0, jv);
      amin = cfma(vb.pv, vS, amin);
      amax = cfma(vb.pv, vF, amax);
      vS = vF = T(0);
      vertex_bins_step(vb, E, hv);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (c[i].nxt == x1) {
        // the bin left (none if the cursor enters its range)
        if (c[i].k > below) J.put(1 + i, jn[i], c[i].id * Y[i]);
        J.step(1 + i, jn[i]);
        Y[i] = B[i] * c[i].d;
        suf_cursor_step(c[i], E, big);
      }
    }
    x0 = x1;
  }
  // remaining vertex bins (the sweep ended inside or past them): no range
  for (int k = (int)vb.k - 1; k < h; ++k) {
    J.put(0, jv, (gmin * vS + gmax * vF) * vb.idv);
    J.step(0, jv);
    amin = cfma(vb.pv, vS, amin);
    amax = cfma(vb.pv, vF, amax);
    vS = vF = T(0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!pres[i]) continue;
    J.tail(i, -QF[i]);  // g_max QF_n(hv), added to every bin by the gather
    const int j = (int)c[i].k + h - 1;  // open bin (-1: below the range, h: past it)
    // bins below the sweep: dF/dm = 1 there (the tail)
    auto q = J.at(1 + i, 0);
    for (int k = 0; k < first[i]; ++k) {
      J.put(1 + i, q, T(0));
      J.step(1 + i, q);
    }
    // the open bin, then those above the sweep: dS/dm = 1 there
    T v = j < 0 ? B[i] : c[i].id * Y[i];
    q = J.at(1 + i, j < 0 ? 0 : j);
    for (int k = j < 0 ? 0 : j; k < h; ++k) {
      J.put(1 + i, q, v);
      J.step(1 + i, q);
      v = B[i];
    }
  }
  pmin = amin;
  pmax = amax;
}

// Entries of one stencil stored at J[(slot * h + k) * EJ + sj], its four
// tails at J[(5 h + i) * EJ + sj] (the workspace layout, [5 h + 4][H][W];
// also used by the host-side checks).  The plane size EJ (= H W) is below
// 2^30 (the descriptor check bounds the grid), so the plane offset is one
// 32 x 32 -> 64-bit product.
template <typename T>
struct JPlanes {
  T* J;
  uint32_t EJ;
  int64_t sj;
  int h;
  using At = T*;
  CP_HD T* at(int slot, int k) const { return J + (int64_t)((uint64_t)(uint32_t)(slot * h + k) * EJ) + sj; }
  CP_HD void step(int, T*& a) const { a += EJ; }
  CP_HD void put(int, T* a, T v) const { *a = v; }
  CP_HD void tail(int i, T v) const { *at(5, i) = v; }  // plane 5 h + i
};

// The same for a wave that holds 64 consecutive vertices of a row: what the
// stencils of the row add to each other (slots v, e and w) is summed in LDS, G
// [h][66] with a column on either side for the neighbours outside, and only
// the sums, the entries for the rows above and below and the two edge columns
// go to the workspace.  The lanes of a wave leave a bin at different times, so
// every entry stored directly is a request of its own: 54 for a vertex of ten
// bins, and the sweep waited on them for a third of its time.  One wave's LDS
// operations run in order, so the sums are reproducible.
template <typename T>
struct JRow {
  JPlanes<T> P;
  T* G;
  int lane;
  T te, tw;  // tails of the e and w neighbour
  static constexpr int GX = 66;
  struct At {
    T *g, *l;  // workspace or LDS, by slot
  };
  static __device__ __forceinline__ bool in_row(int slot) { return slot == 0 || slot == 1 || slot == 3; }
  __device__ __forceinline__ At at(int slot, int k) const {
    return {in_row(slot) ? nullptr : P.at(slot, k), G + k * GX + lane + 1 + (slot == 1 ? 1 : slot == 3 ? -1 : 0)};
  }
  __device__ __forceinline__ void step(int slot, At& a) const {
    if (in_row(slot))
      a.l += GX;
    else
      a.g += P.EJ;
  }
  __device__ __forceinline__ void put(int slot, const At& a, T v) const {
    if (in_row(slot))
      __hip_atomic_fetch_add(a.l, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    else
      *a.g = v;
  }
  __device__ __forceinline__ void tail(int i, T v) {
    if (i == 0)
      te = v;
    else if (i == 2)
      tw = v;
    else
      P.tail(i, v);
  }
};

// Whether the adjoint sums rows on chip (sweep and gather agree on it): eight
// bins on, as far as the row buffers beside the staged planes leave the waves
// that the registers allow, on fields whose workspace is past half of the
// 256 MB last-level cache.  Direct entries depend on the data (how far the
// lanes of a wave drift apart), row sums do not.  FP32, 1024^2, direct over
// three ensembles and row sums: 6 bins 176-181 and 191 us, 8 bins 228-334 and
// 241, 10 bins 281-434 and 300, 18 bins 606-933 and 620, 20 bins 702-1059 and
// 893; 2048 x 1100 x 10 bins 631-860 and 670; 600 x 512 x 10 bins (66 MB)
// 104-133 and 122.  FP64, 1024^2: 8 bins 474-501 and 445, 13 bins 729-841 and
// 710, 16 bins 908-1035 and 1335.
__host__ __device__ constexpr bool hist_rows_fit(int h, size_t el) { return h >= 8 && h <= (el == 4 ? 18 : 13); }
__host__ __device__ constexpr bool hist_row_sums(int h, size_t el, int64_t vertices) {
  return hist_rows_fit(h, el) && hist_ws_planes(h) * (int64_t)el * vertices >= (int64_t)128 << 20;
}
// LDS of a sweep tile (elements): staged planes, then a row buffer per wave
__host__ __device__ constexpr size_t hist_sweep_lds(int h, int E, int nt, bool rows) {
  return (size_t)hist_planes(h) * E + (rows ? (size_t)(nt / 64) * h * 66 : 0);
}

// Both sides of one stencil (centre e in the staged tile, grid position
// (gy, gx)) into J; returns the probabilities; an invalid stencil emits NaN
// for its own bins and those of its present neighbours.
template <typename T, typename JOut>
__host__ __device__ void hist_stencil_jac(const HistLds<T>& L, const HistSuf<T>& U, const T* par, int EP, int PX,
                                          int e, int gy, int gx, int H, int W, T gmin, T gmax, JOut& J, T& pmin,
                                          T& pmax) {
  const int h = L.h;
  const int en[4] = {e + 1, e - PX, e - 1, e + PX};
  const bool pres[4] = {gx + 1 < W, gy > 0, gx > 0, gy + 1 < H};
  bool ok = L.valid(e);
#pragma unroll
  for (int k = 0; k < 4; ++k) ok = ok && (!pres[k] || L.valid(en[k]));
  if (!ok) {
    for (int k = 0; k < h; ++k) J.put(0, J.at(0, k), qnan<T>());
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (pres[i]) {
        for (int k = 0; k < h; ++k) J.put(1 + i, J.at(1 + i, k), qnan<T>());
        J.tail(i, T(0));
      }
    pmin = pmax = qnan<T>();
    return;
  }
  const T lov = par[e], hiv = par[EP + e];
  T lo[4], hi[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    lo[k] = par[en[k]] - lov;
    hi[k] = par[EP + en[k]] - lov;
  }
  hist_jac_both(U, e, en, pres, hiv - lov, lo, hi, gmin, gmax, J, pmin, pmax);
}

// Sweep tile of the adjoint: 64 x TY stencils (params staged with a
// one-vertex halo), entries written to the workspace J
// ([5 h + 4][H][W]: one plane per slot and bin, then the four tails, so the
// lanes of a wave that emit the same entry write consecutive words); a
// gather kernel then adds the five entries of every parameter.  If f.pmin is non-null the probabilities
// are written too (fused forward + adjoint).  NT threads; each takes the rows
// ly, ly + NT/64, ... of its column.
template <typename T, int TY, int NT = kFwdTX * TY>
__device__ __forceinline__ void tile_hist_sweep(const FieldPtrs<T>& f, int ty0, int tx0, T* lds, int tid, T* J) {
  constexpr int TX = kFwdTX, EX = TX + 2, EY = TY + 2, E = EX * EY;
  static_assert(NT % TX == 0 && TY % (NT / TX) == 0, "rows must split evenly over the threads");
  const int h = f.nb;
  stage<T, EY, EX, NT>(lds, f.params, 2 + h, f.ps, f.rs, f.H, f.W, ty0 - 1, tx0 - 1, tid);
  __syncthreads();
  hist_stage_validity<T, NT>(lds, E, h, tid);
  hist_stage_suffix<T, NT>(lds, E, h, tid);
  __syncthreads();
  const int lx = tid % TX, x = tx0 + lx;
  const bool rows = hist_row_sums(h, sizeof(T), (int64_t)f.H * f.W);
  T* G = lds + (size_t)hist_planes(h) * E + (size_t)(tid / TX) * h * JRow<T>::GX;
  for (int ly = tid / TX; ly < TY; ly += NT / TX) {
    const int y = ty0 + ly;
    if (x < f.W && y < f.H) {
      const HistLds<T> L{lds, E, h, T(1) / T(h)};
      const HistSuf<T> U{lds, E, h};
      const int64_t at = (int64_t)y * f.rs + x;
      const int64_t sj = (int64_t)y * f.W + x;
      T pmin, pmax;
      JPlanes<T> Jo{J, (uint32_t)((int64_t)f.H * f.W), sj, h};
      if (rows) {
        // (the active lanes are the first of the wave)
        const int n = f.W - tx0 < TX ? f.W - tx0 : TX;
        for (int i = lx; i < h * JRow<T>::GX; i += n) G[i] = T(0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        JRow<T> Jr{Jo, G, lx, T(0), T(0)};
        hist_stencil_jac(L, U, lds, E, EX, (ly + 1) * EX + lx + 1, y, x, f.H, f.W, f.gmin[at], f.gmax[at], Jr, pmin,
                         pmax);
        // tails from the west and east neighbours' stencils in the row
        T tails = T(0);
        const T fw = __shfl_up(Jr.te, 1, 64), fe = __shfl_down(Jr.tw, 1, 64);
        if (lx > 0) tails += fw;
        if (lx < TX - 1 && x + 1 < f.W) tails += fe;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        T* to = Jo.at(0, 0);
        const T* g = G + lx + 1;
        for (int k = 0; k < h; ++k, to += Jo.EJ, g += JRow<T>::GX) *to = *g + tails;
        // the columns beside the tile, at the stencils of its ends
        if (lx == 0 && x > 0) {
          Jo.tail(2, Jr.tw);
          for (int k = 0; k < h; ++k) *Jo.at(3, k) = G[k * JRow<T>::GX];
        }
        if (lx == TX - 1 && x + 1 < f.W) {
          Jo.tail(0, Jr.te);
          for (int k = 0; k < h; ++k) *Jo.at(1, k) = G[k * JRow<T>::GX + TX + 1];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      } else {
        hist_stencil_jac(L, U, lds, E, EX, (ly + 1) * EX + lx + 1, y, x, f.H, f.W, f.gmin[at], f.gmax[at], Jo, pmin,
                         pmax);
      }
      if (f.pmin) {
        f.pmin[at] = pmin;
        f.pmax[at] = pmax;
      }
    }
  }
  __syncthreads();
}

// gather of the two-kernel adjoint: every mass of u adds its own stencil's
// entry and the entries of its four neighbours' stencils that refer to u
// (own, east's w slot, west's e slot, north's s slot, south's n slot)
template <typename T>
CP_HD void hist_gather_vertex(const FieldPtrs<T>& f, const T* __restrict__ J, int64_t id) {
  const int64_t plane = (int64_t)f.H * f.W;
  if (id >= plane) return;
  const int y = (int)(id / f.W), x = (int)(id - (int64_t)y * f.W);
  const int h = f.nb;
  const int64_t at = (int64_t)y * f.rs + x;
  f.grad[at] = T(0);
  f.grad[f.ps + at] = T(0);
  const auto e = [&](int64_t v, int slot, int k) { return J[(int64_t)(slot * h + k) * plane + v]; };
  // tails of the four stencils: u is the west (east, south, north) neighbour
  // of its east (west, north, south) neighbour
  const T te = x + 1 < f.W ? e(id + 1, 5, 2) : T(0), tw = x > 0 ? e(id - 1, 5, 0) : T(0);
  const T tn = y > 0 ? e(id - f.W, 5, 3) : T(0), ts = y + 1 < f.H ? e(id + f.W, 5, 1) : T(0);
  // (a row summed on chip has its east and west entries but for the edges of
  // the 64-vertex tiles)
  const bool rows = hist_row_sums(h, sizeof(T), plane);
  const bool ge = x + 1 < f.W && (!rows || (x + 1) % kFwdTX == 0), gw = x > 0 && (!rows || x % kFwdTX == 0);
  for (int k = 0; k < h; ++k) {
    T g = e(id, 0, k);
    if (ge) g += e(id + 1, 3, k) + te;
    if (gw) g += e(id - 1, 1, k) + tw;
    if (y > 0) g += e(id - f.W, 4, k) + tn;
    if (y + 1 < f.H) g += e(id + f.W, 2, k) + ts;
    f.grad[(int64_t)(2 + k) * f.ps + at] = g;
  }
}

// The same gather for V = 16 / sizeof(T) vertices of one row per thread
// (W >= V): group q covers V vertices of row q / ceil(W / V), the last of a row
// its last V, so that some of them are gathered twice where V does not divide W
// (by the same operations, to the same values).  Vectors are at element
// alignment: the own and north / south entries, and the east / west ones
// shifted by one vertex (at a row end the lane takes no entry, and every
// address stays inside the workspace: the shifted rows of slots 1 and 3, of the
// tail planes and the rows above / below of slots 4 and 2 lie between plane 1
// and the last tail plane).  Terms are added in the scalar gather's order and
// absent ones skipped, so the sums are bit-identical to it.
template <typename T>
__host__ __device__ constexpr int gather_vec() {
  return 16 / (int)sizeof(T);
}
__host__ __device__ constexpr int64_t gather_groups(int H, int W, int V) { return (int64_t)H * ((W + V - 1) / V); }

template <typename T>
CP_HD void hist_gather_vec(const FieldPtrs<T>& f, const T* __restrict__ J, int64_t q) {
  constexpr int V = gather_vec<T>();
  typedef T Vec __attribute__((ext_vector_type(V)));
  if (q >= gather_groups(f.H, f.W, V)) return;
  const int64_t plane = (int64_t)f.H * f.W;
  const int gr = (f.W + V - 1) / V;
  const int y = (int)(q / gr), g0 = (int)(q - (int64_t)y * gr) * V, x = g0 < f.W - V ? g0 : f.W - V;
  const int64_t id = (int64_t)y * f.W + x;
  const int h = f.nb;
  const int64_t at = (int64_t)y * f.rs + x;
  const auto st = [&](int64_t v, const Vec& r) { __builtin_memcpy(f.grad + v, &r, sizeof(Vec)); };
  const Vec z = Vec(T(0));
  st(at, z);
  st(f.ps + at, z);
  const bool hasn = y > 0, hass = y + 1 < f.H;
  const auto ld = [&](int slot, int k, int64_t v) {  // V entries from vertex v on
    Vec r;
    __builtin_memcpy(&r, J + (int64_t)(slot * h + k) * plane + v, sizeof(Vec));
    return r;
  };
  const Vec te = ld(5, 2, id + 1), tw = ld(5, 0, id - 1);
  const Vec tn = ld(5, 3, hasn ? id - f.W : id), ts = ld(5, 1, hass ? id + f.W : id);
  if (hist_row_sums(h, sizeof(T), plane)) {
    // east and west entries only at the edges of the 64-vertex tiles: vertex
    // x + je has one to its east (none: je = V), x + jw to its west
    const int r = x % kFwdTX, je = r + V < kFwdTX || x - r + kFwdTX >= f.W ? V : kFwdTX - 1 - r;
    const int jw = r == 0 ? (x > 0 ? 0 : V) : (r + V > kFwdTX ? kFwdTX - r : V);
    for (int k = 0; k < h; ++k) {
      Vec g = ld(0, k, id);
      const Vec n = ld(4, k, hasn ? id - f.W : id), s = ld(2, k, hass ? id + f.W : id);
      T e = T(0), w = T(0);
      if (je < V) e = J[(int64_t)(3 * h + k) * plane + id + je + 1];
      if (jw < V) w = J[(int64_t)(h + k) * plane + id + jw - 1];
#pragma unroll
      for (int j = 0; j < V; ++j) {
        T t = g[j];
        if (j == je) t += e + te[j];
        if (j == jw) t += w + tw[j];
        if (hasn) t += n[j] + tn[j];
        if (hass) t += s[j] + ts[j];
        g[j] = t;
      }
      st((int64_t)(2 + k) * f.ps + at, g);
    }
    return;
  }
  for (int k = 0; k < h; ++k) {
    Vec g = ld(0, k, id);
    const Vec e = ld(3, k, id + 1), w = ld(1, k, id - 1);
    const Vec n = ld(4, k, hasn ? id - f.W : id), s = ld(2, k, hass ? id + f.W : id);
#pragma unroll
    for (int j = 0; j < V; ++j) {
      T t = g[j];
      if (x + j + 1 < f.W) t += e[j] + te[j];
      if (x + j > 0) t += w[j] + tw[j];
      if (hasn) t += n[j] + tn[j];
      if (hass) t += s[j] + ts[j];
      g[j] = t;
    }
    st((int64_t)(2 + k) * f.ps + at, g);
  }
}

}  // namespace cp
