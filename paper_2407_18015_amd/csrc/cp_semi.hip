// cp_semi.hip -- semianalytical histogram estimator (Sec. 4.4.2).
//
// c samples are drawn from each vertex histogram; for each sample the
// probability that a neighbour lies above (below) it is closed-form: the
// neighbour's bin is found by one multiply, and the masses of the earlier
// bins come from cumulative sums prepared once per staged vertex (the paper's
// prefix-sum step), so the work per sample does not grow with the number of
// bins except for locating the sample's own bin.  The products are averaged:
//   P_min ~ T (1/c) sum_i prod_n S_n(x_i),   P_max ~ T (1/c) sum_i prod_n F_n(x_i),
//   t1 ~ T (1/c) sum_i S_e F_n S_w F_s(x_i), t2 with S and F exchanged,
// T = the vertex's total mass.  Sample i of vertex (y, x) uses word i mod 4 of
// Philox4x32-10 with counter (i / 4, y*W + x, field_id, 2) under key seed,
// u = ((word >> 8) + 1/2) 2^-24, r = u T, bin j = #{k in 1..h-1 : C_k <= r}
// (C_k = m_0 + ... + m_{k-1}), f = (r - C_j) / m_j clamped to [0, 1] (0 for an
// empty bin), x = lo + Delta (j + f): the inverse of the histogram CDF.
//
// A tile of vertices stages lo, hi and the masses with a one-vertex halo and
// replaces the masses by the cumulative masses in place (FP64 running sums
// rounded once).  A wave then takes one vertex after the other, its lanes the
// Philox blocks of four samples: all five histograms are wave-uniform, so what
// a sample needs of them is laid out once per vertex in small tables,
//   own:  the least 24-bit integer n = word >> 8 of every bin, x at that
//         integer and the slope of x in n,
//   near: (C_k, m_k) of every neighbour and bin,
// whose entries (ten bins: 240 and 176 bytes) lie in different banks, so the
// lanes' reads of different bins do not conflict.
//
// Positions and tails in FP64 for both dtypes, in vertex-local coordinates: in
// FP32 a position carries an error of one unit in the last place of the
// distribution width, which is h units of a bin, and the neighbour's tail
// inherits it for every sample alike.
//
// Bound by vector issue: about 65 FP64 or integer instructions of four cycles
// a sample.  1024^2 x 10 bins x 1000 samples, a thread per vertex -> this:
// 5.51 -> 2.07 ms (40^2: 1086 -> 30 us).  Five waves per SIMD are asked for: 96
// registers, of which 5 to 10 spill (24 to 44 bytes of scratch a lane; ten bins 7);
// four waves without spills took 5% longer, no bound 15%.  Which calls take this
// form: semi_by_thread.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "cp_hist.hpp"
#include "cp_internal.hpp"
#include "cp_philox.hpp"
#include "cp_tiles.hpp"
#include "cp_wave.hpp"

namespace cp {

namespace {

template <typename T>
struct SemiArgs {
  const T* params;
  T* pmin;
  T* pmax;
  T* terms;  // [2][H][rs]: t1, t2
  int H, W, nb, ns;
  int64_t rs, ps;
  uint32_t k0, k1, fid;
};

// Few samples: one thread per vertex, looping over its samples in tiles of
// 64 x TY staged vertices; the sample's bin by counting the cumulative masses.
template <typename T>
__device__ __forceinline__ T clamp01(T v) {
  return v < T(0) ? T(0) : (v > T(1) ? T(1) : v);
}

template <typename T, int TY>
__global__ __launch_bounds__(kFwdTX* TY) void k_semi_vertex(SemiArgs<T> a, int tiles_x, int ntiles) {
  constexpr int TX = kFwdTX, EX = TX + 2, EY = TY + 2, E = EX * EY, NT = TX * TY;
  extern __shared__ __align__(16) unsigned char smem[];
  T* lds = reinterpret_cast<T*>(smem);
  const int t = xcd_tile(blockIdx.x, ntiles);
  const int ty0 = (t / tiles_x) * TY, tx0 = (t % tiles_x) * TX, tid = threadIdx.x;
  const int h = a.nb;
  stage<T, EY, EX, NT>(lds, a.params, 2 + h, a.ps, a.rs, a.H, a.W, ty0 - 1, tx0 - 1, tid);
  __syncthreads();
  hist_stage_validity<T, NT>(lds, E, h, tid);
  // cumulative masses over the mass planes: plane k - 1 of `cum` holds C_k,
  // k = 1..h (C_h = T); the thread that checked a vertex sums it
  T* cum = lds + (size_t)2 * E;
  for (int e = tid; e < E; e += NT) {
    double c = 0.0;
    for (int k = 0; k < h; ++k) {
      c += (double)cum[k * E + e];
      cum[k * E + e] = (T)c;
    }
  }
  __syncthreads();
  const int lx = tid % TX, ly = tid / TX;
  const int x = tx0 + lx, y = ty0 + ly;
  if (x >= a.W || y >= a.H) return;
  const HistLds<T> L{lds, E, h, T(1) / T(h)};
  const int e = (ly + 1) * EX + lx + 1;
  const int en[4] = {e + 1, e - EX, e - 1, e + EX};
  const bool pres[4] = {x + 1 < a.W, y > 0, x > 0, y + 1 < a.H};
  bool ok = L.valid(e);
#pragma unroll
  for (int i = 0; i < 4; ++i) ok = ok && (!pres[i] || L.valid(en[i]));
  T out[4] = {qnan<T>(), qnan<T>(), qnan<T>(), qnan<T>()};
  if (ok) {
    using A = double;
    const A lov = (A)lds[e];
    const A dv = ((A)lds[E + e] - lov) / A(h);
    const T Tv = cum[(h - 1) * E + e];
    A lo[4], id[4], tot[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] = (A)lds[en[i]] - lov;
      id[i] = A(h) / ((A)lds[E + en[i]] - (A)lds[en[i]]);
      tot[i] = (A)cum[(h - 1) * E + en[i]];
    }
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const uint32_t at = (uint32_t)((int64_t)y * a.W + x);
    const PhiloxKeys keys = philox_keys<false>(a.k0, a.k1);
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    for (int i = 0; i < a.ns; ++i) {
      if ((i & 3) == 0) {
        w[0] = (uint32_t)(i >> 2);
        w[1] = at;
        w[2] = a.fid;
        w[3] = 2u;
        philox(w, keys);
      }
      const A r = u24_of<A>(w[i & 3]) * (A)Tv;
      int j = 0;
      for (int k = 1; k < h; ++k) j += (A)cum[(k - 1) * E + e] <= r ? 1 : 0;
      const A cj = j > 0 ? (A)cum[(j - 1) * E + e] : A(0);
      const A mj = (A)cum[j * E + e] - cj;
      const A f = mj > A(0) ? clamp01((r - cj) / mj) : A(0);
      const A xs = dv * (A(j) + f);
      A S[4], F[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        S[n] = A(1);
        F[n] = A(1);
        if (!pres[n]) continue;
        const A z = (xs - lo[n]) * id[n];
        if (!(z > A(0))) {
          S[n] = tot[n];
          F[n] = A(0);
        } else if (!(z < A(h))) {
          S[n] = A(0);
          F[n] = tot[n];
        } else {
          const int k = min((int)z, h - 1);
          const A below = k > 0 ? (A)cum[(k - 1) * E + en[n]] : A(0);
          F[n] = fma((A)cum[k * E + en[n]] - below, z - A(k), below);
          S[n] = tot[n] - F[n];
        }
      }
      acc[0] += S[0] * S[1] * S[2] * S[3];
      acc[1] += F[0] * F[1] * F[2] * F[3];
      acc[2] += S[0] * F[1] * S[2] * F[3];
      acc[3] += F[0] * S[1] * F[2] * S[3];
    }
    const double sc = (double)Tv / (double)a.ns;
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = (T)(acc[q] * sc);
    // the alternating pattern needs all four neighbours
    if (!(pres[0] && pres[1] && pres[2] && pres[3])) out[2] = out[3] = T(0);
  }
  const int64_t o = (int64_t)y * a.rs + x;
  if (a.pmin) a.pmin[o] = out[0];
  if (a.pmax) a.pmax[o] = out[1];
  if (a.terms) {
    a.terms[o] = out[2];
    a.terms[a.ps + o] = out[3];
  }
}

struct alignas(16) Pair {
  double a, b;
};

// a bin of the vertex: its least integer n = word >> 8, x there, slope of x in n
struct Bin {
  double x, slope;
  uint32_t n, pad;
};

// bytes of one wave's tables: near [4][h + 1] and the affine map of every
// neighbour [4] (Pairs), then the bins [2^ST]
constexpr int semi_pairs(int h) { return 4 * (h + 1) + 4; }
inline int semi_table_bytes(int h, int st) { return (int)sizeof(Pair) * semi_pairs(h) + ((int)sizeof(Bin) << st); }

// r of the 24-bit integer n, rounded as u24_of and one product
__device__ __forceinline__ double semi_r(uint32_t n, double T) {
  return ((double)n + 0.5) * 5.9604644775390625e-8 * T;
}

// TX x TY vertices per block of four waves; 2^ST >= h
template <typename T, int TX, int TY, int ST>
__global__ __launch_bounds__(256, 5) void k_semi(SemiArgs<T> a, int tiles_x, int ntiles, int table_at, int table_bytes) {
  constexpr int EX = TX + 2, EY = TY + 2, E = EX * EY, NT = 256;
  extern __shared__ __align__(16) unsigned char smem[];
  T* lds = reinterpret_cast<T*>(smem);
  const int t = xcd_tile(blockIdx.x, ntiles);
  const int ty0 = (t / tiles_x) * TY, tx0 = (t % tiles_x) * TX, tid = threadIdx.x;
  const int h = a.nb;
  stage<T, EY, EX, NT>(lds, a.params, 2 + h, a.ps, a.rs, a.H, a.W, ty0 - 1, tx0 - 1, tid);
  __syncthreads();
  hist_stage_validity<T, NT>(lds, E, h, tid);
  // cumulative masses over the mass planes: plane k - 1 of `cum` holds C_k,
  // k = 1..h (C_h = T); the thread that checked a vertex sums it
  T* cum = lds + (size_t)2 * E;
  for (int e = tid; e < E; e += NT) {
    double c = 0.0;
    for (int k = 0; k < h; ++k) {
      c += (double)cum[k * E + e];
      cum[k * E + e] = (T)c;
    }
  }
  __syncthreads();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Pair* near = reinterpret_cast<Pair*>(smem + table_at + wave * table_bytes);
  Pair* map = near + 4 * (h + 1);
  Bin* own = reinterpret_cast<Bin*>(map + 4);
  const PhiloxKeys keys = philox_keys(a.k0, a.k1);
  const double dh = (double)h, ih = 1.0 / dh, ins = 1.0 / (double)a.ns;
  const int nb_i = lane >> 4, to_nb = nb_i == 0 ? 1 : nb_i == 1 ? -EX : nb_i == 2 ? -1 : EX;

  for (int v = wave; v < TX * TY; v += 4) {
    const int lx = v % TX, ly = v / TX, x = tx0 + lx, y = ty0 + ly;
    if (x >= a.W || y >= a.H) continue;
    const int e = (ly + 1) * EX + lx + 1;
    const int en[4] = {e + 1, e - EX, e - 1, e + EX};
    const bool pres[4] = {x + 1 < a.W, y > 0, x > 0, y + 1 < a.H};
    bool ok = lds[e] == lds[e];
#pragma unroll
    for (int i = 0; i < 4; ++i) ok = ok && (!pres[i] || lds[en[i]] == lds[en[i]]);
    double out[4] = {0.0, 0.0, 0.0, 0.0};
    const double lov = (double)lds[e], dv = ((double)lds[E + e] - lov) * ih;
    const double Tv = (double)cum[(h - 1) * E + e];
    if (ok) {
      // lanes 16 i .. 16 i + 15: entries of neighbour i; an absent one has
      // S = F = 1 everywhere
      const int ei = e + to_nb;
      const bool has = nb_i == 0 ? pres[0] : nb_i == 1 ? pres[1] : nb_i == 2 ? pres[2] : pres[3];
      for (int k = lane & 15; k <= h; k += 16) {
        Pair p{1.0, 0.0};
        if (has) {
          p.a = k > 0 ? (double)cum[(k - 1) * E + ei] : 0.0;
          p.b = k < h ? (double)cum[k * E + ei] - p.a : 0.0;
        }
        near[nb_i * (h + 1) + k] = p;
      }
      if ((lane & 15) == 0) {
        Pair m{0.0, 0.0};
        if (has) {
          const double lo = (double)lds[ei];
          m.a = 1.0 / ((double)lds[E + ei] - lo);
          m.b = (lov - lo) * m.a;
        }
        map[nb_i] = m;
      }
      // bin j holds the integers from its own (the least n with C_j <= r(n))
      // up to the next bin's; none reaches the bins above h - 1
      const int j = lane;
      if (j < (1 << ST)) {
        Bin o{0.0, 0.0, 0xffffffffu, 0u};
        if (j < h) {
          const double cj = j > 0 ? (double)cum[(j - 1) * E + e] : 0.0, mj = (double)cum[j * E + e] - cj;
          double g = 0.0;
          if (j > 0 && Tv > 0.0) g = fmin(fmax(ceil(cj / Tv * 16777216.0 - 0.5), 0.0), 16777216.0);
          uint32_t n = (uint32_t)g;
          if (j > 0 && n > 0 && cj <= semi_r(n - 1, Tv)) n -= 1;
          if (j > 0 && !(cj <= semi_r(n, Tv))) n += 1;
          // (a bin of a single integer needs no slope: kept finite)
          const double im = mj > 0.0 ? 1.0 / mj : 0.0;
          const double f = fmin(fmax((semi_r(n, Tv) - cj) * im, 0.0), 1.0);
          o = Bin{dv * ((double)j + f), dv * fmin(5.9604644775390625e-8 * Tv * im, 1.0), n, 0u};
        }
        own[j] = o;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();

      double iw[4], off[4], tot[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        iw[i] = map[i].a;
        off[i] = map[i].b;
        tot[i] = pres[i] ? near[i * (h + 1) + h].a : 2.0;
      }
      double acc[4] = {0.0, 0.0, 0.0, 0.0};
      const uint32_t at = (uint32_t)((int64_t)y * a.W + x);
      const auto block = [&](int b, auto all) {
        uint32_t w[4] = {(uint32_t)b, at, a.fid, 2u};
        philox(w, keys);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const uint32_t n = w[s] >> 8;
          const Bin* o = own;
#pragma unroll
          for (int st = ST - 1; st >= 0; --st) o = n >= o[1 << st].n ? o + (1 << st) : o;
          const double xs = fma((double)(n - o->n), o->slope, o->x);
          double S[4], F[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double z = fmin(fmax(fma(xs, iw[i], off[i]), 0.0), 1.0) * dh;
            const Pair p = near[i * (h + 1) + (int)z];
            F[i] = fma(p.b, __builtin_amdgcn_fract(z), p.a);
            S[i] = tot[i] - F[i];
          }
          if (!decltype(all)::value && 4 * b + s >= a.ns) S[0] = F[0] = 0.0;
          const double sa = S[0] * S[2], fa = F[0] * F[2], sb = S[1] * S[3], fb = F[1] * F[3];
          acc[0] = fma(sa, sb, acc[0]);
          acc[1] = fma(fa, fb, acc[1]);
          acc[2] = fma(sa, fb, acc[2]);
          acc[3] = fma(fa, sb, acc[3]);
        }
      };
      // (the pass that holds a partial block looks at every sample)
      const int blocks = semi_blocks(a.ns), full = a.ns & 3 ? (blocks - 1) & ~63 : blocks;
      for (int b = lane; b < full; b += 64) block(b, std::true_type{});
      if (full + lane < blocks) block(full + lane, std::false_type{});
      // the tables are read before the next vertex overwrites them
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // row 0..3 of the wave: sums 0, 2, 1, 3
      out[0] = row_sum(pair_sum<16>(pair_sum<32>(acc[0], acc[1]), pair_sum<32>(acc[2], acc[3])));
    }
    if ((lane & 15) == 0) {
      const int q = lane >> 4;  // min, t1, max, t2
      // the alternating pattern needs all four neighbours
      const bool inside = pres[0] && pres[1] && pres[2] && pres[3];
      T r = (T)(out[0] * (Tv * ins));
      if ((q & 1) && !inside) r = T(0);
      if (!ok) r = qnan<T>();
      const int64_t o = (int64_t)y * a.rs + x;
      T* to = q == 0 ? a.pmin : q == 2 ? a.pmax : a.terms ? a.terms + (q == 3 ? a.ps : 0) : nullptr;
      if (to) to[o] = r;
    }
  }
}

int cdiv_s(int p, int q) { return (p + q - 1) / q; }

template <typename T, int TX, int TY, int ST>
hipError_t launch_semi(const SemiArgs<T>& a, hipStream_t st) {
  const int tx = cdiv_s(a.W, TX), ty = cdiv_s(a.H, TY), n = tx * ty;
  const int at = (int)(sizeof(T) * (2 + a.nb) * (TX + 2) * (TY + 2) + 15) / 16 * 16, tb = semi_table_bytes(a.nb, ST);
  hipLaunchKernelGGL((k_semi<T, TX, TY, ST>), dim3(n), dim3(256), at + 4 * tb, st, a, tx, n, at, tb);
  return hipGetLastError();
}

// 16 x 4 vertices per block (16 a wave); fields with fewer than two such
// blocks per CU take 8 x 2
template <typename T, int ST>
hipError_t launch_semi_tiles(const SemiArgs<T>& a, hipStream_t st) {
  if ((int64_t)cdiv_s(a.W, 16) * cdiv_s(a.H, 4) >= 512) return launch_semi<T, 16, 4, ST>(a, st);
  return launch_semi<T, 8, 2, ST>(a, st);
}

template <typename T, int TY>
hipError_t launch_semi_vertex(const SemiArgs<T>& a, hipStream_t st) {
  const int tx = cdiv_s(a.W, kFwdTX), ty = cdiv_s(a.H, TY), n = tx * ty;
  const size_t lds = sizeof(T) * (size_t)(2 + a.nb) * (kFwdTX + 2) * (TY + 2);
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_semi_vertex<T, TY>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_semi_vertex<T, TY>), dim3(n), dim3(kFwdTX * TY), lds, st, a, tx, n);
  return hipGetLastError();
}

template <typename T>
hipError_t semi_typed(const Field& f, const void* params, void* pmin, void* pmax, void* terms, hipStream_t st) {
  SemiArgs<T> a;
  a.params = static_cast<const T*>(params);
  a.pmin = static_cast<T*>(pmin);
  a.pmax = static_cast<T*>(pmax);
  a.terms = static_cast<T*>(terms);
  a.H = f.H;
  a.W = f.W;
  a.nb = f.nb;
  a.ns = f.ns;
  a.rs = f.rs;
  a.ps = f.plane();
  a.k0 = (uint32_t)f.seed;
  a.k1 = (uint32_t)(f.seed >> 32);
  a.fid = f.fid;
  if (semi_by_thread(f.ns, f.nb, sizeof(T), (int64_t)f.H * f.W)) {
    // tile height: the staged planes (the masses overwritten by their
    // cumulative sums) must fit the LDS
    const size_t per_row = sizeof(T) * (size_t)(2 + f.nb) * (kFwdTX + 2);
    if (per_row * 6 <= 64 * 1024) return launch_semi_vertex<T, 4>(a, st);
    if (per_row * 4 <= 160 * 1024) return launch_semi_vertex<T, 2>(a, st);
    return launch_semi_vertex<T, 1>(a, st);
  }
  // search steps: 2^ST bins (at most 32); 32 bins in FP64 take 41 KB of LDS
  static_assert(kMaxBins <= 32, "search table");
  if (f.nb <= 4) return launch_semi_tiles<T, 2>(a, st);
  if (f.nb <= 8) return launch_semi_tiles<T, 3>(a, st);
  if (f.nb <= 16) return launch_semi_tiles<T, 4>(a, st);
  return launch_semi_tiles<T, 5>(a, st);
}

}  // namespace

hipError_t semi_forward(const Field& f, const void* params, void* pmin, void* pmax, void* terms, hipStream_t st) {
  if (f.dtype == CP_F64) return semi_typed<double>(f, params, pmin, pmax, terms, st);
  return semi_typed<float>(f, params, pmin, pmax, terms, st);
}

}  // namespace cp
