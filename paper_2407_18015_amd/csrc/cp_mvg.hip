// cp_mvg.hip -- multivariate Gaussian over the 5-point stencil, Monte Carlo.
//
// The paper compares its closed forms with the correlated Gaussian model of
// prior work, sampled by Monte Carlo (Sec. 5.2: 1000 samples; Sec. 5.3: 2000
// samples).  Here a wave64 owns a vertex (or two); lane l takes samples l,
// l+64, ....
//
// Sample i of vertex (y, x): Philox4x32-10 with counter (i, y*W+x, field_id,
// b) and key (seed lo, seed hi); the four words of block b = 0 give uniforms
// u0..u3, words 0-1 of block 1 give u4, u5, each u = (r >> 8 + 1/2) 2^-24.
// Box-Muller pairs (u0,u1), (u2,u3), (u4,u5) give z0..z4, which drive
// (e, n, w, s, v): x = mu + L z.
//   hit estimator:         [x_v < min_n x_n]              (needs block 1)
//   conditional estimator: Phi((min_n x_n - c) / L44),   c = mu_v + sum_{j<4} L4j z_j
// The conditional estimator integrates the vertex given its neighbours in
// closed form (the paper's semianalytical idea of Sec. 4.4.2: sample part of
// the stencil, integrate the rest), has the same expectation, lower variance,
// needs one Philox block per sample, and is differentiable: the adjoint is
// its pathwise derivative.  Maxima use Phi((c - max_n x_n) / L44).
#include <hip/hip_runtime.h>

#include "cp_internal.hpp"
#include "cp_mc_math.hpp"
#include "cp_philox.hpp"
#include "cp_wave.hpp"

namespace cp {

namespace {

// ((word >> 8) + 1/2) 2^-24 in one fused multiply-add (scaling by a power of
// two is exact: the same value as u24_of<float>)
__device__ __forceinline__ float u24(uint32_t r) {
  return __builtin_fmaf((float)(r >> 8), 5.9604644775390625e-8f, 2.98023223876953125e-8f);
}

struct MvgArgs {
  const double* par;
  float* pmin;
  float* pmax;
  const float* gmin;
  const float* gmax;
  double* grad;
  double* jmu;  // [5][H][W] workspace (adjoint)
  int H, W, ns;
  int64_t rs, ps;
  uint32_t k0, k1, fid;
};

// The neighbours' values of a sample, a contraction of four rows of L with the
// sample's deviates, on the matrix cores.  v_mfma_f32_4x4x1 forms
// D[i][j] += A[i] B[j] in each of its 16 blocks of four lanes: with lane l
// holding row l mod 4 of the left matrix and its own sample's z_k as B, lane l
// receives the four values of its own sample.  The four instructions
// (k = 0..3) issue beside the vector unit, which this kernel keeps busy: 1.61
// against 1.81 ms with the 16 fused multiply-adds (500^2 x 2000).
//
// DIFF (the conditional estimator): rows L_nk - L_4k, so the values are x_n - c,
// differenced in FP64 and rounded once, with the deviates' kDeviateScale.
// A row whose neighbour is absent repeats the first present one, which leaves
// minimum and maximum as they are; without any neighbour all rows are +inf.
//
// Otherwise (the hit estimator, whose counts are whole numbers that a rounding
// can change, and the adjoint) the rows of L: each value is then the chain of FP32
// fused multiply-adds mu_n - mu_v + L_n0 z_0 + ... in the order of k.  A row
// whose neighbour is absent is NaN, which minimum and maximum skip.
typedef float f32x4 __attribute__((ext_vector_type(4)));
struct MvgStencil {
  float row[4];  // lane l: row of neighbour l mod 4
  f32x4 d;       // mu_n - mu_v (wave-uniform)
  float L44;
  int first;      // first present neighbour, 4: none
};

//
// Loads of absent values are skipped with DIFF and made elsewhere without it, by
// measurement (500^2 x 64: conditional 109 us skipped and 117 made, hits 130 and 122).
template <bool DIFF>
__device__ __forceinline__ void load_stencil(const MvgArgs& a, int v, int lane, MvgStencil& s) {
  const int y = v / a.W, x = v - y * a.W;
  const int64_t at = (int64_t)y * a.rs + x;
  const double mv = a.par[at];
  const bool pres[4] = {x + 1 < a.W, y > 0, x > 0, y + 1 < a.H};
  const int64_t off[4] = {1, -a.rs, -1, a.rs};
  float d0 = __builtin_inff();
  s.first = 4;
#pragma unroll
  for (int i = 3; i >= 0; --i) {
    if constexpr (DIFF) {
      s.d[i] = pres[i] ? (float)(a.par[at + off[i]] - mv) : 0.0f;
    } else {
      const double mn = a.par[at + (pres[i] ? off[i] : 0)];
      s.d[i] = pres[i] ? (float)(mn - mv) : 0.0f;
    }
    d0 = pres[i] ? s.d[i] : d0;
    s.first = pres[i] ? i : s.first;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) s.d[i] = pres[i] ? s.d[i] : DIFF ? d0 : __builtin_nanf("");
  const int own = lane & 3;
  const bool has = own == 0 ? pres[0] : own == 1 ? pres[1] : own == 2 ? pres[2] : pres[3];
  const int n = has ? own : DIFF ? s.first : 4;
  const double* L = a.par + a.ps + at;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if constexpr (DIFF) {
      const double l = k <= n && n < 4 ? L[(int64_t)(n * (n + 1) / 2 + k) * a.ps] : 0.0;
      s.row[k] = (float)((l - L[(int64_t)(10 + k) * a.ps]) * (double)kDeviateScale);
    } else {
      const bool in = k <= n && n < 4;
      const float l = (float)L[(int64_t)(in ? n * (n + 1) / 2 + k : 0) * a.ps];
      s.row[k] = in ? l : 0.0f;
    }
  }
  s.L44 = (float)L[14 * a.ps];
}

__device__ __forceinline__ f32x4 stencil_values(const MvgStencil& s, const float (&z)[4]) {
  f32x4 r = s.d;
#pragma unroll
  for (int k = 0; k < 4; ++k) r = __builtin_amdgcn_mfma_f32_4x4x1f32(s.row[k], z[k], r, 0, 0, 0);
  return r;
}

__device__ __forceinline__ float min4(const f32x4& v) {
  return __builtin_fminf(__builtin_fminf(__builtin_fminf(v[0], v[1]), v[2]), v[3]);
}
__device__ __forceinline__ float max4(const f32x4& v) {
  return __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(v[0], v[1]), v[2]), v[3]);
}

// One wave owns V vertices and takes the samples i = lane, lane + 64, ... of
// each: the first rounds of their Philox blocks, as far as they depend on the
// sample alone, are formed once (500^2 x 2000, V = 1: 1.71 ms, 2: 1.61, 4:
// 1.73).
//
// Bound by vector issue: 105 instructions a sample, 36 of them the generator's,
// ten transcendental (eight cycles each).  500^2 x 2000: 1.71 -> 1.53 ms.  With q the upper tail of |r|,
// Phi(r) = [r >= 0] - copysign(q, r): the first part is counted by the scalar
// unit, and q is summed with its full relative precision.
//
// VEC: the generator's keys in vector registers, which costs a wave as much as some
// 150 samples gain (500^2, conditional estimator, in vector / in scalar registers: 64 samples 148 /
// 109 us, 128 167 / 147, 256 238 / 238, 320 279 / 286; 64 hits 158 / 122).
template <int V, bool HIT, bool VEC>
__global__ __launch_bounds__(256) void k_mvg_fwd(MvgArgs a) {
  const int lane = threadIdx.x & 63;
  const int v0 = __builtin_amdgcn_readfirstlane((blockIdx.x * 4 + (threadIdx.x >> 6)) * V);
  const int nv = a.H * a.W;
  if (v0 >= nv) return;
  const PhiloxKeys keys = philox_keys<VEC>(a.k0, a.k1);
  MvgStencil s[V];
  float inv[V], invm[V], L4[HIT ? V : 1][4];
  double qmin[V], qmax[V];
  int nmin[V], nmax[V];
#pragma unroll
  for (int u = 0; u < V; ++u) {
    load_stencil<!HIT>(a, min(v0 + u, nv - 1), lane, s[u]);
    if constexpr (HIT) {
      const int v = min(v0 + u, nv - 1), y = v / a.W;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        L4[u][k] = (float)a.par[(int64_t)(11 + k) * a.ps + (int64_t)y * a.rs + (v - y * a.W)];
    }
    // r in upper_tail's scale; without neighbours both rows' extremes are +inf
    // and both estimates 1
    inv[u] = float(kTailScale) / s[u].L44;
    invm[u] = s[u].first < 4 ? -inv[u] : inv[u];
    qmin[u] = qmax[u] = 0.0;
    nmin[u] = nmax[u] = 0;
  }
  // (in a vector register, for the full-rate form)
  uint32_t sign = 0x80000000u;
  asm volatile("" : "+v"(sign));
  const auto add = [&](float r, bool on, int& n, double& q) {
    // copysign(q, r) in one full-rate instruction (q >= 0, or NaN)
    const float t = __builtin_bit_cast(
        float, __builtin_amdgcn_bitop3_b32(__builtin_bit_cast(uint32_t, upper_tail7(r)),
                                           __builtin_bit_cast(uint32_t, r), sign, 0xF8));
    n += __popcll(__ballot(on && __builtin_bit_cast(int, r) >= 0));
    q += (double)(on ? t : 0.0f);
  };
  const auto sample = [&](int i, bool on) {
    float z[V][4];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      uint32_t c[4] = {(uint32_t)i, (uint32_t)(v0 + u), a.fid, 0u};
      philox(c, keys);
      if constexpr (HIT) {
        box_muller(u24(c[0]), u24(c[1]), z[u][0], z[u][1]);
        box_muller(u24(c[2]), u24(c[3]), z[u][2], z[u][3]);
      } else {
        box_muller_scaled(u24(c[0]), u24(c[1]), z[u][0], z[u][1]);
        box_muller_scaled(u24(c[2]), u24(c[3]), z[u][2], z[u][3]);
      }
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const f32x4 x = stencil_values(s[u], z[u]);
      float lo = min4(x), hi = max4(x);
      if constexpr (HIT) {
        uint32_t c1[4] = {(uint32_t)i, (uint32_t)(v0 + u), a.fid, 1u};
        philox(c1, keys);
        float z4, z5;
        box_muller(u24(c1[0]), u24(c1[1]), z4, z5);
        const float cm = fmaf(L4[u][3], z[u][3],
                              fmaf(L4[u][2], z[u][2], fmaf(L4[u][0], z[u][0], L4[u][1] * z[u][1])));
        const float xv = fmaf(s[u].L44, z4, cm);
        // no neighbour, or none that is not NaN: +-inf
        lo = __builtin_fminf(lo, __builtin_inff());
        hi = __builtin_fmaxf(hi, -__builtin_inff());
        nmin[u] += __popcll(__ballot(on && xv < lo));
        nmax[u] += __popcll(__ballot(on && xv > hi));
      } else {
        add(lo * inv[u], on, nmin[u], qmin[u]);
        add(hi * invm[u], on, nmax[u], qmax[u]);
      }
    }
  };
  const int full = a.ns & ~63;
  for (int i0 = 0; i0 < full; i0 += 64) sample(i0 + lane, true);
  if (full < a.ns) sample(full + lane, full + lane < a.ns);
#pragma unroll
  for (int u = 0; u < V; ++u) {
    double t = 0.0;
    if constexpr (!HIT) {
      // lanes 0..31: minimum, 32..63: maximum
      t = pair_sum<32>(qmin[u], qmax[u]);
      t = row_sum(pair_sum<16>(t, t));
    }
    if (v0 + u < nv && (lane & 31) == 0) {
      const int v = v0 + u, y = v / a.W, x = v - y * a.W;
      (lane ? a.pmax : a.pmin)[(int64_t)y * a.rs + x] =
          (float)(((double)(lane ? nmax[u] : nmin[u]) - t) / (double)a.ns);
    }
  }
}

// Pathwise derivative of the conditional estimator.  With n* the argmin,
// r = (x_n* - c)/L44:  dr/dmu_n* = 1/L44, dr/dmu_v = -1/L44,
// dr/dL_n*j = z_j/L44, dr/dL_4j = -z_j/L44 (j<4), dr/dL44 = -r/L44; the
// maximum mirrors it.  L is local to the stencil (written directly); the
// mean plane is shared by five stencils, so its per-stencil partials go to a
// workspace and a second kernel gathers them.
//
// Bound by vector issue: 138 instructions a sample, and about 400 a wave before
// and after them (512^2 x 1000: 1.04 -> 1.01 ms; the 20 sums over the wave took
// six shuffles each before, now four values share a register after two).
//
// A chain of FP32 sums per lane, so the order and the rounding of every
// operation of a sample are part of the result.
__global__ __launch_bounds__(256) void k_mvg_bwd(MvgArgs a) {
  const int lane = threadIdx.x & 63;
  const int v = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (v >= a.H * a.W) return;
  const int y = v / a.W, x = v - y * a.W;
  const PhiloxKeys keys = philox_keys(a.k0, a.k1);
  MvgStencil s;
  load_stencil<false>(a, v, lane, s);
  const int64_t at = (int64_t)y * a.rs + x;
  float L4[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) L4[k] = (float)a.par[(int64_t)(11 + k) * a.ps + at];
  const float iL44 = 1.0f / s.L44;
  const float gmn = a.gmin[at] * iL44, gmx = a.gmax[at] * iL44;
  // sums 0..4: mean of v, e, n, w, s; 5 + k: entry k of L
  float acc[20];
#pragma unroll
  for (int k = 0; k < 20; ++k) acc[k] = 0.f;
  const auto sample = [&](int i, bool on) {
    uint32_t c0[4] = {(uint32_t)i, (uint32_t)v, a.fid, 0u};
    philox(c0, keys);
    float z[4];
    box_muller(u24(c0[0]), u24(c0[1]), z[0], z[1]);
    box_muller(u24(c0[2]), u24(c0[3]), z[2], z[3]);
    const f32x4 xn = stencil_values(s, z);
    const float cm = fmaf(L4[3], z[3], fmaf(L4[2], z[2], fmaf(L4[0], z[0], L4[1] * z[1])));
    const float lo = min4(xn), hi = max4(xn);
    const float rmin = (lo - cm) * iL44, rmax = (cm - hi) * iL44;
    const float px = phi_pdf(rmax);
    const float gm = on ? gmn * phi_pdf(rmin) : 0.f, gx = on ? gmx * px : 0.f;
    const float c4 = on ? fmaf(gmx, px, -gm) : 0.f;
    // the first neighbour that attains the extreme takes it
    float cr[4], rm = gm, rx = gx;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const bool im = xn[r] == lo, ix = xn[r] == hi;
      cr[r] = (im ? rm : 0.f) - (ix ? rx : 0.f);
      rm = im ? 0.f : rm;
      rx = ix ? 0.f : rx;
    }
    cr[3] = rm - rx;
    acc[0] += c4;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[1 + r] += cr[r];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int k = 0; k <= r; ++k) acc[5 + r * (r + 1) / 2 + k] = fmaf(cr[r], z[k], acc[5 + r * (r + 1) / 2 + k]);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[15 + j] = fmaf(c4, z[j], acc[15 + j]);
    acc[19] -= on ? fmaf(gx, rmax, gm * rmin) : 0.f;
  };
  // The first neighbour keeps both extremes if its values are NaN; without
  // neighbours the estimate is the constant 1.
  bool nan = false;
  const float any = ((s.d[0] + s.d[1]) + (s.d[2] + s.d[3])) + ((s.row[0] + s.row[1]) + (s.row[2] + s.row[3]));
  if (__ballot(any != any)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bool is = s.d[r] != s.d[r];
#pragma unroll
      for (int k = 0; k <= r; ++k) {
        const float l = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s.row[k]), r));
        is = is || l != l;
      }
      nan = nan || (s.first == r && is);
    }
  }
  if (nan) {
    const float bad = __builtin_nanf("");
    acc[0] = bad;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (s.first != r) continue;
      acc[1 + r] = bad;
#pragma unroll
      for (int k = 0; k <= r; ++k) acc[5 + r * (r + 1) / 2 + k] = bad;
    }
#pragma unroll
    for (int k = 15; k < 20; ++k) acc[k] = bad;
  } else if (s.first < 4) {
    const int full = a.ns & ~63;
    for (int i0 = 0; i0 < full; i0 += 64) sample(i0 + lane, true);
    if (full < a.ns) sample(full + lane, full + lane < a.ns);
  }
  // 20 sums over the wave, four to a register: row q of register m holds sum
  // 4 m + {0, 2, 1, 3}[q]
  const double inv_ns = 1.0 / (double)a.ns;
  const int64_t plane = (int64_t)a.H * a.W;
  const int q = lane >> 4, slot = (q & 1) * 2 + (q >> 1);
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const double p0 = pair_sum<32>((double)acc[4 * m], (double)acc[4 * m + 1]);
    const double p1 = pair_sum<32>((double)acc[4 * m + 2], (double)acc[4 * m + 3]);
    const double t = row_sum(pair_sum<16>(p0, p1)) * inv_ns;
    const int k = 4 * m + slot;
    if ((lane & 15) == 0) {
      if (k < 5)
        a.jmu[k * plane + v] = t;
      else
        a.grad[(int64_t)(k - 4) * a.ps + at] = t;
    }
  }
}

// grad_mu(u) = J_v(u) + J_w(east) + J_e(west) + J_s(north) + J_n(south)
__global__ __launch_bounds__(256) void k_mvg_gather(MvgArgs a) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t plane = (int64_t)a.H * a.W;
  if (id >= plane) return;
  const int y = (int)(id / a.W), x = (int)(id - (int64_t)y * a.W);
  double g = a.jmu[id];
  if (x + 1 < a.W) g += a.jmu[3 * plane + id + 1];
  if (x > 0) g += a.jmu[1 * plane + id - 1];
  if (y > 0) g += a.jmu[4 * plane + id - a.W];
  if (y + 1 < a.H) g += a.jmu[2 * plane + id + a.W];
  a.grad[(int64_t)y * a.rs + x] = g;
}

__global__ __launch_bounds__(256) void k_philox_raw(int64_t n, const uint32_t* ctr, uint32_t k0, uint32_t k1,
                                                  uint32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  uint32_t c[4] = {ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]};
  philox(c, philox_keys(k0, k1));
#pragma unroll
  for (int k = 0; k < 4; ++k) out[4 * i + k] = c[k];
}

// two vertices per wave once that still leaves four waves per SIMD
constexpr int64_t kMvgPairVertices = 8192;
// samples from which on the generator's keys are worth vector registers
constexpr int kMvgVectorKeys = 256;

template <bool HIT, bool VEC>
void launch_fwd(const MvgArgs& a, bool two, dim3 grid, hipStream_t st) {
  if (two)
    hipLaunchKernelGGL((k_mvg_fwd<2, HIT, VEC>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((k_mvg_fwd<1, HIT, VEC>), grid, dim3(256), 0, st, a);
}

MvgArgs make_args(const Field& f, const double* params) {
  MvgArgs a{};
  a.par = params;
  a.H = f.H;
  a.W = f.W;
  a.ns = f.ns;
  a.rs = f.rs;
  a.ps = f.plane();
  a.k0 = (uint32_t)f.seed;
  a.k1 = (uint32_t)(f.seed >> 32);
  a.fid = f.fid;
  return a;
}

}  // namespace

hipError_t mvg_forward(const Field& f, const double* params, float* pmin, float* pmax, hipStream_t st) {
  MvgArgs a = make_args(f, params);
  a.pmin = pmin;
  a.pmax = pmax;
  const int64_t nv = (int64_t)f.H * f.W;
  const bool two = nv >= kMvgPairVertices;
  const dim3 grid((unsigned)((nv + (two ? 8 : 4) - 1) / (two ? 8 : 4)));
  if (f.ns >= kMvgVectorKeys)
    f.est == CP_MC_HIT ? launch_fwd<true, true>(a, two, grid, st) : launch_fwd<false, true>(a, two, grid, st);
  else
    f.est == CP_MC_HIT ? launch_fwd<true, false>(a, two, grid, st) : launch_fwd<false, false>(a, two, grid, st);
  return hipGetLastError();
}

hipError_t mvg_backward(const Field& f, const double* params, const float* gmin, const float* gmax, double* grad,
                        hipStream_t st, const Scratch& scr) {
  MvgArgs a = make_args(f, params);
  a.gmin = gmin;
  a.gmax = gmax;
  a.grad = grad;
  const int64_t nv = (int64_t)f.H * f.W;
  void* ws = nullptr;
  hipError_t e = adjoint_scratch(sizeof(double) * 5 * (size_t)nv, st, scr, &ws);
  if (e != hipSuccess) return e;
  a.jmu = static_cast<double*>(ws);
  hipLaunchKernelGGL(k_mvg_bwd, dim3((unsigned)((nv + 3) / 4)), dim3(256), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mvg_gather, dim3((unsigned)((nv + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t philox_raw(int64_t n, const uint32_t* ctr, uint64_t seed, uint32_t* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_philox_raw, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, ctr, (uint32_t)seed,
                     (uint32_t)(seed >> 32), out);
  return hipGetLastError();
}

}  // namespace cp
