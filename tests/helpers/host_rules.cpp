// host_rules.cpp -- host-only build of the library's dispatch rules (test
// infrastructure; built by tests/test_host_rules.py with the HIP compiler's
// host pass only).
//
//   host_rules blocks <samples>
//     Philox blocks of four samples of the semianalytical estimator.
//   host_rules thread <samples> <bins> <bytes of an element> <vertices>
//     whether that estimator gives a vertex to a thread (1) or a wave (0).
//   host_rules quotients <dtype> <log2 of the ranges' scale> <seed>
//     of a million ranges in [1, 2) times the scale and members within them: how
//     many of BinOf's quotients of 2^-36 and more differ from the division, and
//     how many of the bins of 32 do (dtype: 0 FP32, 1 FP64).
//   host_rules gather <dtype> <H> <W> <bins> <row stride> <seed>
//     the histogram adjoint's gather of a random workspace, vertex by vertex and
//     by vectors (as the library launches them for a width that holds one): rows
//     summed on chip (1) or not (0), then how many values differ in any bit.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "cp_fit.hpp"
#include "cp_hist_bwd.hpp"
#include "cp_internal.hpp"

template <typename T>
static void quotients(int scale, unsigned seed) {
  std::mt19937_64 rng(seed);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  long wrong = 0, bins = 0;
  for (int i = 0; i < 1000000; ++i) {
    const T range = (T)std::ldexp(1.0 + u(rng), scale);
    // quotients over 36 binades, every other one beside an edge of the 32 bins
    T a = (T)((double)range * std::exp2(-36.0 * u(rng)));
    if (i & 1) a = std::nextafter((T)((double)range * (double)(rng() % 33) / 32.0), u(rng) < 0.5 ? T(0) : range);
    const cp::BinOf<T> b(T(0), range, 32);
    const volatile T d = a / range;
    const T q = d;
    wrong += q >= T(1.4551915228366852e-11) && b.quotient(a) != q;
    int j = (int)(q * T(32));
    j = j > 31 ? 31 : j;
    bins += b(a) != j;
  }
  std::printf("%ld %ld\n", wrong, bins);
}

template <typename T>
static int gather(int H, int W, int h, int rs, unsigned seed) {
  const int64_t plane = (int64_t)H * W, ps = (int64_t)H * rs;
  std::vector<T> J((size_t)(cp::hist_ws_planes(h) * plane)), a((size_t)((2 + h) * ps), T(0)), b = a;
  uint64_t r = seed * 2 + 1;
  for (T& v : J) {  // 24 bits of a linear congruential generator
    r = r * 6364136223846793005ull + 1442695040888963407ull;
    v = (T)(int32_t)(r >> 40) * T(1.0 / (1 << 23)) - T(1);
  }
  cp::FieldPtrs<T> f{};
  f.H = H;
  f.W = W;
  f.nb = h;
  f.rs = rs;
  f.ps = ps;
  f.grad = a.data();
  for (int64_t i = 0; i < plane + 3; ++i) cp::hist_gather_vertex<T>(f, J.data(), i);
  f.grad = b.data();
  const int64_t groups = cp::gather_groups(H, W, cp::gather_vec<T>());
  for (int64_t i = 0; i < groups + 3; ++i) cp::hist_gather_vec<T>(f, J.data(), i);
  long differ = 0;
  for (size_t i = 0; i < a.size(); ++i) differ += std::memcmp(&a[i], &b[i], sizeof(T)) != 0;
  std::printf("%d %ld\n", cp::hist_row_sums(h, sizeof(T), plane) ? 1 : 0, differ);
  return 0;
}

int main(int argc, char** argv) {
  if (argc == 3 && !std::strcmp(argv[1], "blocks")) {
    std::printf("%d\n", cp::semi_blocks(std::atoi(argv[2])));
    return 0;
  }
  if (argc == 6 && !std::strcmp(argv[1], "thread")) {
    std::printf("%d\n", cp::semi_by_thread(std::atoi(argv[2]), std::atoi(argv[3]), (size_t)std::atoi(argv[4]),
                                           std::atoll(argv[5])));
    return 0;
  }
  if (argc == 5 && !std::strcmp(argv[1], "quotients")) {
    const int scale = std::atoi(argv[3]);
    const unsigned seed = (unsigned)std::atoi(argv[4]);
    std::atoi(argv[2]) ? quotients<double>(scale, seed) : quotients<float>(scale, seed);
    return 0;
  }
  if (argc == 8 && !std::strcmp(argv[1], "gather")) {
    int v[6];
    for (int i = 0; i < 6; ++i) v[i] = std::atoi(argv[2 + i]);
    return v[0] ? gather<double>(v[1], v[2], v[3], v[4], v[5]) : gather<float>(v[1], v[2], v[3], v[4], v[5]);
  }
  std::fprintf(stderr, "usage: see the head of this file\n");
  return 2;
}
