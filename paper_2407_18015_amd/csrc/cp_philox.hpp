// cp_philox.hpp -- Philox4x32-10 (Salmon et al., "Parallel random numbers:
// as easy as 1, 2, 3", SC'11): a counter-based generator, so every sample's
// random words are a pure function of (counter, key) and results do not
// depend on the launch configuration.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cp {

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

// a ^ b ^ c in one instruction (the compiler makes two v_xor_b32 of it, twenty
// of the hundred-odd instructions of a block): Gaussian Monte Carlo forward at
// 500^2 x 2000 samples 1.90 -> 1.70 ms, adjoint at 512^2 x 1000 1.12 -> 1.04.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The key words of the ten rounds.  In vector registers: gfx950 issues the
// plain FP32 and 32-bit logical instructions every two cycles, but every four
// where one operand is a scalar register.  The first two rounds' words are
// mostly wave-uniform in the samplers and stay with the scalar unit.  VEC =
// false (where registers are short): all in scalar registers.
struct PhiloxKeys {
  uint32_t a[10], b[10];
};
template <bool VEC = true>
__device__ __forceinline__ PhiloxKeys philox_keys(uint32_t k0, uint32_t k1) {
  PhiloxKeys k;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    k.a[r] = k0 + (uint32_t)r * kPhiloxW0;
    k.b[r] = k1 + (uint32_t)r * kPhiloxW1;
    if (VEC && r >= 2) asm volatile("" : "+v"(k.a[r]), "+v"(k.b[r]));
  }
  return k;
}

// Ten rounds on the counter c in place.  Each round's two 32 x 32 -> 64-bit
// products are formed whole (one v_mad_u64_u32 each rather than a high and a
// low multiply: a third faster on gfx950).
__device__ __forceinline__ void philox(uint32_t c[4], const PhiloxKeys& k) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)kPhiloxM0 * c[0], p1 = (uint64_t)kPhiloxM1 * c[2];
    const uint32_t h1 = (uint32_t)(p1 >> 32), h0 = (uint32_t)(p0 >> 32);
    const uint32_t n0 = r < 2 ? h1 ^ c[1] ^ k.a[r] : xor3(h1, c[1], k.a[r]);
    const uint32_t n2 = r < 2 ? h0 ^ c[3] ^ k.b[r] : xor3(h0, c[3], k.b[r]);
    c[0] = n0;
    c[1] = (uint32_t)p1;
    c[2] = n2;
    c[3] = (uint32_t)p0;
  }
}

// Uniform in (0, 1] from the top 24 bits of a word: ((r >> 8) + 1/2) 2^-24,
// exact in FP64; in FP32 the values above 1/2 need a 25th bit and round to
// the nearest even multiple of 2^-24 (by at most 2^-25; the top one to 1).
template <typename T>
__device__ __forceinline__ T u24_of(uint32_t r) {
  return (T(r >> 8) + T(0.5)) * T(5.9604644775390625e-8);
}

}  // namespace cp
