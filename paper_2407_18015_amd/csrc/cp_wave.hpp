// cp_wave.hpp -- sums over the 64 lanes of a wave (FP64), for the kernels that
// give a wave a vertex and its lanes the samples.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cp {

// sum over the 16 lanes of a row, in every lane of it
__device__ __forceinline__ double row_sum(double v) {
#define CP_ROW_STEP(CTRL)                                                                               \
  {                                                                                                     \
    const uint64_t b = __builtin_bit_cast(uint64_t, v);                                                 \
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);               \
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);       \
    v += __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);                                           \
  }
  CP_ROW_STEP(0xB1)   // quad_perm: lane ^ 1
  CP_ROW_STEP(0x4E)   // quad_perm: lane ^ 2
  CP_ROW_STEP(0x141)  // row_half_mirror
  CP_ROW_STEP(0x140)  // row_mirror
#undef CP_ROW_STEP
  return v;
}

// Two sums at once: lanes of the lower half (SWAP 32) or of the even rows
// (SWAP 16) receive a's partial sums, the others b's.
template <int SWAP>
__device__ __forceinline__ double pair_sum(double a, double b) {
  const uint64_t p = __builtin_bit_cast(uint64_t, a), q = __builtin_bit_cast(uint64_t, b);
  uint64_t r[2] = {0, 0};
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const uint32_t x = (uint32_t)(p >> 32 * w), y = (uint32_t)(q >> 32 * w);
    const auto t = SWAP == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                              : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    r[0] |= (uint64_t)(uint32_t)t[0] << 32 * w;
    r[1] |= (uint64_t)(uint32_t)t[1] << 32 * w;
  }
  return __builtin_bit_cast(double, r[0]) + __builtin_bit_cast(double, r[1]);
}

}  // namespace cp
