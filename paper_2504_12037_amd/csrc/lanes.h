// Register moves between the lanes of a 64-lane wave, no LDS traffic.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tnvan {

// Moves between the lanes of a wave by a power of two (register moves: DPP
// inside rows of 16, the row swaps beyond).
template <int CTRL>
__device__ inline uint32_t dpp32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, false);
}
// the value of lane ^ D
template <int D>
__device__ inline uint32_t xor32(uint32_t v) {
  if constexpr (D == 1) return dpp32<0xB1>(v);
  else if constexpr (D == 2) return dpp32<0x4E>(v);
  else if constexpr (D == 4) return dpp32<0x1B>(dpp32<0x141>(v));   // half-row mirror, quad mirror
  else if constexpr (D == 8) return dpp32<0x128>(v);                // rotate the row by 8
  else {
    // swap rows of one copy with rows of the other: one result keeps the
    // own row, the other holds the partner's, by the lane's half
    const auto p = D == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false)
                           : __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return p[0] ^ p[1] ^ v;
  }
}
template <int D, typename T>
__device__ inline T lane_xor(T v) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, xor32<D>(__builtin_bit_cast(uint32_t, v)));
  } else {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    return __builtin_bit_cast(T, ((unsigned long long)xor32<D>((uint32_t)(u >> 32)) << 32) |
                                     (unsigned long long)xor32<D>((uint32_t)u));
  }
}
// butterfly over the lane distances LO, 2 LO, ... below HI
template <int LO, int HI, typename T, typename F>
__device__ inline T lanes_fold(T v, F f) {
  if constexpr (LO < HI) return lanes_fold<2 * LO, HI>(f(v, lane_xor<LO>(v)), f);
  else return v;
}
template <int LO, int HI, typename T>
__device__ inline T lanes_sum(T v) {
  return lanes_fold<LO, HI>(v, [](T a, T b) { return a + b; });
}
template <int LO, int HI, typename T>
__device__ inline T lanes_max(T v) {
  return lanes_fold<LO, HI>(v, [](T a, T b) { return b > a ? b : a; });
}

}  // namespace tnvan
