// The power-of-two rescale of messages in the level and wide-step kernels:
// one rule, on which ln Z_R's same bits in both rest (contract.hip's clamps
// the exponent for its grouped steps; below a largest entry of 2^2, as
// here, the two agree).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tnvan {

template <typename real> struct MsgBits;
template <> struct MsgBits<float> {
  using U = uint32_t;
  __device__ static U bits(float x) { return __float_as_uint(x); }
  // e with max 2^-e in [0.5, 1)
  __device__ static int expo(U b) { return (int)((b >> 23) & 0xffu) - 126; }
  // 2^-e
  __device__ static float scale(U b) { return __uint_as_float((253u << 23) - (b & 0x7f800000u)); }
};
template <> struct MsgBits<double> {
  using U = unsigned long long;
  __device__ static U bits(double x) { return (U)__double_as_longlong(x); }
  __device__ static int expo(U b) { return (int)((b >> 52) & 0x7ffull) - 1022; }
  __device__ static double scale(U b) {
    return __longlong_as_double((long long)((2045ull << 52) - (b & (0x7ffull << 52))));
  }
};

}  // namespace tnvan
