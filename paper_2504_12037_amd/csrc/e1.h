// E_1(s_W) = -sum_{W-W edges} J s_i s_j - sum_{i in W} h_i s_i (Eq. 4) of a
// block of samples, one per thread.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.h"
#include "wave.h"

namespace tnvan {

constexpr int kE1Threads = 256;
struct E1Term {
  double J;
  int32_t a, b;   // spins; b < 0: a field
};

// The terms go through LDS, kE1Threads at a time (a thread that reads them
// one by one waits for memory at each), and the sample's spins are a bit mask
// up to 128 of them.  Four partial sums.  Measured on three 16x16 lattices,
// 8192 samples each: 13.5 us term by term in a launch of its own, and beside
// the unary factors (chain.hip) ln Z_R and E_1 together 54 -> 40 us.
__device__ inline void e1_block(const E1Args &a, int q, int64_t b0, E1Term *terms) {
  const MadeInst mi = a.mi[q];
  if (b0 >= mi.B) return;   // uniform over the block
  const InstDesc D = a.inst[q];
  const int32_t *wa = a.ww_a + D.ww_off, *wb = a.ww_b + D.ww_off;
  const double *wJ = a.ww_J + D.ww_off, *hW = a.hW + a.hw_off[q];
  const int64_t b = b0 + threadIdx.x, bs = b < mi.B ? b : b0;
  const int8_t *s = a.spins + mi.spin_off + bs * mi.n;
  const bool bits = mi.n <= 128;
  const SpinBits sb = bits ? load_bits_row(s, mi.n) : SpinBits{{0u, 0u, 0u, 0u}};
  const int total = D.n_ww + mi.n;
  double e[4] = {0, 0, 0, 0};
  for (int k0 = 0; k0 < total; k0 += kE1Threads) {
    const int k = k0 + threadIdx.x;
    __syncthreads();
    E1Term t{0.0, 0, -1};
    if (k < D.n_ww) t = E1Term{wJ[k], wa[k], wb[k]};
    else if (k < total) t = E1Term{hW[k - D.n_ww], k - D.n_ww, -1};
    terms[threadIdx.x] = t;
    __syncthreads();
    const int m = total - k0 < kE1Threads ? total - k0 : kE1Threads;
    auto sum = [&](auto negative) {
      for (int i = 0; i < m; i += 4)   // (past the terms: zero couplings)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const E1Term x = terms[(i + u) & (kE1Threads - 1)];
          const double v = negative(x) ? -x.J : x.J;
          if (i + u < m) e[u] -= v;
        }
    };
    if (mi.n <= 32)
      sum([&](const E1Term &x) { return (((sb.m[0] >> x.a) ^ (x.b < 0 ? 0u : sb.m[0] >> (x.b & 31))) & 1u) != 0; });
    else if (bits)
      sum([&](const E1Term &x) { return (sb.sigma(x.a) * (x.b < 0 ? 1.f : sb.sigma(x.b))) < 0.f; });
    else
      sum([&](const E1Term &x) { return s[x.a] * (x.b < 0 ? 1 : s[x.b]) < 0; });
  }
  if (b < mi.B) a.e1[mi.sample_off + b] = (e[0] + e[1]) + (e[2] + e[3]);
}

}  // namespace tnvan
