// Wide steps of a single-spin elimination program (output scopes of 12 to 20
// spins): one step over the whole chip.
//
// A graph of width 18 holds nearly all its work in a few tens of steps of
// 2^12 to 2^18 entries per sample, while a training batch of it has a few
// tens of samples: a workgroup per sample leaves most of the chip idle.  So
// the steps run as launches of their own over (workgroups of 2^11 entries,
// samples), independent steps together, with the light steps between them in
// the level kernel (sweep.hip, one workgroup per sample).  The schedule
// (sweep.h) picks which output bits a workgroup's entries cover.
//
// What bounds it is memory: the forward step reads each input entry pair and
// writes each output entry once, the reverse step reads the output's and the
// inputs' entries and writes the inputs' once.  The joint weights stay in
// LDS: the sums over the output bits that an input lacks are taken there,
// and only where those bits exceed the workgroup's are partial sums written
// (a second launch adds them).  The arena is [sample][entry], so a wave's
// accesses are runs of at least 32 entries.
//
// Measured on a 1000-spin random 3-regular graph at width 18 (40 wide steps,
// 2.6 M entries a sample), 64 samples, FP32: ln Z_R and its adjoint through
// autograd 50.4 -> 2.76 ms against the step-by-step kernel; the wide steps
// take 0.49 ms forward and 1.03 ms in reverse (2.7 and 2.6 TB/s over the
// entries they read and write), the light steps 0.62 ms in all.
//
// The arithmetic per entry is that of the step-by-step kernel in
// contract.hip, in the same order: ln Z_R is the same bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lanes.h"
#include "launch.h"
#include "msgbits.h"
#include "sweep.h"
#include "uload.h"

namespace tnvan {

namespace {

constexpr int kT = kWideThreads, kR = kWideRegs;

// the workgroup's step of the group and its place among the step's
// workgroups
__device__ inline const WideStep *find_step(const WideStep *steps, int w0, int &blk) {
  const WideStep *ws = steps + w0;
  for (;;) {
    const int n = 1 << (uload(&ws->w) - kWideChunk);
    if (blk < n) return ws;
    blk -= n;
    ++ws;
  }
}

// p0, p1 [r] (spin +1 and -1) times the transfer factors and unary factors
// of entries o[r], then the inputs' entries in turn; kEnd: the last product
// of spin -1 is added to the finished one of spin +1 (into p0).  A step with
// a table starts from T phi and rounds that last product and sum once, one
// without from phi times the edges' factors, each product and the sum
// rounded.
template <typename real, bool kEnd>
__device__ inline void wide_products(const WideArgs<real> &a, const WideStep *ws, int blk,
                                     const real *arena, const typename MsgBits<real>::U *mx,
                                     const real *phi, const int (&o)[kR], real (&p0)[kR],
                                     real (&p1)[kR]) {
  const int w = uload(&ws->w), n_in = uload(&ws->n_in), gpos = uload(&ws->gpos);
  const int64_t tpos = uload(&ws->t_off);
  const real ph0 = phi[2 * gpos], ph1 = phi[2 * gpos + 1];
  if (tpos >= 0) {
    const real *T0 = a.T + tpos, *T1 = T0 + ((int64_t)1 << w);
    real t0[kR], t1[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      t0[r] = T0[o[r]];
      t1[r] = T1[o[r]];
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      p0[r] = kEnd ? t0[r] * ph0 : p0[r] * t0[r] * ph0;
      p1[r] = kEnd ? t1[r] * ph1 : p1[r] * t1[r] * ph1;
    }
  } else {
    real t0[kR], t1[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) t0[r] = t1[r] = 1;
    const int n_e = uload(&ws->n_edge), e0 = uload(&ws->edge_off);
    for (int e = 0; e < n_e; ++e) {
      // J s_x s_o > 0: factor 1, else exp(-2 beta |J|); bit 1 <=> spin -1
      const int eb = uload(&a.edges[e0 + e].bv);
      const real es = uload(a.esmall + e0 + e);
      const bool pos = es > (real)0;
      const real sm = pos ? es : -es;
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        const int ob = (o[r] >> eb) & 1;
        t0[r] *= ((ob == 0) == pos) ? (real)1 : sm;
        t1[r] *= ((ob == 1) == pos) ? (real)1 : sm;
      }
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      p0[r] = kEnd ? ph0 * t0[r] : p0[r] * ph0 * t0[r];
      p1[r] = kEnd ? ph1 * t1[r] : p1[r] * ph1 * t1[r];
    }
  }
  for (int k = 0; k < n_in; ++k) {
    const WideInput *in = ws->in + k;
    const int32_t *tab = a.tab + uload(&in->idx);
    const int base = uload(&in->off) + (tab[threadIdx.x] | uload(tab + kT + kR + blk));
    const int xs = 1 << uload(&in->xbit);
    const real sc = MsgBits<real>::scale(mx[uload(&in->step)]);
    real m0[kR], m1[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const real *m = arena + (base + uload(tab + kT + r));
      m0[r] = m[0];
      m1[r] = m[xs];
    }
    if (kEnd && k == n_in - 1) {
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        p0[r] *= m0[r] * sc;
        if (tpos >= 0) {
          p0[r] = __builtin_fma(p1[r], m1[r] * sc, p0[r]);
        } else {
          p1[r] *= m1[r] * sc;
          // (a rounded product: not one operation with the sum)
          asm volatile("" : "+v"(p1[r]));
          p0[r] += p1[r];
        }
      }
    } else {
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        p0[r] *= m0[r] * sc;
        p1[r] *= m1[r] * sc;
      }
    }
  }
}

template <typename real>
__device__ inline void wide_entries(const WideArgs<real> &a, const WideStep *ws, int blk, int (&o)[kR]) {
  const int32_t *tab = a.tab + uload(&ws->out);
  const int base = tab[threadIdx.x] | uload(tab + kT + kR + blk);
#pragma unroll
  for (int r = 0; r < kR; ++r) o[r] = base | uload(tab + kT + r);
}

// forward: out[o] = sum_x T[x, o] phi[x] prod_k m_k
template <typename real>
__global__ __launch_bounds__(kT) void wide_fwd_kernel(WideArgs<real> a) {
  using FB = MsgBits<real>;
  using U = typename FB::U;
  __shared__ U sh[kT / 64];
  real *mem = a.mem + (int64_t)blockIdx.y * a.stride;
  U *mx = reinterpret_cast<U *>(mem + a.state);
  int blk = blockIdx.x;
  const WideStep *ws = find_step(a.steps, a.w0, blk);
  int o[kR];
  wide_entries(a, ws, blk, o);
  real p0[kR], p1[kR];
  wide_products<real, true>(a, ws, blk, mem, mx, mem + a.state + a.n_steps, o, p0, p1);
  real *out = mem + uload(&ws->off);
  U lmax = 0;   // (positive numbers compare as their bits)
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    out[o[r]] = p0[r];
    const U b = FB::bits(p0[r]);
    lmax = b > lmax ? b : lmax;
  }
  lmax = lanes_max<1, 64>(lmax);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = lmax;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 1; k < kT / 64; ++k) lmax = sh[k] > lmax ? sh[k] : lmax;
    atomicMax(mx + uload(&ws->step), lmax);
  }
}

// reverse: joint weights c(o, x) = rho[o] 2^-e T[x, o] phi[x] prod_k m_k in
// LDS, their sums over o (plain, and signed by each edge's output spin), and
// each input's rho: c summed over the output bits not in its scope, over its
// scaled entry
template <typename real>
__global__ __launch_bounds__(kT) void wide_bwd_kernel(WideArgs<real> a) {
  using FB = MsgBits<real>;
  using U = typename FB::U;
  __shared__ real c[2 << kWideChunk];
  __shared__ real sums[(1 + kWideEdges) * (kT / 64)];
  real *mem = a.mem + (int64_t)blockIdx.y * a.stride;
  const U *mx = reinterpret_cast<const U *>(mem + a.state);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int blk = blockIdx.x;
  const WideStep *ws = find_step(a.steps, a.w0, blk);
  int o[kR];
  wide_entries(a, ws, blk, o);
  {
    real p0[kR], p1[kR];
    const real *out = mem + uload(&ws->off);
    const real sct = FB::scale(mx[uload(&ws->step)]);
#pragma unroll
    for (int r = 0; r < kR; ++r) p0[r] = out[o[r]];
#pragma unroll
    for (int r = 0; r < kR; ++r) p0[r] = p1[r] = p0[r] * sct;
    wide_products<real, false>(a, ws, blk, mem, mx, mem + a.state + a.n_steps, o, p0, p1);
    const int n_e = uload(&ws->n_edge), e0 = uload(&ws->edge_off);
    for (int k = 0; k <= n_e; ++k) {
      const int eb = k ? uload(&a.edges[e0 + k - 1].bv) : 31;
      real v = 0;
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        const real d = p0[r] - p1[r];
        v += ((o[r] >> eb) & 1) ? -d : d;
      }
      v = lanes_sum<1, 64>(v);
      if (lane == 0) sums[k * (kT / 64) + wave] = v;
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      c[tid + r * kT] = p0[r];
      c[(1 << kWideChunk) + tid + r * kT] = p1[r];
    }
  }
  __syncthreads();
  const int n_e = uload(&ws->n_edge), n_in = uload(&ws->n_in);
  if (tid <= n_e) {
    real v = 0;
#pragma unroll
    for (int k = 0; k < kT / 64; ++k) v += sums[tid * (kT / 64) + k];
    mem[a.red + uload(&ws->red) + blk * (1 + n_e) + tid] = v;
  }
  // (every read of an input's entries by this workgroup is behind the
  // barrier, and no other workgroup reads those it writes in place)
  for (int k = 0; k < n_in; ++k) {
    const WideInput *in = ws->in + k;
    const int freem = uload(&in->free), nf = __popc(freem), ns = kWideChunk - nf;
    const int32_t *idx = a.tab + uload(&in->idx), *dep = a.tab + uload(&in->dep);
    const int jb = uload(idx + kT + kR + blk), xs = 1 << uload(&in->xbit), part = uload(&in->part);
    const real sc = FB::scale(mx[uload(&in->step)]);
    real *dst = mem + uload(&in->off);
    // 2^lc lanes share a sum: each takes one pattern of the lowest lc free
    // bits and walks the others
    int lc = 8 - (ns + 1);
    lc = lc < 0 ? 0 : lc > 6 ? 6 : lc;
    lc = lc < nf ? lc : nf;
    int high = freem;
    for (int b = 0; b < lc; ++b) high &= high - 1;
    const int low = freem & ~high, nit = 1 << __popc(high);
    int row = 0;
    int64_t rowlen = 0;
    if (part >= 0) {
      row = uload(a.tab + uload(&in->row) + blk);
      rowlen = (int64_t)1 << uload(&in->bits);
    }
    for (int t = tid; t < 1 << (ns + 1 + lc); t += kT) {
      const int e = t >> lc, x = e >> ns;
      const uint32_t d = (uint32_t)dep[e & ((1 << ns) - 1)];
      int at = ((int)(d & ((1u << kWideChunk) - 1)) | (x << kWideChunk));
      const int j = jb | (int)(d >> kWideChunk) | (x ? xs : 0);
      for (int b = 0, m = low; b < lc; ++b, m &= m - 1)
        if ((t >> b) & 1) at |= m & -m;
      real m = 0;
      if (part < 0) m = dst[j];
      real s0 = 0, s1 = 0, s2 = 0, s3 = 0;
      int z = 0;
      if (nit >= 4) {
        for (int i = 0; i < nit; i += 4) {
          const int z1 = (z - high) & high, z2 = (z1 - high) & high, z3 = (z2 - high) & high;
          s0 += c[at | z];
          s1 += c[at | z1];
          s2 += c[at | z2];
          s3 += c[at | z3];
          z = (z3 - high) & high;
        }
      } else {
        for (int i = 0; i < nit; ++i) {
          s0 += c[at | z];
          z = (z - high) & high;
        }
      }
      real mu = (s0 + s1) + (s2 + s3);
      for (int sh = 1; sh < 1 << lc; sh <<= 1) mu += __shfl_xor(mu, sh, 64);
      if ((t & ((1 << lc) - 1)) == 0) {
        if (part < 0) {
          m *= sc;
          dst[j] = m > 0 ? mu / m : (real)0;
        } else {
          mem[a.part + part + row * rowlen + j] = mu;
        }
      }
    }
  }
}

// the rho of inputs whose sums were split over workgroups
template <typename real>
__global__ __launch_bounds__(kT) void wide_fin_kernel(WideArgs<real> a) {
  using FB = MsgBits<real>;
  using U = typename FB::U;
  real *mem = a.mem + (int64_t)blockIdx.y * a.stride;
  const U *mx = reinterpret_cast<const U *>(mem + a.state);
  int f = a.f1 - 1;
  while (f > a.f0 && uload(&a.fins[f].first) > (int)blockIdx.x) --f;
  const WideFin w = uload(a.fins + f);
  const int j = ((int)blockIdx.x - w.first) * kT + threadIdx.x;
  if (j >= 1 << w.nbits) return;
  const real *p = mem + a.part + w.part + j;
  real s[4] = {0, 0, 0, 0};
  int r = 0;
  for (; r + 4 <= w.rows; r += 4)
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] += p[(int64_t)(r + u) << w.nbits];
  for (; r < w.rows; ++r) s[0] += p[(int64_t)r << w.nbits];
  real *dst = mem + w.off + j;
  const real m = *dst * FB::scale(mx[w.step]);
  *dst = m > 0 ? ((s[0] + s[1]) + (s[2] + s[3])) / m : (real)0;
}

}  // namespace

template <typename real>
hipError_t launch_wide(const WideArgs<real> &a, const WideGroup &g, int n_samples, bool bwd,
                       hipStream_t st) {
  if (n_samples <= 0 || g.blocks <= 0) return hipSuccess;
  WideArgs<real> w = a;
  w.w0 = g.w0;
  w.f0 = g.f0;
  w.f1 = g.f1;
  // (samples beyond a launch's grid: further launches)
  for (int b = 0; b < n_samples; b += 65535) {
    const int n = std::min(65535, n_samples - b);
    w.mem = a.mem + (int64_t)b * a.stride;
    if (!bwd) {
      hipLaunchKernelGGL(wide_fwd_kernel<real>, dim3(g.blocks, n), dim3(kT), 0, st, w);
      continue;
    }
    hipLaunchKernelGGL(wide_bwd_kernel<real>, dim3(g.blocks, n), dim3(kT), 0, st, w);
    if (g.fblocks > 0)
      hipLaunchKernelGGL(wide_fin_kernel<real>, dim3(g.fblocks, n), dim3(kT), 0, st, w);
  }
  return hipGetLastError();
}

template hipError_t launch_wide<float>(const WideArgs<float> &, const WideGroup &, int, bool, hipStream_t);
template hipError_t launch_wide<double>(const WideArgs<double> &, const WideGroup &, int, bool, hipStream_t);

}  // namespace tnvan
