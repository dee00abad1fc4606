// Level kernels: single-spin elimination programs (random graphs) contracted
// level by level (Sec. 2, Eqs. 2-4), their adjoint, and the second-order jets
// of the magnetisation moments.
//
// A workgroup of up to eight waves takes a tile of S samples.  Each wave runs its
// own program (sweep.h) of units of a level's steps: E = 64 / S output
// entries times S samples per pass, samples fastest, so the arena is
// [entry][S] and a pass reads and writes runs of 64 words.  One barrier ends
// a forward level; a reverse level has two phases (joint weights; marginals
// and sums).
//
// What bounds it: the chain of dependent memory round trips down the
// elimination tree.  The forward arena (messages live at one time) stays in
// LDS where it fits; the adjoint keeps every message in device memory, its
// joint weights in LDS.  With enough tiles to fill the chip what bounds it
// is instruction issue, so a unit is kept lean: its record is one vector
// load of the wave, one record ahead, as are its lane word (the lane's
// gather index into every input) and first transfer factors; reductions are
// register moves.
//
// Measured against the step-by-step kernel (contract.hip; the jets: one
// thread per sample) on random 3-regular graphs at width 10, FP32: N = 256,
// 4096 samples, ln Z_R 489 -> 135 us, adjoint 2065 -> 719 us; jets of two
// N = 128 graphs, 2048 samples each, 13.7 -> 0.17 ms.
//
// The arithmetic per entry is that of the step-by-step kernel in
// contract.hip, in the same order, so ln Z_R is the same bit for bit at
// every tile size and in both kernels.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lanes.h"
#include "launch.h"
#include "msgbits.h"
#include "sweep.h"
#include "uload.h"

namespace tnvan {

namespace {

constexpr int kThreads = 64 * kSweepWaves;   // most

__device__ inline float sexp(float x) { return expf(x); }
__device__ inline double sexp(double x) { return exp(x); }

struct SLay {
  size_t mx, phi, fab, gs, M, C, red, scr, arena, end;
};
__host__ __device__ inline size_t up8(size_t x) { return (x + 7) & ~(size_t)7; }

// mode: 0 forward, 1 adjoint, 2 jets, 3 a segment between wide steps (its
// forward or its reverse part)
__host__ __device__ inline SLay sweep_layout(const InstDesc &D, const SweepInst &W, int S, int mode,
                                             bool global_arena, int rs) {
  SLay L{};
  size_t o = 0;
  L.mx = o;  o = up8(o + (size_t)D.n_steps * S * rs);
  L.phi = o; o = up8(o + (size_t)D.nr * 2 * S * rs);
  L.fab = o; o = up8(o + (size_t)D.nr * S * rs);
  if (mode == 1 || mode == 3) {
    L.gs = o;  o = up8(o + (size_t)S * rs);
    L.M = o;   o = up8(o + (size_t)D.nr * S * rs);
    L.C = o;   o = up8(o + (size_t)D.n_rr * rs);
    L.red = o; o = up8(o + (size_t)W.slots * S * rs);
    L.scr = o; o = up8(o + (size_t)W.scr * S * rs);
  }
  if (!global_arena) {
    L.arena = o;
    o = up8(o + (size_t)W.arena * (mode == 2 ? 3 : 1) * S * rs);
  }
  L.end = o;
  return L;
}

// A message entry: a number, or its jet in the uniform field (coefficients
// c0, c1, c2 stored [entry][coefficient][S]).
template <typename real, bool kJet> struct Val;
template <typename real> struct Val<real, false> {
  real c0;
  __device__ static Val load(const real *a, int e, int S, int s) { return {a[e * S + s]}; }
  __device__ void store(real *a, int e, int S, int s) const { a[e * S + s] = c0; }
  __device__ static Val spin(real t, int) { return {t}; }
  __device__ void mul(const Val &b, real sc) { c0 *= b.c0 * sc; }
};
template <typename real> struct Val<real, true> {
  real c0, c1, c2;
  __device__ static Val load(const real *a, int e, int S, int s) {
    const real *p = a + e * 3 * S + s;
    return {p[0], p[S], p[2 * S]};
  }
  __device__ void store(real *a, int e, int S, int s) const {
    real *p = a + e * 3 * S + s;
    p[0] = c0;
    p[S] = c1;
    p[2 * S] = c2;
  }
  // t e^{eta sigma}: the eliminated spin's +1 (x = 0) or -1
  __device__ static Val spin(real t, int x) { return {t, x ? -t : t, t / 2}; }
  __device__ void mul(const Val &b, real sc) {
    const real b0 = b.c0 * sc, b1 = b.c1 * sc, b2 = b.c2 * sc;
    const real n1 = c0 * b1 + c1 * b0, n2 = c0 * b2 + c1 * b1 + c2 * b0;
    c0 = c0 * b0;
    c1 = n1;
    c2 = n2;
  }
};

// A copy in a register of its own, made here: a value loaded in the pass
// before and loaded again in this one would otherwise be copied at the end
// of the pass, after the new load, and wait for it.
__device__ inline uint32_t own_copy(uint32_t v) {
  uint32_t r;
  asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
  return r;
}
__device__ inline float own_copy(float v) { return __uint_as_float(own_copy(__float_as_uint(v))); }
__device__ inline double own_copy(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  return __longlong_as_double((long long)(((unsigned long long)own_copy((uint32_t)(u >> 32)) << 32) |
                                          own_copy((uint32_t)u)));
}

// A record of the wave's program, one word per lane; a word read from it is
// wave-uniform.
struct Rec {
  int v;
  __device__ int operator[](int k) const { return __builtin_amdgcn_readlane(v, k); }
};

// A unit of output entries: fields of its record.
template <typename real>
struct Unit {
  int w, n_in, dense, n_edge, n, off, tpos, step, gpos;
  const Rec &r;
  __device__ explicit Unit(const Rec &rec) : r(rec) {
    const int d = r[0];
    w = (d >> 12) & 15;
    n_in = (d >> 16) & 7;
    dense = (d >> 19) & 1;
    n_edge = (d >> 20) & 7;
    n = 1 << ((d >> 24) & 15);
    off = r[1];
    tpos = r[2];
    const int sg = r[4];
    step = sg & 0xffff;
    gpos = sg >> 16;
  }
};

// the offset of walk position c (a constant) by the 4-bit positions of code
template <int C>
__device__ inline int walk_at(int code) {
  int e = 0;
#pragma unroll
  for (int b = 0; b < kSweepWalk; ++b)
    if ((C >> b) & 1) e += (1 << ((code >> (4 * b)) & 15)) & 0x7fff;
  return e;
}

// Per lane: each input's arena word at the unit's first entry and its scale;
// per unit the walk positions and the distance of its two entries.  lw: the
// lane word.
template <typename real, int NI>
struct UnitIn {
  int base[NI ? NI : 1], xs[NI ? NI : 1], code[NI ? NI : 1];
  real sc[NI ? NI : 1];
  template <int S>
  __device__ void set(const Rec &r, const typename MsgBits<real>::U *mx, int s, int lw) {
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int m = r[9 + 2 * k];
      base[k] = r[8 + 2 * k] + ((lw >> (8 * k)) & 0xff);
      xs[k] = 1 << ((m >> 12) & 15);
      code[k] = m;
      sc[k] = MsgBits<real>::scale(mx[(m >> 16) * S + s]);
    }
  }
  template <int C> __device__ int at(int k) const { return base[k] + walk_at<C>(code[k]); }
};

// f(integral constant c) for c = 0 .. N - 1
template <int N, typename F>
__device__ inline void each(F f) {
  if constexpr (N > 0) {
    each<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// forward unit: out[o] = sum_x T[x, o] phi[x] prod_k m_k.  A dense step
// (no input, or the message over the eliminated spin alone) forms
// A[x] = phi[x] m[x] first and accumulates T A; a general one multiplies
// T phi by the messages in turn and adds the last product of spin -1 to the
// finished one of spin +1 with one rounding.  tp: T at the first pass.
template <typename real, bool kJet, int S, int NI, int NC>
__device__ inline typename MsgBits<real>::U unit_fwd(const Unit<real> &u, const real *T, const real tp[2],
                                const typename MsgBits<real>::U *mx, const real *phi, real *arena,
                                int s, int lo, int lw) {
  using V = Val<real, kJet>;
  UnitIn<real, NI> in;
  constexpr int E = 64 / S;
  const real *T0 = T + u.tpos + lo, *T1 = T0 + (1 << u.w);
  real t0[NC], t1[NC];
  t0[0] = tp[0];
  t1[0] = tp[1];
#pragma unroll
  for (int c = 1; c < NC; ++c) {
    t0[c] = T0[c * E];
    t1[c] = T1[c * E];
  }
  in.template set<S>(u.r, mx, s, lw);
  const real ph0 = phi[2 * u.gpos * S + s], ph1 = phi[(2 * u.gpos + 1) * S + s];
  // (positive numbers compare as their bits)
  typename MsgBits<real>::U lmax = 0;
  auto largest = [&](real x) {
    const auto b = MsgBits<real>::bits(x);
    lmax = b > lmax ? b : lmax;
  };
  if (NI <= 1 && u.dense) {
    V A0 = V::spin(ph0, 0), A1 = V::spin(ph1, 1);
    if (NI == 1) {
      // (base without the lane: the input has the two entries alone)
      A0.mul(V::load(arena, in.base[0], S, s), in.sc[0]);
      A1.mul(V::load(arena, in.base[0] + 1, S, s), in.sc[0]);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      V r;
      r.c0 = __builtin_fma(t1[c], A1.c0, t0[c] * A0.c0);
      if constexpr (kJet) {
        r.c1 = __builtin_fma(t1[c], A1.c1, t0[c] * A0.c1);
        r.c2 = __builtin_fma(t1[c], A1.c2, t0[c] * A0.c2);
      }
      r.store(arena, u.off + lo + c * E, S, s);
      largest(r.c0);
    }
    return lmax;
  }
  V p0[NC], p1[NC];
  each<NC>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
    p0[c] = V::spin(t0[c] * ph0, 0);
    p1[c] = V::spin(t1[c] * ph1, 1);
#pragma unroll
    for (int k = 0; k + 1 < NI; ++k) {
      const int e = in.template at<c>(k);
      p0[c].mul(V::load(arena, e, S, s), in.sc[k]);
      p1[c].mul(V::load(arena, e + in.xs[k], S, s), in.sc[k]);
    }
  });
  each<NC>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
    V r = p0[c];
    if constexpr (NI > 0) {
      const int e = in.template at<c>(NI - 1);
      const V m0 = V::load(arena, e, S, s), m1 = V::load(arena, e + in.xs[NI - 1], S, s);
      r.mul(m0, in.sc[NI - 1]);
      if constexpr (kJet) {
        p1[c].mul(m1, in.sc[NI - 1]);
        r.c0 += p1[c].c0;
        r.c1 += p1[c].c1;
        r.c2 += p1[c].c2;
      } else {
        r.c0 = __builtin_fma(p1[c].c0, m1.c0 * in.sc[NI - 1], r.c0);
      }
    }
    r.store(arena, u.off + lo + c * E, S, s);
    largest(r.c0);
  });
  return lmax;
}

// first reverse phase of a unit: the joint weights
// c(o, x) = rho[o] 2^-e T[x, o] phi[x] prod_k m_k into scratch planes
// [x][o][S], and this lane's part of the sums over o of c(o, +) - c(o, -),
// plain (v[0]) and signed by each edge's output spin.
template <typename real, int S, int NI, int NC>
__device__ inline void unit_joint(const Unit<real> &u, const real *T, const real tp[2],
                                  const typename MsgBits<real>::U *mx, const real *phi,
                                  const real *arena, real *scr, int s, int lo, int lw, bool on,
                                  real v[1 + kSweepEdges]) {
  using FB = MsgBits<real>;
  UnitIn<real, NI> in;
  constexpr int E = 64 / S;
  const real *T0 = T + u.tpos + lo, *T1 = T0 + (1 << u.w);
  real p0[NC], p1[NC], raw[NC];
  p0[0] = tp[0];
  p1[0] = tp[1];
#pragma unroll
  for (int c = 0; c < NC; ++c) raw[c] = arena[(u.off + lo + c * E) * S + s];
#pragma unroll
  for (int c = 1; c < NC; ++c) {
    p0[c] = T0[c * E];
    p1[c] = T1[c * E];
  }
  in.template set<S>(u.r, mx, s, lw);
  const real ph0 = phi[2 * u.gpos * S + s], ph1 = phi[(2 * u.gpos + 1) * S + s];
  const real sct = FB::scale(mx[u.step * S + s]);
  each<NC>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
    const real r = u.w == 0 ? (raw[c] > 0 ? (real)1 / raw[c] : (real)0) : raw[c] * sct;
    p0[c] = r * p0[c] * ph0;
    p1[c] = r * p1[c] * ph1;
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int e = in.template at<c>(k);
      p0[c] *= arena[e * S + s] * in.sc[k];
      p1[c] *= arena[(e + in.xs[k]) * S + s] * in.sc[k];
    }
  });
  const int ebits = u.r[6], o0 = u.r[7], sb = u.r[3];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int o = lo + c * E;
    const real d = on ? p0[c] - p1[c] : (real)0;
    v[0] += d;
#pragma unroll
    for (int r = 0; r < kSweepEdges; ++r)
      if (r < u.n_edge) v[1 + r] += (((o0 + o) >> ((ebits >> (8 * r)) & 0xff)) & 1) ? -d : d;
    scr[(sb + o) * S + s] = p0[c];
    scr[(sb + (1 << u.w) + o) * S + s] = p1[c];
  }
}

// f(NI, NC) for the unit's input count and passes (at most kNC)
template <int kNC, typename F>
__device__ inline void unit_dispatch(int n_in, int nc, F f) {
  auto by_nc = [&](auto ni) {
    switch (nc) {
      case 1: f(ni, std::integral_constant<int, 1>{}); break;
      case 2: f(ni, std::integral_constant<int, 2>{}); break;
      case 4: if constexpr (kNC >= 4) f(ni, std::integral_constant<int, 4>{}); break;
      default: if constexpr (kNC >= 8) f(ni, std::integral_constant<int, 8>{}); break;
    }
  };
  switch (n_in) {
    case 0: by_nc(std::integral_constant<int, 0>{}); break;
    case 1: by_nc(std::integral_constant<int, 1>{}); break;
    case 2: by_nc(std::integral_constant<int, 2>{}); break;
    case 3: by_nc(std::integral_constant<int, 3>{}); break;
    default: by_nc(std::integral_constant<int, 4>{}); break;
  }
}

// Lanes past a unit's n entries (a power of two) do the work of entry
// lane mod n again, which their lane words match: they store the same value
// to the same place, and nothing branches on them.
template <typename real, int kMode, bool kGlobal, int kLogS>
__device__ inline void sweep_tile(const SweepArgs<real> &w, const int tile, char *smem) {
  using FB = MsgBits<real>;
  using U = typename FB::U;
  constexpr bool kSeg = kMode == 3, kBwd = kMode == 1 || kSeg, kJet = kMode == 2;
  constexpr int kNC = 1 << sweep_walk(kMode, (int)sizeof(real));
  const ContractArgs<real> &a = w.c;
  const int tid = threadIdx.x, lane = tid & 63;
  const int nthr = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = kSeg ? w.seg.q : uload(a.tile_inst + tile);
  const InstDesc D = uload(a.inst + q);
  constexpr int logS = kLogS, S = 1 << logS, logE = 6 - logS, E = 1 << logE;
  const int64_t b0 = kSeg ? w.seg.b0 + tile : uload(a.tile_start + tile);
  const int64_t Bq = uload(a.inst_B + q);
  const int nb = (int)((Bq - b0) < S ? (Bq - b0) : S);
  const int s = lane & (S - 1), lo_ = lane >> logS;
  const SLay L = sweep_layout(D, uload(w.insts + q), S, kMode, kGlobal, (int)sizeof(real));
  U *mx = reinterpret_cast<U *>(smem + L.mx);
  real *phi = reinterpret_cast<real *>(smem + L.phi);
  real *fab = reinterpret_cast<real *>(smem + L.fab);
  real *gs = reinterpret_cast<real *>(smem + L.gs);
  real *Mg = reinterpret_cast<real *>(smem + L.M);
  real *Cw = reinterpret_cast<real *>(smem + L.C);
  real *red = reinterpret_cast<real *>(smem + L.red);
  real *scr = reinterpret_cast<real *>(smem + L.scr);
  real *arena = kGlobal ? a.garena + (int64_t)blockIdx.x * a.garena_stride
                        : reinterpret_cast<real *>(smem + L.arena);
  const int8_t *spq = a.spins + uload(a.inst_spin_off + q);
  const real beta = (real)D.beta;

  // the wave's program, one record loaded ahead
  const int32_t *pr = w.prog + (int64_t)(kSeg ? w.seg.prog[wave] : uload(w.insts[q].prog + wave)) * kSweepRec +
                      (lane < kSweepRec ? lane : kSweepRec - 1);
  int ahead = *pr;
  const int32_t *w_lanes = w.lanes + lo_;
  real *state = arena + (kSeg ? w.seg.state : 0);
  if (kSeg && !w.seg.first) {
    // mx, phi, fab as the launch before left them; M and C too
    for (int i = tid; i < D.n_steps; i += nthr) mx[i] = reinterpret_cast<const U *>(state)[i];
    for (int i = tid; i < 2 * D.nr; i += nthr) phi[i] = state[D.n_steps + i];
    for (int i = tid; i < D.nr; i += nthr) fab[i] = state[D.n_steps + 2 * D.nr + i];
    if (w.seg.rev) {
      for (int i = tid; i < D.nr; i += nthr) Mg[i] = state[D.n_steps + 3 * D.nr + i];
      for (int i = tid; i < D.n_rr; i += nthr) Cw[i] = state[D.n_steps + 4 * D.nr + i];
    }
  }
  if (!kSeg || w.seg.first)
  for (int i = tid; i < D.n_steps * S; i += nthr) mx[i] = 0;
  // unary factors of R, normalised so that the larger of the two is one
  if (!kSeg || w.seg.first)
  for (int i = tid; i < D.nr * S; i += nthr) {
    const int p = i >> logS, ss = i & (S - 1);
    real f = a.hR[D.hr_off + p];
    if (ss < nb) {
      const int8_t *sp = spq + (b0 + ss) * D.nw;
      const int k0 = a.fld_ptr[D.fld_off + p], k1 = a.fld_ptr[D.fld_off + p + 1];
      for (int k = k0; k < k1; ++k)
        f += a.fld_J[D.fld_nnz_off + k] * (real)sp[a.fld_w[D.fld_nnz_off + k]];
    }
    const real af = beta * (f < 0 ? -f : f);
    const real small = sexp(-2 * af);
    phi[(2 * p) * S + ss] = f >= 0 ? (real)1 : small;
    phi[(2 * p + 1) * S + ss] = f >= 0 ? small : (real)1;
    fab[p * S + ss] = af;
  }
  if constexpr (kBwd) {
    for (int i = tid; i < S; i += nthr)
      gs[i] = i < nb && (!kSeg || w.seg.rev) ? (real)a.grad[a.inst_sample_off[q] + b0 + i] : (real)0;
    if (!kSeg || w.seg.first)
      for (int k = tid; k < D.n_rr; k += nthr) Cw[k] = 0;
    if (kSeg && w.seg.first)
      for (int k = tid; k < D.nr; k += nthr) Mg[k] = 0;
  }
  __syncthreads();

  // the lane word and the transfer factors of a unit's first pass, loaded
  // one record ahead by the words of the record before (the first record's
  // by its own)
  real tn[2];
  int lwn;
  auto load_ahead = [&](int tpos, int w, int logn, int words) {
    const real *t = a.T + tpos + (lo_ & ((1 << logn) - 1));
    tn[0] = t[0];
    tn[1] = t[1 << w];
    lwn = w_lanes[words];
  };
  {
    const Rec r{ahead};
    load_ahead(r[2], (r[0] >> 12) & 15, (r[0] >> 24) & 15, r[19]);
  }
  for (;;) {
    const Rec r{(int)own_copy((uint32_t)ahead)};
    const real tp[2] = {own_copy(tn[0]), own_copy(tn[1])};
    const int lw = (int)own_copy((uint32_t)lwn);
    const int d = r[0], op = d & 15;
    __builtin_amdgcn_sched_barrier(0);
    pr += kSweepRec;
    ahead = *pr;
    load_ahead(r[16], r[17] & 15, r[17] >> 8, r[18]);
    __builtin_amdgcn_sched_barrier(0);
    if (__builtin_expect((d >> 4) & 0xff, 0))
      for (int k = (d >> 4) & 0xff; k > 0; --k) __syncthreads();
    if (op == SWEEP_END) break;
    if (op == SWEEP_FWD) {
      const Unit<real> u(r);
      const int lo = lo_ & (u.n - 1);
      U lmax = 0;
      unit_dispatch<kNC>(u.n_in, u.n > E ? u.n >> logE : 1, [&](auto ni, auto nc) {
        lmax = unit_fwd<real, kJet, S, decltype(ni)::value, decltype(nc)::value>(
            u, a.T, tp, mx, phi, arena, s, lo, lw);
      });
      lmax = lanes_max<S, 64>(lmax);
      if (lane < S) atomicMax(&mx[u.step * S + s], lmax);
    } else if (op == SWEEP_LOGZ) {
      if (!kBwd || a.logz) {
        // (the instance's descriptors again: not held through the program)
        int q2 = q;
        asm volatile("" : "+s"(q2));
        const InstDesc D = uload(a.inst + q2);
        const SweepInst W = uload(w.insts + q2);
        double m1 = 0, vr = 0;
        int esum = 0;
        for (int t = lo_; t < D.n_steps; t += E) esum += FB::expo(mx[t * S + s]);
        esum = lanes_sum<S, 64>(esum);
        // the sum of beta |f| as eight chains of every eighth position, added
        // pairwise: the same additions at every S
        double fs[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          fs[j] = 0;
          if (j * E >= 8) continue;
          if (j * E + lo_ < 8)
            for (int p = j * E + lo_; p < D.nr; p += 8) fs[j] += (double)fab[p * S + s];
          fs[j] = lanes_sum<S, (S * 8 < 64 ? S * 8 : 64)>(fs[j]);
        }
        double acc = D.log_const + (((fs[0] + fs[1]) + (fs[2] + fs[3])) + ((fs[4] + fs[5]) + (fs[6] + fs[7])));
        for (int i = 0; i < W.n_close; ++i) {
          const int32_t *cl = w.close + W.close_off + 2 * i;   // arena entry, step
          const Val<real, kJet> z = Val<real, kJet>::load(arena, cl[0], S, s);
          esum -= FB::expo(mx[cl[1] * S + s]);
          acc += log((double)z.c0);
          if constexpr (kJet) {
            const double r1 = (double)z.c1 / (double)z.c0, r2 = (double)z.c2 / (double)z.c0;
            m1 += r1;
            vr += 2.0 * r2 - r1 * r1;
          }
        }
        if (lane < nb) {
          const int64_t g = uload(a.inst_sample_off + q) + b0 + lane;
          if (a.logz) a.logz[g] = __builtin_fma((double)esum, 0.69314718055994530942, acc);
          if constexpr (kJet) {
            w.mean[g] = m1;
            w.var[g] = vr;
          }
        }
      }
    } else if constexpr (kBwd) {
      if (op == SWEEP_JOINT) {
        const Unit<real> u(r);
        const bool on = lo_ < u.n;
        const int lo = lo_ & (u.n - 1);
        const int slot = r[5];
        real v[1 + kSweepEdges];
#pragma unroll
        for (int k = 0; k <= kSweepEdges; ++k) v[k] = 0;
        unit_dispatch<kNC>(u.n_in, u.n > E ? u.n >> logE : 1, [&](auto ni, auto nc) {
          unit_joint<real, S, decltype(ni)::value, decltype(nc)::value>(
              u, a.T, tp, mx, phi, arena, scr, s, lo, lw, on, v);
        });
#pragma unroll
        for (int k = 0; k <= kSweepEdges; ++k)
          if (k <= u.n_edge) {
            v[k] = lanes_sum<S, 64>(v[k]);
            if (lane < S) red[(slot + k) * S + s] = v[k];
          }
      } else if (op == SWEEP_MARG) {
        const int lc = (d >> 12) & 15, n = 1 << ((d >> 16) & 15);
        const bool on = lo_ < n;
        const int lo = lo_ & (n - 1);
        const int high = r[5], nit = 1 << __popc(high), code = r[2], nc = n >> logE;
        const real sc = FB::scale(mx[r[4] * S + s]);
        real *slot = arena + (r[3] + (lo >> lc)) * S + s;
        const real *col0 = scr + (r[1] + lw) * S + s;
        for (int c = 0; c < nc || c == 0; ++c) {
          const real raw = *slot;
          int at = 0;
#pragma unroll
          for (int b = 0; b < kSweepWalk; ++b)
            at += ((c >> b) & 1) ? (1 << ((code >> (4 * b)) & 15)) & 0x7fff : 0;
          const real *col = col0 + at * S;
          // the subsets z of the summed bits, four at a time
          real m0 = 0, m1 = 0, m2 = 0, m3 = 0;
          int z = 0;
          if (nit >= 4) {
            for (int k = 0; k < nit; k += 4) {
              const int z1 = (z - high) & high, z2 = (z1 - high) & high, z3 = (z2 - high) & high;
              m0 += col[z * S];
              m1 += col[z1 * S];
              m2 += col[z2 * S];
              m3 += col[z3 * S];
              z = (z3 - high) & high;
            }
          } else {
            for (int k = 0; k < nit; ++k) {
              m0 += col[z * S];
              z = (z - high) & high;
            }
          }
          real mu = (m0 + m1) + (m2 + m3);
          if (lc) {
            // the sums of the lanes that share an entry
            real part[7];
            part[0] = mu;
            part[1] = lanes_sum<S, 2 * S>(mu);
            part[2] = lanes_sum<2 * S, 4 * S>(part[1]);
            if constexpr (logE >= 3) part[3] = lanes_sum<4 * S, 8 * S>(part[2]);
            if constexpr (logE >= 4) part[4] = lanes_sum<8 * S, 16 * S>(part[3]);
            if constexpr (logE >= 5) part[5] = lanes_sum<16 * S, 32 * S>(part[4]);
            if constexpr (logE >= 6) part[6] = lanes_sum<32 * S, 64 * S>(part[5]);
#pragma unroll
            for (int b = 1; b <= logE; ++b) mu = lc == b ? part[b] : mu;
          }
          if (on && (lo & ((1 << lc) - 1)) == 0) {
            const real mm = raw * sc;
            *slot = mm > 0 ? mu / mm : (real)0;
          }
          slot += (E >> lc) * S;
        }
      } else if (op == SWEEP_SUM) {
        // value k of sample s on lane (k, s); more values than lane rows walk
        const int n_edge = (d >> 20) & 7, first = r[1], stride = r[2], n = r[3], gpos = r[4];
        const int e0 = r[5], e1 = r[6], e2 = r[7], e3 = r[8];
        for (int kk = 0; kk <= n_edge; kk += E) {
          const int k = kk + lo_;
          real sum = 0;
          for (int i = 0; i < n && k <= n_edge; ++i) sum += red[(first + i * stride + k) * S + s];
          const real g = lanes_sum<1, S>(gs[s] * sum);
          if (k == 0) Mg[gpos * S + s] = sum;
          else if (k <= n_edge && s == 0) Cw[k == 1 ? e0 : k == 2 ? e1 : k == 3 ? e2 : e3] = g;
        }
      }
    }
  }
  if constexpr (!kBwd) return;
  if constexpr (kSeg) {
    __syncthreads();
    if (!w.seg.rev) {
      for (int i = tid; i < D.n_steps; i += nthr) reinterpret_cast<U *>(state)[i] = mx[i];
      if (w.seg.first) {
        for (int i = tid; i < 2 * D.nr; i += nthr) state[D.n_steps + i] = phi[i];
        for (int i = tid; i < D.nr; i += nthr) state[D.n_steps + 2 * D.nr + i] = fab[i];
      }
    }
    if (!w.seg.last) {
      if (w.seg.first || w.seg.rev) {
        for (int i = tid; i < D.nr; i += nthr) state[D.n_steps + 3 * D.nr + i] = Mg[i];
        for (int i = tid; i < D.n_rr; i += nthr) state[D.n_steps + 4 * D.nr + i] = Cw[i];
      }
      return;
    }
    // the wide steps' sums over their workgroups, one sum per wave at a time
    for (int i = wave; i < w.seg.n_sums; i += nthr / 64) {
      const WideSum ws = uload(w.seg.sums + i);
      const real *p = arena + w.seg.red + ws.first;
      real v = 0;
      for (int k = lane; k < ws.n; k += 64) v += p[k * ws.stride];
      v = lanes_sum<1, 64>(v);
      if (lane == 0) {
        if (ws.edge < 0) Mg[-1 - ws.edge] = v;
        else Cw[ws.edge] = gs[0] * v;
      }
    }
    __syncthreads();
  }

  // ------------------------------------------------- per-tile partial row
  int q2 = q;
  asm volatile("" : "+s"(q2));
  const InstDesc D2 = uload(a.inst + q2);
  const int64_t prow = uload(a.inst_partial_off + q2) +
                       (kSeg ? b0 : (int64_t)(tile - uload(a.inst_first_tile + q2))) * D2.n_partial;
  for (int p = tid; p < D2.nr; p += nthr) {
    real acc = 0;
    for (int k = 0; k < S; ++k) acc += gs[k] * Mg[p * S + k];
    a.partial[prow + p] = acc;
  }
  for (int k = tid; k < D2.n_wr; k += nthr) {
    const int p = a.wr_pos[D2.wr_off + k], wi = a.wr_w[D2.wr_off + k];
    real acc = 0;
    for (int ss = 0; ss < nb; ++ss)
      acc += gs[ss] * (real)spq[(b0 + ss) * D2.nw + wi] * Mg[p * S + ss];
    a.partial[prow + D2.nr + k] = acc;
  }
  for (int k = tid; k < D2.n_rr; k += nthr) a.partial[prow + D2.nr + D2.n_wr + k] = Cw[k];
}

// One workgroup per tile, or (a grid of fewer workgroups) each walking tiles
// a grid apart; a workgroup's arena in device memory is its own.
// (single precision: four waves per SIMD, two workgroups per CU)
template <typename real, int kMode, bool kGlobal, int kLogS>
__global__ __launch_bounds__(kThreads, sizeof(real) == 4 ? (kMode == 0 ? 4 : 6) : 4) void sweep_kernel(SweepArgs<real> w, int n_tiles) {
  extern __shared__ __align__(16) char smem[];
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    sweep_tile<real, kMode, kGlobal, kLogS>(w, tile, smem);
    __syncthreads();
  }
}

}  // namespace

size_t sweep_lds_bytes(const InstDesc &D, const SweepInst &W, int S, int mode, bool global_arena,
                       int real_size) {
  return sweep_layout(D, W, S, mode, global_arena, real_size).end;
}

template <typename real>
hipError_t launch_sweep(const SweepArgs<real> &a, int n_tiles, size_t lds, int mode,
                        bool global_arena, int waves, int max_grid, hipStream_t st) {
  if (n_tiles <= 0) return hipSuccess;
  if ((mode == 1 && !global_arena) || waves < 1 || waves > kSweepWaves) return hipErrorInvalidValue;
  void (*k)(SweepArgs<real>, int) = nullptr;
  auto pick = [&](auto ls) {
    constexpr int L = decltype(ls)::value;
    k = mode == 0   ? (global_arena ? sweep_kernel<real, 0, true, L> : sweep_kernel<real, 0, false, L>)
        : mode == 1 ? sweep_kernel<real, 1, true, L>
                    : (global_arena ? sweep_kernel<real, 2, true, L> : sweep_kernel<real, 2, false, L>);
  };
  switch (a.c.S) {
    case 1: pick(std::integral_constant<int, 0>{}); break;
    case 2: pick(std::integral_constant<int, 1>{}); break;
    case 4: pick(std::integral_constant<int, 2>{}); break;
    case 8: pick(std::integral_constant<int, 3>{}); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int grid = max_grid > 0 ? std::min(n_tiles, max_grid) : n_tiles;
  hipLaunchKernelGGL(k, dim3(grid), dim3(64 * waves), lds, st, a, n_tiles);
  return hipGetLastError();
}

template <typename real>
hipError_t launch_sweep_segment(const SweepArgs<real> &a, int n_samples, size_t lds, hipStream_t st) {
  if (n_samples <= 0) return hipSuccess;
  void (*k)(SweepArgs<real>, int) = sweep_kernel<real, 3, true, 0>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(n_samples), dim3(64 * kSweepWaves), lds, st, a, n_samples);
  return hipGetLastError();
}

template hipError_t launch_sweep_segment<float>(const SweepArgs<float> &, int, size_t, hipStream_t);
template hipError_t launch_sweep_segment<double>(const SweepArgs<double> &, int, size_t, hipStream_t);
template hipError_t launch_sweep<float>(const SweepArgs<float> &, int, size_t, int, bool, int, int, hipStream_t);
template hipError_t launch_sweep<double>(const SweepArgs<double> &, int, size_t, int, bool, int, int, hipStream_t);

}  // namespace tnvan
