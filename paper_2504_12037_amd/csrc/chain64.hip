// Chains of narrow dense steps in double precision on the matrix cores.
//
// An FP64 net's lattice strips (sets of chains, program.h) run here instead
// of the general kernel: the transfer-matrix recursion of chainr.hip,
//   A_{t+1} = d_{t+1} * (A_t T_t) / 2^e_t,
// per wave for 16 samples, the products transposed (out^T = T^T A^T) on
// 16x16x4 FP64 matrix-core tiles.  Lane l holds, for sample l & 15, the
// states 16 t + 4 r + (l >> 4) in register [t][r]: the product's output
// layout, and chunk r of tile t of the next product's operand, so a chain
// runs from register to register.  The transfer tables are read as compiled
// (16 lanes read 128 consecutive bytes), zero outside the step's states.
//
// The adjoint keeps the state of every step in device memory and walks back
// with R_t = d ln Z / d out_t:
//   Lambda_t = T_t R_t,  p_t = A_t * Lambda_t,  R_{t-1} = d_t * Lambda_t / 2^e_{t-1}
//   G_t = T_t o sum_s g_s A_t[s] R_t[s]^T      (contraction over the samples)
//   Q_t = S_o^T (G_t^T S_x)
// with the spin-product columns S_x and S_o of chainr.hip: Q holds the
// step's edge correlations and magnetisations summed over the 16 samples,
// stored by the same destination table; the W-R sums come from p_t.
//
// What bounds it: 5 x CT^2 x 4 products of 64 cycles per step, and the
// checkpoints (16 x 16 x 32 states of 8 bytes per two-tile wave, written and
// read once); at two waves per SIMD neither is hidden fully.  The three
// 16x16 lattices with 8192 samples each, forward + adjoint: 7.40 ms on the
// general kernel, 0.37 ms here (0.35 ms in the adjoint kernel, whose
// products alone take about 0.11 ms and whose checkpoints 0.09 ms).
#include <hip/hip_runtime.h>

#include "lanes.h"
#include "launch.h"
#include "uload.h"
#include "wave.h"

namespace tnvan {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int CW = 16;       // samples per wave
constexpr int kWaves = 4;    // waves per workgroup

__device__ inline d4 mfma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// e with m 2^-e in [0.5, 1), and 2^-e
__device__ inline int expo64(double m) {
  const int e = (int)((__double_as_longlong(m) >> 52) & 0x7ff) - 1022;
  return e > 1022 ? 1022 : e;
}
__device__ inline double pow2neg64(int e) {
  return __longlong_as_double((long long)(1023 - e) << 52);
}

// transfer entries of the forward product (also those of G): T[x][o],
// x = 16 xt + 4 r + lg, o = 16 nt + ls
template <int CT>
__device__ inline void load_t(const double *T, const Chain64Step &sd, int ls, int lg,
                              double (&t)[CT][CT][4]) {
  const int K = 1 << sd.g, N = 1 << sd.w;
#pragma unroll
  for (int nt = 0; nt < CT; ++nt)
#pragma unroll
    for (int xt = 0; xt < CT; ++xt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = 16 * xt + 4 * r + lg, o = 16 * nt + ls;
        const bool in = x < K && o < N;
        const double v = T[in ? (x << sd.w) | o : 0];
        t[nt][xt][r] = in ? v : 0.0;
      }
}
// transfer entries of Lambda: T[x][o], x = 16 xt + ls, o = 16 nt + 4 r + lg
template <int CT>
__device__ inline void load_q(const double *T, const Chain64Step &sd, int xt, int ls, int lg,
                              double (&t)[CT][4]) {
  const int K = 1 << sd.g, N = 1 << sd.w;
#pragma unroll
  for (int nt = 0; nt < CT; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int x = 16 * xt + ls, o = 16 * nt + 4 * r + lg;
      const bool in = x < K && o < N;
      const double v = T[in ? (x << sd.w) | o : 0];
      t[nt][r] = in ? v : 0.0;
    }
}

template <int CT> struct Spins { static constexpr int v = CT == 1 ? 4 : CT == 2 ? 5 : 6; };

// unary factors of a group's positions of the lane's sample
template <int GR>
__device__ inline void load_u(const double *ub, int us, const Chain64Step &sd, double (&u)[GR]) {
#pragma unroll
  for (int j = 0; j < GR; ++j) u[j] = ub[(int64_t)(sd.gpos + (j < sd.g ? j : 0)) * us];
}

// diagonal of a group: the product of its spins' factors (1 for the
// favoured value, |u| for the other; the sign bit of u favours -1, which a
// factor too small for a double keeps as -0), zero past its states.  kClass:
// the sign by the class of u (-inf, -normal, -denormal or -0), one comparison,
// which suits the reverse walk (the adjoint of a 16x16 lattice, 1000 samples,
// 112 against 117 us) and not the recursion forward (an 8x8 one 18.9 against
// 18.6)
template <int CT, int GR, bool kClass>
__device__ inline void diag(const double (&u)[GR], int g, int lg, double (&d)[CT][4]) {
  auto ph = [&](int j, bool minus) {
    if (j >= GR) return 1.0;
    const double v = u[j < GR ? j : 0];
    const bool neg = kClass ? __builtin_amdgcn_class(v, 0x3C) : (bool)__builtin_signbit(v);
    return j < g ? (minus == neg ? 1.0 : fabs(v)) : 1.0;
  };
  const double fl = ph(0, lg & 1) * ph(1, lg & 2);
  double fr[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) fr[r] = ph(2, r & 1) * ph(3, r & 2) * fl;
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const double ft = ph(4, t & 1) * ph(5, t & 2);
#pragma unroll
    for (int r = 0; r < 4; ++r) d[t][r] = 16 * t + 4 * r + lg < 1 << g ? fr[r] * ft : 0.0;
  }
}

// out^T = T^T A^T
template <int CT>
__device__ inline void product(const double (&t)[CT][CT][4], const double (&x)[CT][4], d4 (&acc)[CT]) {
#pragma unroll
  for (int nt = 0; nt < CT; ++nt) acc[nt] = d4{0, 0, 0, 0};
#pragma unroll
  for (int xt = 0; xt < CT; ++xt)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int nt = 0; nt < CT; ++nt) acc[nt] = mfma64(t[nt][xt][r], x[xt][r], acc[nt]);
}

struct Wave {
  int i, q, c, lane, ls, lg;   // i: the task in its launch
  int64_t b0, B;
  int us;                   // samples that a position of U holds
};

// The forward recursion of one chain, the state of every step to keep(t, x)
// and its exponent to expo(t, e).  Returns the closing entry; esum: the sum
// of the exponents.
template <int CT, typename Keep, typename Expo>
__device__ inline double forward(const Chain64Args &a, const Wave &k, const InstDesc &D,
                                 const ChainDesc &cd, int &esum, Keep keep, Expo expo) {
  constexpr int GR = Spins<CT>::v;
  const Chain64Step *cs = a.csteps + cd.cs_off;
  const int64_t b = k.b0 + k.ls;
  const double *ub = a.U + a.u_off[k.q] + ((b < k.B ? b : k.B - 1) - a.w0);
  double x[CT][4];
  const Chain64Step s0 = uload(cs);
  {
    double u[GR];
    load_u<GR>(ub, k.us, s0, u);
    diag<CT, GR, false>(u, s0.g, k.lg, x);
  }
  esum = 0;
  double raw = 1.0;
  // step t with its operands loaded; loads step t + 1's into the other set
  // (two sets in turn: a loaded value is never copied)
  auto step = [&](int t, const double (&tc)[CT][CT][4], const double (&uc)[GR],
                  double (&tn)[CT][CT][4], double (&un)[GR]) -> bool {
    const bool last = t == cd.n_steps - 1;
    const Chain64Step sn = uload(cs + (last ? t : t + 1));
    load_t<CT>(a.T + sn.t_off, sn, k.ls, k.lg, tn);
    load_u<GR>(ub, k.us, uload(cs + (t + 2 < cd.n_steps ? t + 2 : cd.n_steps - 1)), un);
    keep(t, x);
    d4 acc[CT];
    product<CT>(tc, x, acc);
    if (last) {
      raw = __shfl(acc[0][0], k.ls, 64);
      return true;
    }
    double m = 0;
#pragma unroll
    for (int n = 0; n < CT; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) m = fmax(m, acc[n][r]);
    const int e = expo64(lanes_max<16, 64>(m));
    const double sc = pow2neg64(e);
    double d[CT][4];
    diag<CT, GR, false>(uc, sn.g, k.lg, d);
#pragma unroll
    for (int n = 0; n < CT; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) x[n][r] = acc[n][r] * sc * d[n][r];
    expo(t, e);
    esum += e;
    return false;
  };
  double tA[CT][CT][4], tB[CT][CT][4], uA[GR], uB[GR];
  load_t<CT>(a.T + s0.t_off, s0, k.ls, k.lg, tA);
  load_u<GR>(ub, k.us, uload(cs + (cd.n_steps > 1 ? 1 : 0)), uA);
  for (int t = 0;; t += 2) {
    if (step(t, tA, uA, tB, uB)) break;
    if (step(t + 1, tB, uB, tA, uA)) break;
  }
  return raw;
}

__device__ inline bool wave_task(const Chain64Args &a, Wave &k) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int i = blockIdx.x * kWaves + wave;
  if (i >= a.n_tasks) return false;
  k.i = i;
  k.lane = threadIdx.x & 63;
  k.ls = k.lane & 15;
  k.lg = k.lane >> 4;
  k.q = uload(a.task_inst + a.task_base + i);
  k.c = uload(a.task_chain + a.task_base + i);
  k.b0 = uload(a.task_start + a.task_base + i);
  k.B = uload(a.inst_B + k.q);
  k.us = (int)k.B < a.win ? (int)k.B : a.win;   // (32 bits: a scalar minimum)
  return true;
}

template <int CT>
__device__ inline void fwd_task(const Chain64Args &a, const Wave &k) {
  const InstDesc D = uload(a.inst + k.q);
  const ChainDesc cd = uload(a.chains + uload(&a.cinst[k.q].chain_off) + k.c);
  int esum;
  const double raw = forward<CT>(a, k, D, cd, esum, [](int, const double (&)[CT][4]) {},
                                 [](int, int) {});
  const int64_t b = k.b0 + k.ls;
  if (k.lg == 0 && b < k.B)
    a.cpart[a.cpart_off[k.q] + (int64_t)k.c * k.B + b] =
        __builtin_fma((double)esum, 0.69314718055994530942, log(raw));
}

// chains of one and two tiles in one launch (the two-tile tasks first: the
// waves of the shorter chains fill what they leave), four tiles in their own
template <bool kWide>
__global__ __launch_bounds__(64 * kWaves) void chain64_fwd_kernel(Chain64Args a) {
  Wave k;
  if (!wave_task(a, k)) return;
  if constexpr (kWide) fwd_task<4>(a, k);
  else if (k.i < a.n_two) fwd_task<2>(a, k);
  else fwd_task<1>(a, k);
}

// LDS of a wave: exponents [step][16], g A and R by sample (rows padded)
__host__ __device__ constexpr int row64(int ct) { return 16 * ct + 2; }
__host__ __device__ inline size_t wave_lds(int ct, int max_steps) {
  return ((size_t)max_steps * CW * 4 + 15) / 16 * 16 + (size_t)2 * CW * row64(ct) * 8;
}

template <int CT>
__device__ inline void bwd_task(const Chain64Args &a, const Wave &k, char *base) {
  constexpr int GR = Spins<CT>::v, LD = row64(CT);
  int *ex = reinterpret_cast<int *>(base);
  double *ga = reinterpret_cast<double *>(base + ((size_t)a.max_steps * CW * 4 + 15) / 16 * 16);
  double *rs = ga + CW * LD;
  const InstDesc D = uload(a.inst + k.q);
  const ChainDesc cd = uload(a.chains + uload(&a.cinst[k.q].chain_off) + k.c);
  const Chain64Step *cs = a.csteps + cd.cs_off;
  const int ls = k.ls, lg = k.lg;
  const int64_t b = k.b0 + ls;
  double *ck = a.ckpt + (int64_t)k.i * a.max_steps * a.ck_tiles * 256 + (int64_t)k.lane * 4;
  auto slot = [&](int t, int xt) { return reinterpret_cast<d4 *>(ck + ((int64_t)t * CT + xt) * 256); };
  int esum;
  const double raw = forward<CT>(
      a, k, D, cd, esum,
      [&](int t, const double (&x)[CT][4]) {
#pragma unroll
        for (int xt = 0; xt < CT; ++xt) *slot(t, xt) = d4{x[xt][0], x[xt][1], x[xt][2], x[xt][3]};
      },
      [&](int t, int e) {
        if (lg == 0) ex[t * CW + ls] = e;
      });
  if (a.write_logz && lg == 0 && b < k.B)
    a.cpart[a.cpart_off[k.q] + (int64_t)k.c * k.B + b] =
        __builtin_fma((double)esum, 0.69314718055994530942, log(raw));
  __builtin_amdgcn_wave_barrier();

  const int64_t bc = b < k.B ? b : k.B - 1;   // past the batch: clamped, weight 0
  const double g = b < k.B ? a.grad[a.inst_sample_off[k.q] + b] : 0.0;
  const int8_t *sp = a.spins + a.inst_spin_off[k.q] + bc * D.nw;
  const bool bits = D.nw <= 128;
  const SpinBits sb = bits ? load_bits_row(sp, D.nw) : SpinBits{{0u, 0u, 0u, 0u}};
  const double *ub = a.U + a.u_off[k.q] + (bc - a.w0);
  double *prow = a.partial + a.inst_partial_off[k.q] + (k.b0 / CW) * (int64_t)D.n_partial;
  // R of the closing entry (state 0: register 0 of lane group 0)
  double R[CT][4];
#pragma unroll
  for (int t = 0; t < CT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) R[t][r] = 0.0;
  R[0][0] = lg == 0 && raw > 0.0 ? 1.0 / raw : 0.0;
  // a step's operands are loaded in the step after it, each where its
  // registers were last used
  Chain64Step c = uload(cs + cd.n_steps - 1);
  d4 A[CT];
  double q[CT][CT][4], tf[CT][CT][4], u[GR];
#pragma unroll
  for (int xt = 0; xt < CT; ++xt) load_q<CT>(a.T + c.t_off, c, xt, ls, lg, q[xt]);
#pragma unroll
  for (int xt = 0; xt < CT; ++xt) A[xt] = *slot(cd.n_steps - 1, xt);
  load_t<CT>(a.T + c.t_off, c, ls, lg, tf);
  load_u<GR>(ub, k.us, c, u);
  for (int t = cd.n_steps - 1; t >= 0; --t) {
    const int tp = t > 0 ? t - 1 : 0;
    const Chain64Step cn = uload(cs + tp);
    float sx[CT][4], so[CT][4];
    int dst[4];
#pragma unroll
    for (int xt = 0; xt < CT; ++xt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sx[xt][r] = a.Tsx[c.sx_off + xt * 256 + (ls + 16 * r) * 4 + lg];
        so[xt][r] = a.Tsx[c.sx_off + (CT + xt) * 256 + (ls + 16 * r) * 4 + lg];
      }
    // cell (column ls, row 4 r + lg): its lane and register in the table
#pragma unroll
    for (int r = 0; r < 4; ++r) dst[r] = a.Tdq[c.dq_off + (ls + 16 * r) * 4 + lg];
    // g A and R by sample, for the contraction over the samples
#pragma unroll
    for (int xt = 0; xt < CT; ++xt)
#pragma unroll
      for (int r = 0; r < 4; ++r) rs[ls * LD + 16 * xt + 4 * r + lg] = R[xt][r];
    // Lambda = T R
    d4 lam[CT];
#pragma unroll
    for (int xt = 0; xt < CT; ++xt) lam[xt] = d4{0, 0, 0, 0};
#pragma unroll
    for (int nt = 0; nt < CT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int xt = 0; xt < CT; ++xt) lam[xt] = mfma64(q[xt][nt][r], R[nt][r], lam[xt]);
#pragma unroll
    for (int xt = 0; xt < CT; ++xt) load_q<CT>(a.T + cn.t_off, cn, xt, ls, lg, q[xt]);
#pragma unroll
    for (int xt = 0; xt < CT; ++xt)
#pragma unroll
      for (int r = 0; r < 4; ++r) ga[ls * LD + 16 * xt + 4 * r + lg] = g * A[xt][r];
    // W-R correlations of the group: the magnetisation of spin j times the
    // width-set spin, summed over the samples
    for (int n = 0; n < c.n_wri; ++n) {
      const int wr = n == 0 ? c.wri[0] : n == 1 ? c.wri[1] : n == 2 ? c.wri[2] : c.wri[3];
      const int we = n == 0 ? c.wre[0] : n == 1 ? c.wre[1] : n == 2 ? c.wre[2] : c.wre[3];
      const int j = wr & 0xff, wi = wr >> 8;
      double m = 0;
#pragma unroll
      for (int xt = 0; xt < CT; ++xt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double p = A[xt][r] * lam[xt][r];
          m += ((16 * xt + 4 * r + lg) >> j) & 1 ? -p : p;
        }
      m *= g * (bits ? (double)sb.sigma(wi) : (double)sp[wi]);
      m = lanes_sum<1, 64>(m);
      if (k.lane == 0) prow[D.nr + we] = m;
    }
#pragma unroll
    for (int xt = 0; xt < CT; ++xt) A[xt] = *slot(tp, xt);
    __builtin_amdgcn_wave_barrier();
    // G = T o (sum over samples of g A R), G^T S_x, S_o^T (G^T S_x)
    double oa[CT][4], ob[CT][4];
    d4 Q = d4{0, 0, 0, 0};
#pragma unroll
    for (int xt = 0; xt < CT; ++xt)
#pragma unroll
      for (int cch = 0; cch < 4; ++cch) {
        oa[xt][cch] = ga[(4 * cch + lg) * LD + 16 * xt + ls];
        ob[xt][cch] = rs[(4 * cch + lg) * LD + 16 * xt + ls];
      }
#pragma unroll
    for (int nt = 0; nt < CT; ++nt) {
      d4 h[CT], pt = d4{0, 0, 0, 0};
#pragma unroll
      for (int xt = 0; xt < CT; ++xt) h[xt] = d4{0, 0, 0, 0};
#pragma unroll
      for (int cch = 0; cch < 4; ++cch)
#pragma unroll
        for (int xt = 0; xt < CT; ++xt) h[xt] = mfma64(oa[xt][cch], ob[nt][cch], h[xt]);
#pragma unroll
      for (int xt = 0; xt < CT; ++xt)
#pragma unroll
        for (int r = 0; r < 4; ++r) pt = mfma64(h[xt][r] * tf[nt][xt][r], (double)sx[xt][r], pt);
#pragma unroll
      for (int r = 0; r < 4; ++r) Q = mfma64((double)so[nt][r], pt[r], Q);
    }
    load_t<CT>(a.T + cn.t_off, cn, ls, lg, tf);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (dst[r] >= 0) prow[dst[r]] = Q[r];
    const double sc = t > 0 ? pow2neg64(ex[tp * CW + ls]) : 0.0;
    double d[CT][4];
    diag<CT, GR, true>(u, c.g, lg, d);
#pragma unroll
    for (int xt = 0; xt < CT; ++xt)
#pragma unroll
      for (int r = 0; r < 4; ++r) R[xt][r] = d[xt][r] * lam[xt][r] * sc;
    load_u<GR>(ub, k.us, cn, u);
    c = cn;
    __builtin_amdgcn_wave_barrier();
  }
}

template <bool kWide>
__global__ __launch_bounds__(64 * kWaves, kWide ? 1 : 2) void chain64_bwd_kernel(Chain64Args a) {
  extern __shared__ __align__(16) char smem[];
  Wave k;
  if (!wave_task(a, k)) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  char *base = smem + (size_t)wave * wave_lds(kWide ? 4 : 2, a.max_steps);
  if constexpr (kWide) bwd_task<4>(a, k, base);
  else if (k.i < a.n_two) bwd_task<2>(a, k, base);
  else bwd_task<1>(a, k, base);
}

// Unary factors u of every (position, sample of the pass): exp(-2 beta |f|),
// its sign bit set for f < 0, and the sums of beta |f| per run of kUnaryChunk
// positions; one thread per (sample, run).  f is the field plus the W-R couplings times the
// width-set spins (Sec. 2).
__global__ __launch_bounds__(256) void unary64_kernel(Chain64Args a, const int32_t *list,
                                                      const int64_t *f_off, double *U,
                                                      double *fabp) {
  const int q = list[blockIdx.z];
  const InstDesc D = a.inst[q];
  const int64_t B = a.inst_B[q];
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, b = a.w0 + i;
  const int p0 = blockIdx.y * kUnaryChunk;
  if (p0 >= D.nr || b >= B || i >= a.win) return;
  const int us = (int)B < a.win ? (int)B : a.win;
  const int p1 = p0 + kUnaryChunk < D.nr ? p0 + kUnaryChunk : D.nr;
  const int8_t *sp = a.spins + a.inst_spin_off[q] + b * D.nw;
  double *Uq = U + a.u_off[q];
  double fab = 0;
  for (int p = p0; p < p1; ++p) {
    double f = a.hR[D.hr_off + p];
    const int k0 = a.fld_ptr[D.fld_off + p], k1 = a.fld_ptr[D.fld_off + p + 1];
    for (int k = k0; k < k1; ++k)
      f += a.fld_J[D.fld_nnz_off + k] * (double)sp[a.fld_w[D.fld_nnz_off + k]];
    const double af = D.beta * fabs(f), sm = exp(-2.0 * af);
    Uq[(int64_t)p * us + i] = f >= 0.0 ? sm : -sm;
    fab += af;
  }
  fabp[f_off[q] + (int64_t)blockIdx.y * B + b] = fab;
}

}  // namespace

size_t chain64_lds(bool wide, int max_steps) { return kWaves * wave_lds(wide ? 4 : 2, max_steps); }

hipError_t launch_unary64(const Chain64Args &a, const int32_t *list, int n_list, int max_chunks,
                          int64_t max_B, const int64_t *f_off, double *U, double *fabp,
                          hipStream_t st) {
  if (n_list <= 0 || max_B <= 0 || max_chunks <= 0) return hipSuccess;
  hipLaunchKernelGGL(unary64_kernel, dim3((unsigned)((max_B + 255) / 256), max_chunks, n_list),
                     dim3(256), 0, st, a, list, f_off, U, fabp);
  return hipGetLastError();
}

hipError_t launch_chain64(const Chain64Args &a, bool wide, bool bwd, hipStream_t st) {
  if (a.n_tasks <= 0) return hipSuccess;
  const dim3 grid((a.n_tasks + kWaves - 1) / kWaves), block(64 * kWaves);
  void (*k)(Chain64Args) = bwd ? (wide ? chain64_bwd_kernel<true> : chain64_bwd_kernel<false>)
                               : (wide ? chain64_fwd_kernel<true> : chain64_fwd_kernel<false>);
  const size_t lds = bwd ? chain64_lds(wide, a.max_steps) : 0;
  if (bwd) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, grid, block, lds, st, a);
  return hipGetLastError();
}

}  // namespace tnvan
