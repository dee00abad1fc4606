// Host walk of the level schedule (csrc/sweep.h): every record of every
// wave's program executed phase by phase, lane by lane in double precision with the index
// arithmetic of the kernels, every access bounds-checked, against the
// step-by-step elimination and the joint weights summed directly.  Random
// graphs of several degrees and leaf counts, tiles of 1 to 64 samples, every
// walk length.  Exit status 0 when everything agrees.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <string>
#include <vector>

#include "../../paper_2504_12037_amd/csrc/compile.h"
#include "../../paper_2504_12037_amd/csrc/sweep.h"

using namespace tnvan;

static int g_fail = 0;
#define CHECK(c)                                                           \
  do {                                                                     \
    if (!(c) && ++g_fail < 20)                                             \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); \
  } while (0)
static bool near(double a, double b) { return std::fabs(a - b) <= 1e-12 * (std::fabs(a) + std::fabs(b) + 1e-300); }

static void check(const HostProgram &P, int S, int waves, int walk) {
  const InstDesc &D = P.insts[0];
  const StepDesc *st = P.steps.data() + D.step_off;
  const int E = 64 / S;
  // messages step by step (no rescale, unary factors 1 and 0.3 + 0.01 p)
  auto phi = [&](int p, int x) { return x ? 0.3 + 0.01 * p : 1.0; };
  std::vector<std::vector<double>> msg(D.n_steps);
  auto gather = [&](const InputDesc &id, int o, int x) {
    int idx = 0;
    for (int b = 0; b < id.nbits; ++b) idx |= (id.src[b] < 0 ? x : (o >> id.src[b]) & 1) << b;
    return idx;
  };
  auto joint = [&](int t, int o, int x) {
    double p = P.T[st[t].t_off + ((int64_t)x << st[t].w) + o] * phi(st[t].gpos, x);
    for (int k = 0; k < st[t].n_in; ++k) {
      const InputDesc &id = P.inputs[st[t].in_off + k];
      p *= msg[id.step].at(st[t].kind == STEP_DENSE ? x : gather(id, o, x));
    }
    return p;
  };
  for (int t = 0; t < D.n_steps; ++t)
    for (int o = 0; o < 1 << st[t].w; ++o) msg[t].push_back(joint(t, o, 0) + joint(t, o, 1));
  for (int bwd = 0; bwd < 2; ++bwd) {
    SweepPlan pl;
    build_sweep(P, {1}, S, waves, bwd, walk, pl);
    const SweepInst &W = pl.insts.at(0);
    // every wave's records with the number of barriers before them, by phase
    struct R { int wave; const int32_t *r; };
    std::vector<std::vector<R>> phases;
    size_t total = 0;
    for (int k = 0; k < waves; ++k) {
      size_t ph = 0;
      for (int64_t i = W.prog[k];; ++i) {
        CHECK((i + 2) * kSweepRec <= (int64_t)pl.prog.size());
        const int32_t *r = &pl.prog.at(i * kSweepRec);
        ph += (r[0] >> 4) & 0xff;
        if (phases.size() <= ph) phases.resize(ph + 1);
        if ((r[0] & 15) == SWEEP_END) {
          CHECK((pl.prog.at((i + 1) * kSweepRec) & 15) == SWEEP_END);
          break;
        }
        phases[ph].push_back({k, r});
        // transfer entries loaded ahead for the next record
        const int32_t *nx = r + kSweepRec;
        const bool un = (nx[0] & 15) == SWEEP_FWD || (nx[0] & 15) == SWEEP_JOINT;
        CHECK(r[16] == (un ? nx[2] : 0) && (r[17] & 15) == (un ? (nx[0] >> 12) & 15 : 0));
        CHECK(r[17] >> 8 == (un ? (nx[0] >> 24) & 15 : 0));
        CHECK(r[18] == (un || (nx[0] & 15) == SWEEP_MARG ? nx[19] : 0));
        CHECK(r[18] + E <= (int)pl.lanes.size() && r[19] + E <= (int)pl.lanes.size());
        if (i == W.prog[k])   // the first record's own words are read as a unit's
          CHECK(r[2] + std::min(E, 1 << ((r[0] >> 24) & 15)) + (1 << ((r[0] >> 12) & 15)) <= (int64_t)P.T.size());
      }
      if (k == 0) total = ph;
      CHECK(ph == total);
    }
    CHECK(phases.size() == total + 1);
    std::vector<double> arena(W.arena, NAN);
    std::vector<int> owner(W.arena, -1);
    auto walk_at = [](int c, int code) {
      int e = 0;
      for (int b = 0; b < kSweepWalk; ++b)
        if ((c >> b) & 1) e += (1 << ((code >> (4 * b)) & 15)) & 0x7fff;
      return e;
    };
    struct U { int t, w, n_in, dense, n_edge, n, off, tpos, scr, gpos, slot, ebits, o0; };
    auto unit = [](const int32_t *r) {
      return U{r[4] & 0xffff, (r[0] >> 12) & 15, (r[0] >> 16) & 7, (r[0] >> 19) & 1, (r[0] >> 20) & 7,
               1 << ((r[0] >> 24) & 15), r[1], r[2], r[3], r[4] >> 16, r[5], r[6], r[7]};
    };
    std::vector<int> read_in(W.arena, -1);
    int phase = 0;
    auto weights = [&](const int32_t *r, const U &u, int lo, int c, double &p0, double &p1) {
      const int o = lo + c * E;
      p0 = P.T.at(u.tpos + o) * phi(u.gpos, 0);
      p1 = P.T.at(u.tpos + o + (1 << u.w)) * phi(u.gpos, 1);
      for (int k = 0; k < u.n_in; ++k) {
        const int m = r[9 + 2 * k], step = m >> 16, xs = 1 << ((m >> 12) & 15);
        const int e = r[8 + 2 * k] + ((pl.lanes.at(r[19] + lo) >> (8 * k)) & 0xff) + walk_at(c, m);
        CHECK(owner.at(e) == step && owner.at(e + xs) == step);
        read_in.at(e) = read_in.at(e + xs) = phase;
        p0 *= arena.at(e);
        p1 *= arena.at(e + xs);
      }
      return u.o0 + o;
    };
    // reverse: rho by direct sums of the joint weights
    std::vector<std::vector<double>> rho(D.n_steps);
    for (int t = 0; t < D.n_steps; ++t) rho[t].assign(msg[t].size(), st[t].w ? 0.0 : 1.0 / msg[t][0]);
    for (int t = D.n_steps - 1; t >= 0; --t)
      for (int k = 0; k < st[t].n_in; ++k) {
        const InputDesc &id = P.inputs[st[t].in_off + k];
        std::vector<double> mu(msg[id.step].size(), 0.0);
        for (int o = 0; o < 1 << st[t].w; ++o)
          for (int x = 0; x < 2; ++x)
            mu[st[t].kind == STEP_DENSE ? x : gather(id, o, x)] += joint(t, o, x) * rho[t][o];
        for (size_t j = 0; j < mu.size(); ++j) rho[id.step][j] = mu[j] / msg[id.step][j];
      }
    std::vector<int> sums(D.nr, 0), made(D.n_steps, 0);
    std::vector<double> scr(W.scr, NAN), red(W.slots, NAN);
    int closed = 0;
    for (auto &ph : phases) {
      // a phase's writes take effect after its reads
      std::vector<std::pair<int, std::pair<int, double>>> writes;
      std::vector<std::pair<int, double>> wscr, wred;
      for (auto &it : ph) {
        const int32_t *r = it.r;
        const int op = r[0] & 15;
        if (op == SWEEP_FWD || op == SWEEP_JOINT) {
          const U u = unit(r);
          const int nc = u.n > E ? u.n / E : 1;
          CHECK(nc <= 1 << walk && u.n <= 1 << u.w && u.o0 + u.n <= 1 << u.w && u.gpos == st[u.t].gpos);
          for (int lo = 0; lo < E; ++lo)   // (lanes past the entries repeat lane mod n)
            CHECK(pl.lanes.at(r[19] + lo) == pl.lanes.at(r[19] + (lo & (u.n - 1))));
          CHECK(u.w == st[u.t].w && u.n_in == st[u.t].n_in && u.n_edge == st[u.t].n_edge);
          double v[1 + kSweepEdges] = {0, 0, 0, 0, 0};
          for (int lo = 0; lo < std::min(E, u.n); ++lo)
            for (int c = 0; c < nc; ++c) {
              double p0, p1;
              const int o = weights(r, u, lo, c, p0, p1);
              if (op == SWEEP_FWD) {
                CHECK(near(p0 + p1, msg[u.t].at(o)));
                writes.push_back({u.off + lo + c * E, {u.t, p0 + p1}});
                ++made[u.t];
                continue;
              }
              const double raw = arena.at(u.off + lo + c * E), rr = u.w == 0 ? 1.0 / raw : raw;
              CHECK(near(rr, rho[u.t].at(o)));
              p0 *= rr;
              p1 *= rr;
              wscr.push_back({u.scr + lo + c * E, p0});
              wscr.push_back({u.scr + (1 << u.w) + lo + c * E, p1});
              v[0] += p0 - p1;
              for (int k = 0; k < u.n_edge; ++k)
                v[1 + k] += ((o >> ((u.ebits >> (8 * k)) & 0xff)) & 1) ? p1 - p0 : p0 - p1;
            }
          if (op == SWEEP_JOINT)
            for (int k = 0; k <= u.n_edge; ++k) wred.push_back({u.slot + k, v[k]});
        } else if (op == SWEEP_MARG) {
          const int lc = (r[0] >> 12) & 15, n = 1 << ((r[0] >> 16) & 15);
          for (int lo = 0; lo < E; ++lo)
            CHECK(pl.lanes.at(r[19] + lo) == pl.lanes.at(r[19] + (lo & (n - 1))));
          CHECK(n >= 1 << lc && 1 << lc <= E && (n <= E || n / E <= 1 << kSweepWalk));
          std::vector<double> part(n >> lc, 0.0);
          for (int i = 0; i < n; ++i) {
            const int lo = i % E, c = i / E;
            int z = 0;
            for (int k = 0; k < 1 << __builtin_popcount((unsigned)r[5]); ++k) {
              part.at(((lo >> lc) + c * (E >> lc))) += scr.at(r[1] + pl.lanes.at(r[19] + lo) + walk_at(c, r[2]) + z);
              z = (z - r[5]) & r[5];
            }
          }
          for (int j = 0; j < n >> lc; ++j) {
            CHECK(owner.at(r[3] + j) == r[4]);
            writes.push_back({r[3] + j, {r[4], part[j] / arena.at(r[3] + j)}});
          }
        } else if (op == SWEEP_SUM) {
          int t = 0;
          while (st[t].gpos != r[4]) ++t;
          ++sums.at(r[4]);
          const int ne = (r[0] >> 20) & 7;
          CHECK(ne == st[t].n_edge);
          for (int k = 0; k <= ne; ++k) {
            double got = 0, w = 0;
            for (int i = 0; i < r[3]; ++i) got += red.at(r[1] + i * r[2] + k);
            const EdgeDesc *e = k ? &P.edges[st[t].edge_off + k - 1] : nullptr;
            for (int o = 0; o < 1 << st[t].w; ++o) {
              const double d = (joint(t, o, 0) - joint(t, o, 1)) * rho[t][o];
              w += e && ((o >> e->bv) & 1) ? -d : d;
            }
            CHECK(!e || e->rr == r[4 + k]);
            CHECK(std::fabs(got - w) <= 1e-11);
          }
        } else if (op == SWEEP_LOGZ) {
          double lz = 0, want = 0;
          for (int i = 0; i < W.n_close; ++i) lz += std::log(arena.at(pl.close.at(W.close_off + 2 * i)));
          for (int t = 0; t < D.n_steps; ++t)
            if (st[t].w == 0) want += std::log(msg[t][0]);
          CHECK(near(lz, want) && it.wave == 0);
          ++closed;
        } else {
          CHECK(op == SWEEP_WAIT);
        }
      }
      auto once = [](auto &v) {
        std::sort(v.begin(), v.end());
        for (size_t i = 0; i + 1 < v.size(); ++i) CHECK(v[i].first != v[i + 1].first);
      };
      once(writes);
      once(wscr);
      once(wred);
      for (auto &w : writes) {
        CHECK(read_in.at(w.first) != phase);   // no entry is read and written in one phase
        arena.at(w.first) = w.second.second;
        owner.at(w.first) = w.second.first;
      }
      for (auto &w : wscr) scr.at(w.first) = w.second;
      for (auto &w : wred) red.at(w.first) = w.second;
      ++phase;
    }
    CHECK(closed == 1);
    for (int t = 0; t < D.n_steps; ++t) CHECK(made[t] == 1 << st[t].w);
    if (bwd)
      for (int n : sums) CHECK(n == 1);
  }
}

// The segments of a program with wide steps: every step once, after its
// inputs; the wide steps' tables cover every entry and index every input as
// the program does; every sum over an input's missing bits is whole.
static void check_wide(const HostProgram &P) {
  const InstDesc &D = P.insts[0];
  const StepDesc *st = P.steps.data() + D.step_off;
  WidePlan pl;
  build_wide(P, {1}, pl);
  std::vector<int> made(D.n_steps, 0), back(D.n_steps, 0);
  int closed = 0;
  size_t n_sums = 0;
  auto whole = [&](int t) {
    for (int k = 0; k < st[t].n_in; ++k) CHECK(made[P.inputs[st[t].in_off + k].step] == 1 << st[P.inputs[st[t].in_off + k].step].w);
  };
  for (auto &sg : pl.segs.at(0)) {
    for (int rev = 0; rev < 2; ++rev) {
      // records by the barriers before them
      std::vector<std::vector<const int32_t *>> phases;
      size_t total = 0;
      for (int k = 0; k < kSweepWaves; ++k) {
        size_t ph = 0;
        for (int64_t i = rev ? sg.bwd[k] : sg.fwd[k];; ++i) {
          CHECK((i + 2) * kSweepRec <= (int64_t)pl.prog.size());
          const int32_t *r = &pl.prog.at(i * kSweepRec);
          ph += (r[0] >> 4) & 0xff;
          if (phases.size() <= ph) phases.resize(ph + 1);
          if ((r[0] & 15) == SWEEP_END) break;
          phases[ph].push_back(r);
        }
        if (k == 0) total = ph;
        CHECK(ph == total);
      }
      for (auto &ph : phases) {
        std::vector<std::pair<int, int>> add;
        for (const int32_t *r : ph) {
          const int op = r[0] & 15, t = r[4] & 0xffff;
          if (op == SWEEP_LOGZ) ++closed;
          if (op != SWEEP_FWD && op != SWEEP_JOINT) continue;
          CHECK(st[t].w < kWideStep && (op == SWEEP_JOINT) == (rev == 1));
          if (!rev) whole(t);
          add.push_back({t, 1 << ((r[0] >> 24) & 15)});
        }
        for (auto &a : add) (rev ? back : made)[a.first] += a.second;
      }
    }
    for (auto &g : sg.groups) {
      int blocks = 0, fblocks = 0;
      std::vector<int> part_use(pl.part.at(0), 0);
      for (int i = g.w0; i < g.w1; ++i) whole(pl.steps.at(i).step);
      for (int i = g.w0; i < g.w1; ++i) {
        const WideStep &w = pl.steps.at(i);
        const StepDesc &sd = st[w.step];
        const int nb = 1 << (w.w - kWideChunk), high = kWideThreads + kWideRegs;
        blocks += nb;
        CHECK(w.w == sd.w && w.w >= kWideStep && w.gpos == sd.gpos && w.off == sd.off_all &&
              w.n_in == sd.n_in && w.n_edge == sd.n_edge && w.t_off == sd.t_off);
        CHECK(w.red + nb * (1 + w.n_edge) <= pl.red.at(0));
        n_sums += 1 + w.n_edge;
        std::vector<int> seen(1 << w.w, 0);
        auto at = [&](int tab, int c, int b) {
          return pl.tab.at(tab + c % kWideThreads) | pl.tab.at(tab + kWideThreads + c / kWideThreads) |
                 pl.tab.at(tab + high + b);
        };
        for (int b = 0; b < nb; ++b)
          for (int c = 0; c < 1 << kWideChunk; ++c) {
            const int o = at(w.out, c, b);
            CHECK((o & 31) == (c & 31));
            ++seen.at(o);
          }
        for (int n : seen) CHECK(n == 1);
        for (int k = 0; k < w.n_in; ++k) {
          const InputDesc &id = P.inputs[sd.in_off + k];
          const WideInput &in = w.in[k];
          CHECK(in.off == st[id.step].off_all && in.step == id.step && in.bits == id.nbits &&
                in.xbit == id.xbit && id.nbits == st[id.step].w);
          const int ns = kWideChunk - __builtin_popcount((unsigned)in.free);
          // terms each entry's sums take (spin +1), by row
          const WideFin *fin = nullptr;
          for (int f = g.f0; f < g.f1; ++f)
            if (in.part >= 0 && pl.fins.at(f).part == in.part) fin = &pl.fins.at(f);
          CHECK((in.part >= 0) == (fin != nullptr));
          if (fin) {
            CHECK(fin->off == in.off && fin->step == in.step && fin->nbits == in.bits);
            CHECK(fin->first == fblocks);
            fblocks += std::max(1, (1 << fin->nbits) / kWideThreads);
          }
          const int rows = fin ? fin->rows : 1;
          std::vector<int> terms((size_t)rows << id.nbits, 0);
          for (int b = 0; b < nb; ++b) {
            const int row = fin ? pl.tab.at(in.row + b) : 0;
            CHECK(row < rows);
            for (int e = 0; e < 1 << ns; ++e) {
              const uint32_t d = (uint32_t)pl.tab.at(in.dep + e);
              const int c0 = (int)(d & ((1u << kWideChunk) - 1));
              const int j = pl.tab.at(in.idx + high + b) | (int)(d >> kWideChunk);
              CHECK(!(c0 & in.free));
              for (int z = 0, m = 0; m < 1 << (kWideChunk - ns); ++m, z = (z - in.free) & in.free) {
                const int o = at(w.out, c0 | z, b);
                int want = 0;
                for (int x = 0; x < id.nbits; ++x)
                  if (id.src[x] >= 0) want |= ((o >> id.src[x]) & 1) << x;
                CHECK(want == j && want == at(in.idx, c0 | z, b));
              }
              ++terms.at(((size_t)row << id.nbits) + j);
            }
          }
          for (int r = 0; r < rows; ++r)
            for (int j = 0; j < 1 << id.nbits; ++j) {
              CHECK(terms[((size_t)r << id.nbits) + j] == !((j >> id.xbit) & 1));
              if (fin) ++part_use.at(fin->part + (r << id.nbits) + j);
            }
          const int nf = w.w - (id.nbits - 1);
          CHECK(((kWideChunk - ns) == nf) == (rows == 1) && rows == 1 << (nf - (kWideChunk - ns)));
        }
      }
      for (int n : part_use) CHECK(n <= 1);
      for (int i = g.w0; i < g.w1; ++i) made[pl.steps[i].step] = back[pl.steps[i].step] = 1 << pl.steps[i].w;
      CHECK(blocks == g.blocks && fblocks == g.fblocks);
    }
  }
  for (int t = 0; t < D.n_steps; ++t) CHECK(made[t] == 1 << st[t].w && back[t] == 1 << st[t].w);
  CHECK(closed == 1 && n_sums == pl.sums.size() && pl.sum_lo.at(1) == (int)pl.sums.size());
}

int main() {
  std::mt19937_64 rng(5);
  int done = 0;
  int wide = 0;
  for (int trial = 0; trial < 90; ++trial) {
    // (the last thirty: wide programs)
    const int n = trial < 60 ? 6 + (int)(rng() % 60) : 45 + (int)(rng() % 20), d = trial < 60 ? 1 + (int)(rng() % 3) : 3;
    std::vector<std::vector<char>> adj(n, std::vector<char>(n, 0));
    std::vector<int32_t> ei, ej, W, order;
    std::vector<double> J;
    for (int k = 0; k < n * d / 2; ++k) {
      int a = (int)(rng() % n), b = (int)(rng() % n);
      if (a > b) std::swap(a, b);
      if (a == b || adj[a][b]) continue;
      adj[a][b] = 1;
      ei.push_back(a);
      ej.push_back(b);
      J.push_back((rng() & 1) ? 0.7 : -0.4);
    }
    std::vector<int> perm(n);
    for (int i = 0; i < n; ++i) perm[i] = i;
    std::shuffle(perm.begin(), perm.end(), rng);
    const int m = trial < 60 ? (int)(rng() % (n / 2)) : (int)(rng() % 6);
    for (int i = 0; i < n; ++i) (i < m ? W : order).push_back(perm[i]);
    std::vector<double> h(n, 0.1);
    tnvan_instance in{};
    in.n_spins = n;
    in.n_edges = (int32_t)ei.size();
    in.edge_i = ei.data();
    in.edge_j = ej.data();
    in.J = J.data();
    in.h = h.data();
    in.beta = 0.8;
    in.n_width = (int32_t)W.size();
    in.width_set = W.data();
    in.n_order = (int32_t)order.size();
    in.order = order.data();
    HostProgram P;
    std::string msg;
    if (trial >= 60) {
      if (compile_instance(in, 17, P, msg) != TNVAN_OK || P.insts[0].max_w < kWideStep || !wide_fits(P, 0)) continue;
      ++wide;
      check_wide(P);
      continue;
    }
    if (compile_instance(in, 12, P, msg) != TNVAN_OK || !sweep_fits(P, 0)) continue;
    ++done;
    for (int S : {1, 2, 4, 16, 64})
      for (int walk = 0; walk <= kSweepWalk; ++walk) check(P, S, 1 << (int)(rng() % 4), walk);
  }
  if (g_fail || done < 20 || wide < 5) return std::fprintf(stderr, "%d failed, %d and %d programs\n", g_fail, done, wide), 1;
  std::printf("sweep schedule ok (%d programs, %d with wide steps)\n", done, wide);
  return 0;
}
