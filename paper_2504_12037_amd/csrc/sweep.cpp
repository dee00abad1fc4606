// Host schedule of the level kernels (see sweep.h).  Pure C++.
#include "sweep.h"

#include <algorithm>
#include <map>

#include "compile.h"

namespace tnvan {

namespace {

// a step the level programs take
bool step_fits(const HostProgram &P, const InstDesc &D, const StepDesc &sd) {
  (void)D;
  if (sd.g != 1 || sd.w > kTabW || sd.t_off < 0 || sd.t_off > INT32_MAX - (2 << kTabW) ||
      sd.n_in > kSweepIn || sd.n_edge > kSweepEdges)
    return false;
  if (sd.kind == STEP_DENSE && sd.n_in > 1) return false;
  for (int k = 0; k < sd.n_edge; ++k) {
    const EdgeDesc &e = P.edges[sd.edge_off + k];
    if (e.bu != sd.w || e.bv < 0 || e.bv >= sd.w) return false;
  }
  for (int k = 0; k < sd.n_in; ++k) {
    const InputDesc &id = P.inputs[sd.in_off + k];
    if (id.xbit < 0 && sd.kind != STEP_DENSE) return false;
  }
  return true;
}

}  // namespace

bool sweep_fits(const HostProgram &P, int q) {
  const InstDesc &D = P.insts[q];
  // (records hold steps and positions in 15 bits)
  if (D.n_steps <= 0 || D.n_steps > 32767 || D.nr > 32767) return false;
  for (int t = 0; t < D.n_steps; ++t)
    if (!step_fits(P, D, P.steps[D.step_off + t])) return false;
  return true;
}

bool wide_fits(const HostProgram &P, int q) {
  const InstDesc &D = P.insts[q];
  if (D.n_steps <= 0 || D.n_steps > 32767 || D.nr > 32767) return false;
  for (int t = 0; t < D.n_steps; ++t) {
    const StepDesc &sd = P.steps[D.step_off + t];
    if (sd.w < kWideStep) {
      if (!step_fits(P, D, sd)) return false;
      continue;
    }
    if (sd.g != 1 || sd.kind != STEP_SINGLE || sd.n_in < 1 || sd.n_edge > kWideEdges ||
        sd.n_in > (sd.t_off < 0 ? kWideIn : kSweepIn))
      return false;
    for (int k = 0; k < sd.n_edge; ++k) {
      const EdgeDesc &e = P.edges[sd.edge_off + k];
      if (e.bu != sd.w || e.bv < 0 || e.bv >= sd.w) return false;
    }
  }
  return true;
}

namespace {

int ilog2(int x) {
  int r = 0;
  while ((1 << r) < x) ++r;
  return r;
}

// first-fit arena with exact-size reuse of freed ranges
struct Reuse {
  std::vector<std::pair<int32_t, int32_t>> free;   // offset, size
  int32_t top = 0;
  int32_t take(int32_t n) {
    size_t best = free.size();
    for (size_t i = 0; i < free.size(); ++i)
      if (free[i].second >= n && (best == free.size() || free[i].second < free[best].second)) best = i;
    if (best == free.size()) {
      const int32_t at = top;
      top += n;
      return at;
    }
    const int32_t at = free[best].first;
    free[best].first += n;
    free[best].second -= n;
    if (free[best].second == 0) free.erase(free.begin() + (long)best);
    return at;
  }
  void give(int32_t at, int32_t n) {
    free.push_back({at, n});
    std::sort(free.begin(), free.end());
    std::vector<std::pair<int32_t, int32_t>> m;
    for (auto &f : free) {
      if (!m.empty() && m.back().first + m.back().second == f.first) m.back().second += f.second;
      else m.push_back(f);
    }
    free.swap(m);
  }
};

// The programs under construction: the units of a phase go to the waves by
// cost, the costliest first, each to the wave with the least so far.
struct Builder {
  int waves;
  std::vector<int32_t> rec[kSweepWaves];
  int bars[kSweepWaves] = {};
  std::vector<std::pair<int, std::vector<int32_t>>> phase;   // cost, record
  void add(int cost, std::vector<int32_t> r) {
    r.resize(kSweepRec, 0);
    phase.push_back({cost, std::move(r)});
  }
  void put(int wave, std::vector<int32_t> r) {
    r.resize(kSweepRec, 0);
    // (eight bits of barriers per record; long waits take empty records)
    while (bars[wave] > 255) {
      std::vector<int32_t> e(kSweepRec, 0);
      e[0] = SWEEP_WAIT | (255 << 4);
      bars[wave] -= 255;
      rec[wave].insert(rec[wave].end(), e.begin(), e.end());
    }
    r[0] |= bars[wave] << 4;
    bars[wave] = 0;
    rec[wave].insert(rec[wave].end(), r.begin(), r.end());
  }
  void flush() {   // the phase's units, then a barrier
    std::stable_sort(phase.begin(), phase.end(),
                     [](const auto &a, const auto &b) { return a.first > b.first; });
    int64_t load[kSweepWaves] = {};
    for (auto &p : phase) {
      int w = 0;
      for (int k = 1; k < waves; ++k)
        if (load[k] < load[w]) w = k;
      load[w] += p.first;
      put(w, std::move(p.second));
    }
    phase.clear();
    for (int k = 0; k < waves; ++k) ++bars[k];
  }
};

// Level programs of one instance: its output arrays, tile and walk limits.
struct Levels {
  const HostProgram &P;
  const InstDesc &D;
  const StepDesc *st;
  int S, waves, max_walk, E, logE, max_w;   // max_w: widest step of the level programs
  std::vector<int32_t> &prog, &lanes;
  std::map<std::vector<int32_t>, int32_t> &known;
  std::vector<int32_t> off;     // arena offset of every step's message
  int32_t scr_max = 0, slot_max = 0;
  Builder B{};

  // lane words, E in a row, each kind once
  int32_t lane_words(const std::vector<int32_t> &w) {
    auto it = known.find(w);
    if (it != known.end()) return it->second;
    const int32_t at = (int32_t)lanes.size();
    lanes.insert(lanes.end(), w.begin(), w.end());
    known[w] = at;
    return at;
  }

  // passes per unit of a level: as many as leave every wave a unit
  int walk_of(const std::vector<int> &at) const {
    int walk = max_walk;
    auto units_at = [&](int wk) {
      int64_t n = 0;
      for (int t : at) n += std::max(1, (1 << st[t].w) >> (logE + wk));
      return n;
    };
    while (walk > 0 && units_at(walk) < waves) --walk;
    return walk;
  }

  // units of a step; slot advances over the level
  void step_units(int t, int wk, SweepOp op, int32_t scr, int32_t &slot) {
    const StepDesc &sd = st[t];
    const int N = 1 << sd.w, per = std::min(N, E << wk);
    int32_t ebits = 0;
    for (int k = 0; k < sd.n_edge; ++k) ebits |= P.edges[sd.edge_off + k].bv << (8 * k);
    for (int o0 = 0; o0 < N; o0 += per) {
      std::vector<int32_t> r(kSweepRec, 0);
      r[0] = op | (sd.w << 12) | (sd.n_in << 16) | ((sd.kind == STEP_DENSE ? 1 : 0) << 19) |
             (sd.n_edge << 20) | (ilog2(per) << 24);
      r[1] = off[t] + o0;
      r[2] = (int32_t)sd.t_off + o0;
      r[3] = scr + o0;
      r[4] = t | (sd.gpos << 16);
      r[5] = slot;
      r[6] = ebits;
      r[7] = o0;
      std::vector<int32_t> lw(E, 0);
      for (int k = 0; k < sd.n_in; ++k) {
        const InputDesc &id = P.inputs[sd.in_off + k];
        const bool dense = sd.kind == STEP_DENSE;   // the message over the spin alone
        int32_t base = off[id.step], meta = 0xfff;
        for (int b = 0; b < id.nbits && !dense; ++b) {
          const int ob = id.src[b];
          if (ob < 0) continue;
          if ((o0 >> ob) & 1) base += 1 << b;
          if (ob < logE) {
            for (int lo = 0; lo < E; ++lo)
              if ((lo >> ob) & 1) lw[lo] |= 1 << (8 * k + b);
          } else if (ob < logE + kSweepWalk) {
            const int at4 = 4 * (ob - logE);
            meta = (meta & ~(15 << at4)) | (b << at4);
          }
        }
        r[8 + 2 * k] = base;
        r[9 + 2 * k] = meta | ((dense ? 0 : id.xbit) << 12) | (id.step << 16);
      }
      r[19] = lane_words(lw);
      slot += 1 + sd.n_edge;
      B.add(8 + (per + E - 1) / E * (2 + sd.n_in), std::move(r));
    }
  }

  void forward(const std::vector<int> &at) {
    int32_t slot = 0;
    const int wk = walk_of(at);
    for (int t : at) step_units(t, wk, SWEEP_FWD, 0, slot);
    B.flush();
  }

  // A level's steps are independent: in tiles of more than two samples they
  // run in batches whose joint weights take no more scratch than the widest
  // step of the program, so that tiles of four and eight fit (each batch is
  // two more phases; smaller tiles fit without).  Adjoint of 4096 samples of
  // a 256-spin random graph at four per tile 1147 -> 721 us, of a 64-spin one
  // at eight 423 -> 262 us.
  void reverse(const std::vector<int> &at) {
    std::vector<int> batch, order(at);
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return st[x].w > st[y].w; });
    int32_t used = 0;
    for (int t : order) {
      const int32_t need = 2 << st[t].w;
      if (used > 0 && S > 2 && used + need > 2 << max_w) {
        reverse_batch(batch);
        batch.clear();
        used = 0;
      }
      batch.push_back(t);
      used += need;
    }
    if (!batch.empty()) reverse_batch(batch);
  }

  void reverse_batch(const std::vector<int> &at) {
    const int wk = walk_of(at);
    int32_t scr = 0, slot = 0;
    std::vector<int32_t> scr_of, slot_of;
    for (int t : at) {
      scr_of.push_back(scr);
      slot_of.push_back(slot);
      step_units(t, wk, SWEEP_JOINT, scr, slot);
      scr += 2 << st[t].w;
    }
    scr_max = std::max(scr_max, scr);
    slot_max = std::max(slot_max, slot);
    B.flush();
    // marginals: lanes that share a sum, and passes per unit
    struct Marg { int i, k, lc; };
    std::vector<Marg> ms;
    int64_t passes = 0;
    for (size_t i = 0; i < at.size(); ++i) {
      const StepDesc &sd = st[at[i]];
      const int per = std::min(1 << sd.w, E << wk);
      std::vector<int32_t> s = {SWEEP_SUM | (sd.n_edge << 20), slot_of[i], 1 + sd.n_edge,
                                (1 << sd.w) / per, sd.gpos};
      for (int k = 0; k < sd.n_edge; ++k) s.push_back(P.edges[sd.edge_off + k].rr);
      B.add(6 + (1 << sd.w) / per, std::move(s));
      for (int k = 0; k < sd.n_in; ++k) {
        const InputDesc &id = P.inputs[sd.in_off + k];
        const int nfree = sd.w + 1 - id.nbits;
        // share a sum among lanes until the workgroup's waves are filled
        // or each lane keeps four terms
        int lc = 0;
        while (lc < logE && lc < nfree &&
               (((1 << id.nbits) << lc) < E ||
                (((1 << id.nbits) << lc) < E * waves && nfree - lc > 2)))
          ++lc;
        ms.push_back({(int)i, k, lc});
        passes += std::max(1, (1 << (id.nbits + lc)) / E);
      }
    }
    int mwalk = kSweepWalk;
    while (mwalk > 0 && (passes >> mwalk) < waves) --mwalk;
    for (const Marg &m : ms) {
      const StepDesc &sd = st[at[m.i]];
      const InputDesc &id = P.inputs[sd.in_off + m.k];
      // output bits of an item's bits: the lanes that share a sum (free
      // output bits, lowest first), then the entry's bits
      const bool dense = sd.kind == STEP_DENSE;
      int rest = ((1 << sd.w) - 1) & ~(dense ? 0 : id.omask);
      std::vector<int> pos;
      for (int b = 0; b < m.lc; ++b) {
        pos.push_back(ilog2(rest & -rest));
        rest &= rest - 1;
      }
      for (int b = 0; b < id.nbits; ++b) pos.push_back(dense || id.src[b] < 0 ? sd.w : id.src[b]);
      const int items = 1 << (id.nbits + m.lc), pm = std::min(items, E << mwalk);
      std::vector<int32_t> lw(E, 0);
      for (int b = 0; b < logE && b < (int)pos.size(); ++b)
        for (int lo = 0; lo < E; ++lo)
          if ((lo >> b) & 1) lw[lo] |= 1 << pos[b];
      int32_t code = 0xfff;
      for (int b = 0; b < kSweepWalk && logE + b < (int)pos.size(); ++b)
        code = (code & ~(15 << (4 * b))) | (pos[logE + b] << (4 * b));
      const int32_t at_lanes = lane_words(lw);
      for (int i0 = 0; i0 < items; i0 += pm) {
        int32_t base = scr_of[m.i];
        for (size_t b = 0; b < pos.size(); ++b)
          if ((i0 >> b) & 1) base += 1 << pos[b];
        std::vector<int32_t> r = {SWEEP_MARG | (m.lc << 12) | (ilog2(pm) << 16), base, code,
                                  off[id.step] + (i0 >> m.lc), id.step, rest};
        r.resize(kSweepRec, 0);
        r[19] = at_lanes;
        B.add(8 + std::max(1, pm / E) * (4 + (1 << __builtin_popcount((unsigned)rest))), std::move(r));
      }
    }
    B.flush();
  }

  // ends the waves' programs and appends them; start[k]: first record
  void finish(int32_t (&start)[kSweepWaves]) {
    for (int k = 0; k < waves; ++k) {
      // before its program a wave loads transfer factors by its first
      // record's own words (2: offset), so a record that holds something else
      // there goes behind an empty one
      if (!B.rec[k].empty() && (B.rec[k][0] & 15) != SWEEP_FWD && (B.rec[k][0] & 15) != SWEEP_JOINT) {
        std::vector<int32_t> e(kSweepRec, 0);
        e[0] = SWEEP_WAIT;
        B.rec[k].insert(B.rec[k].begin(), e.begin(), e.end());
      }
      B.put(k, {SWEEP_END});
      B.put(k, {SWEEP_END});   // the record loaded ahead of the last
      // (word 19, a record's own lane words, serves the first record)
      for (size_t i = 0; i + kSweepRec < B.rec[k].size(); i += kSweepRec) {
        const int32_t *next = &B.rec[k][i + kSweepRec];
        const int op = next[0] & 15;
        if (op == SWEEP_FWD || op == SWEEP_JOINT) {
          B.rec[k][i + 16] = next[2];
          B.rec[k][i + 17] = ((next[0] >> 12) & 15) | (((next[0] >> 24) & 15) << 8);
        }
        if (op == SWEEP_FWD || op == SWEEP_JOINT || op == SWEEP_MARG) B.rec[k][i + 18] = next[19];
      }
      start[k] = (int32_t)(prog.size() / kSweepRec);
      prog.insert(prog.end(), B.rec[k].begin(), B.rec[k].end());
    }
    B = Builder{};
    B.waves = waves;
  }
};

// steps by level (0 without inputs among those with use[t])
std::vector<std::vector<int>> by_level(const HostProgram &P, const InstDesc &D,
                                       const std::vector<char> &use) {
  const StepDesc *st = P.steps.data() + D.step_off;
  std::vector<int> level(D.n_steps, 0);
  std::vector<std::vector<int>> at;
  for (int t = 0; t < D.n_steps; ++t) {
    if (!use[t]) continue;
    for (int k = 0; k < st[t].n_in; ++k) {
      const int u = P.inputs[st[t].in_off + k].step;
      if (use[u]) level[t] = std::max(level[t], level[u] + 1);
    }
    if ((int)at.size() <= level[t]) at.resize(level[t] + 1);
    at[level[t]].push_back(t);
  }
  return at;
}

void closings(const HostProgram &P, const InstDesc &D, const std::vector<int32_t> &off,
              std::vector<int32_t> &close, SweepInst &si) {
  si.close_off = (int32_t)close.size();
  for (int t = 0; t < D.n_steps; ++t)
    if (P.steps[D.step_off + t].w == 0) {
      close.push_back(off[t]);
      close.push_back(t);
    }
  si.n_close = ((int32_t)close.size() - si.close_off) / 2;
}

// Step t as a wide step: its chunk bits, tables, sums and the finishing of
// its inputs; part and red: scratch words taken so far.
void wide_step(const HostProgram &P, const InstDesc &D, int t, int32_t &part, int32_t &red,
               WidePlan &out, WideGroup &g) {
  const StepDesc &sd = P.steps[D.step_off + t];
  const InputDesc *ids = P.inputs.data() + sd.in_off;
  const int blocks = 1 << (sd.w - kWideChunk), all = (1 << sd.w) - 1;
  // output bits of the chunk's positions, ascending
  int chunk = 31;
  std::vector<int> order;
  for (int k = 0; k < sd.n_in; ++k) order.push_back(k);
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return ids[x].nbits > ids[y].nbits; });
  auto take = [&](int mask) {
    for (int b = 0; b < sd.w; ++b)
      if (((mask & ~chunk) >> b) & 1 && __builtin_popcount((unsigned)chunk) < kWideChunk) chunk |= 1 << b;
  };
  for (int k : order) take(all & ~ids[k].omask);
  take(all);
  std::vector<int> cb, hb;
  for (int b = 0; b < sd.w; ++b) ((chunk >> b) & 1 ? cb : hb).push_back(b);
  auto spread = [](int v, const std::vector<int> &bits, size_t from) {
    int o = 0;
    for (size_t b = from; b < bits.size(); ++b)
      if ((v >> (b - from)) & 1) o |= 1 << bits[b];
    return o;
  };
  const int lt = ilog2(kWideThreads);
  std::vector<int> os;   // the parts of o the tables run over
  for (int j = 0; j < kWideThreads; ++j)
    os.push_back(spread(j, std::vector<int>(cb.begin(), cb.begin() + lt), 0));
  for (int j = 0; j < kWideRegs; ++j) os.push_back(spread(j, cb, lt));
  for (int j = 0; j < blocks; ++j) os.push_back(spread(j, hb, 0));
  WideStep w{};
  w.step = t;
  w.gpos = sd.gpos;
  w.w = sd.w;
  w.n_in = sd.n_in;
  w.n_edge = sd.n_edge;
  w.off = sd.off_all;
  w.edge_off = sd.edge_off;
  w.t_off = sd.t_off;
  w.red = red;
  out.sums.push_back({red, 1 + sd.n_edge, blocks, -1 - sd.gpos});
  for (int k = 0; k < sd.n_edge; ++k)
    out.sums.push_back({red + 1 + k, 1 + sd.n_edge, blocks, P.edges[sd.edge_off + k].rr});
  red += blocks * (1 + sd.n_edge);
  w.out = (int32_t)out.tab.size();
  out.tab.insert(out.tab.end(), os.begin(), os.end());
  for (int k = 0; k < sd.n_in; ++k) {
    const InputDesc &id = ids[k];
    WideInput &in = w.in[k];
    in.off = P.steps[D.step_off + id.step].off_all;
    in.step = id.step;
    in.xbit = id.xbit;
    in.bits = id.nbits;
    auto index = [&](int o) {
      int e = 0;
      for (int b = 0; b < id.nbits; ++b)
        if (id.src[b] >= 0 && ((o >> id.src[b]) & 1)) e |= 1 << b;
      return e;
    };
    in.idx = (int32_t)out.tab.size();
    for (int o : os) out.tab.push_back(index(o));
    const int freem = all & ~id.omask;
    for (int b = 0; b < kWideChunk; ++b)
      if ((freem >> cb[b]) & 1) in.free |= 1 << b;
    in.dep = (int32_t)out.tab.size();
    for (int i = 0; i < 1 << kWideChunk; ++i)
      if (!(i & in.free)) out.tab.push_back(i | (int32_t)((uint32_t)index(spread(i, cb, 0)) << kWideChunk));
    in.row = (int32_t)out.tab.size();
    std::vector<int> hf;
    for (int b = 0; b < (int)hb.size(); ++b)
      if ((freem >> hb[b]) & 1) hf.push_back(b);
    for (int j = 0; j < blocks; ++j) {
      int r = 0;
      for (size_t b = 0; b < hf.size(); ++b) r |= ((j >> hf[b]) & 1) << b;
      out.tab.push_back(r);
    }
    in.part = -1;
    if (!hf.empty()) {
      in.part = part;
      part += 1 << (id.nbits + hf.size());
      out.fins.push_back({in.part, in.off, in.step, id.nbits, 1 << hf.size(), g.fblocks});
      g.fblocks += std::max(1, (1 << id.nbits) / kWideThreads);
    }
  }
  out.steps.push_back(w);
}

}  // namespace

void build_sweep(const HostProgram &P, const std::vector<int32_t> &run, int S, int waves, bool bwd,
                 int max_walk, SweepPlan &out) {
  out = SweepPlan{};
  const int E = 64 / S, logE = ilog2(E);
  std::map<std::vector<int32_t>, int32_t> known;
  for (size_t q = 0; q < P.insts.size(); ++q) {
    SweepInst si{};
    if (!run[q]) {
      out.insts.push_back(si);
      continue;
    }
    const InstDesc &D = P.insts[q];
    // (records hold three walk positions, gather indices of eight bits)
    Levels L{P, D, P.steps.data() + D.step_off, S, waves, std::min(max_walk, 8 - logE), E, logE, D.max_w,
             out.prog, out.lanes, known, std::vector<int32_t>(D.n_steps)};
    L.B.waves = waves;
    L.lane_words(std::vector<int32_t>(E, 0));   // zeros first (no unit)
    const auto at = by_level(P, D, std::vector<char>(D.n_steps, 1));
    // arena: every message kept, or ranges reused once their reader's level
    // is over (closing entries stay)
    Reuse ar;
    for (auto &ts : at) {
      for (int t : ts) L.off[t] = bwd ? L.st[t].off_all : ar.take(1 << L.st[t].w);
      if (!bwd)
        for (int t : ts)
          for (int k = 0; k < L.st[t].n_in; ++k) {
            const int u = P.inputs[L.st[t].in_off + k].step;
            ar.give(L.off[u], 1 << L.st[u].w);
          }
    }
    si.arena = bwd ? D.arena_all : ar.top;
    closings(P, D, L.off, out.close, si);
    for (auto &ts : at) L.forward(ts);
    L.B.put(0, {SWEEP_LOGZ});
    if (bwd)
      for (size_t l = at.size(); l-- > 0;) L.reverse(at[l]);
    L.finish(si.prog);
    si.scr = L.scr_max;
    si.slots = L.slot_max;
    out.insts.push_back(si);
  }
}

void build_wide(const HostProgram &P, const std::vector<int32_t> &run, WidePlan &out) {
  out = WidePlan{};
  out.part.assign(P.insts.size(), 0);
  out.red.assign(P.insts.size(), 0);
  const int E = 64;
  std::map<std::vector<int32_t>, int32_t> known;
  for (size_t q = 0; q < P.insts.size(); ++q) {
    out.segs.emplace_back();
    SweepInst si{};
    if (!run[q]) {
      out.sum_lo.push_back((int32_t)out.sums.size());
      out.insts.push_back(si);
      continue;
    }
    const InstDesc &D = P.insts[q];
    const StepDesc *st = P.steps.data() + D.step_off;
    Levels L{P, D, st, 1, kSweepWaves, 1, E, 6, kWideStep - 1, out.prog, out.lanes, known,
             std::vector<int32_t>(D.n_steps)};
    L.B.waves = kSweepWaves;
    L.lane_words(std::vector<int32_t>(E, 0));
    for (int t = 0; t < D.n_steps; ++t) L.off[t] = st[t].off_all;
    si.arena = D.arena_all;
    closings(P, D, L.off, out.close, si);
    std::vector<char> done(D.n_steps, 0);
    auto ready = [&](int t) {
      for (int k = 0; k < st[t].n_in; ++k)
        if (!done[P.inputs[st[t].in_off + k].step]) return false;
      return !done[t];
    };
    int32_t red = 0, part_max = 0;
    out.sum_lo.push_back((int32_t)out.sums.size());
    for (int left = D.n_steps; left > 0;) {
      // (steps come in an order that respects their inputs)
      std::vector<char> use(D.n_steps, 0);
      std::vector<int> wide;
      for (int t = 0; t < D.n_steps; ++t)
        if (st[t].w < kWideStep && ready(t)) {
          use[t] = done[t] = 1;
          --left;
        }
      for (int t = 0; t < D.n_steps; ++t)
        if (st[t].w >= kWideStep && ready(t)) {
          wide.push_back(t);
          done[t] = 1;
          --left;
        }
      WideSegment sg{};
      const auto at = by_level(P, D, use);
      for (auto &ts : at) L.forward(ts);
      if (left == 0) L.B.put(0, {SWEEP_LOGZ});
      L.finish(sg.fwd);
      for (size_t l = at.size(); l-- > 0;) L.reverse(at[l]);
      L.finish(sg.bwd);
      std::fill(use.begin(), use.end(), 0);
      for (int t : wide) use[t] = 1;
      for (auto &ts : by_level(P, D, use)) {
        WideGroup g{};
        g.w0 = (int32_t)out.steps.size();
        g.f0 = (int32_t)out.fins.size();
        int32_t part = 0;
        for (int t : ts) {
          wide_step(P, D, t, part, red, out, g);
          g.blocks += 1 << (st[t].w - kWideChunk);
        }
        g.w1 = (int32_t)out.steps.size();
        g.f1 = (int32_t)out.fins.size();
        part_max = std::max(part_max, part);
        sg.groups.push_back(g);
      }
      out.segs[q].push_back(sg);
    }
    out.part[q] = part_max;
    out.red[q] = red;
    si.scr = L.scr_max;
    si.slots = L.slot_max;
    out.insts.push_back(si);
  }
  out.sum_lo.push_back((int32_t)out.sums.size());
}

}  // namespace tnvan
