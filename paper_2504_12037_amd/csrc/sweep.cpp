// Host schedule of the level kernels (see sweep.h).  Pure C++.
#include "sweep.h"

#include <algorithm>
#include <map>

#include "compile.h"

namespace tnvan {

bool sweep_fits(const HostProgram &P, int q) {
  const InstDesc &D = P.insts[q];
  // (records hold steps and positions in 15 bits)
  if (D.n_steps <= 0 || D.n_steps > 32767 || D.nr > 32767) return false;
  for (int t = 0; t < D.n_steps; ++t) {
    const StepDesc &sd = P.steps[D.step_off + t];
    if (sd.g != 1 || sd.w > kTabW || sd.t_off < 0 || sd.t_off > INT32_MAX - (2 << kTabW) || sd.n_in > kSweepIn ||
        sd.n_edge > kSweepEdges)
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

}  // namespace

void build_sweep(const HostProgram &P, const std::vector<int32_t> &run, int S, int waves, bool bwd,
                 int max_walk, SweepPlan &out) {
  out = SweepPlan{};
  const int E = 64 / S, logE = ilog2(E);
  // lane words, E in a row, each kind once; zeros first (no unit)
  std::map<std::vector<int32_t>, int32_t> known;
  auto lane_words = [&](const std::vector<int32_t> &w) {
    auto it = known.find(w);
    if (it != known.end()) return it->second;
    const int32_t at = (int32_t)out.lanes.size();
    out.lanes.insert(out.lanes.end(), w.begin(), w.end());
    known[w] = at;
    return at;
  };
  lane_words(std::vector<int32_t>(E, 0));
  for (size_t q = 0; q < P.insts.size(); ++q) {
    SweepInst si{};
    if (!run[q]) {
      out.insts.push_back(si);
      continue;
    }
    const InstDesc &D = P.insts[q];
    const StepDesc *st = P.steps.data() + D.step_off;
    std::vector<int> level(D.n_steps, 0);
    int nl = 0;
    for (int t = 0; t < D.n_steps; ++t) {
      for (int k = 0; k < st[t].n_in; ++k)
        level[t] = std::max(level[t], level[P.inputs[st[t].in_off + k].step] + 1);
      nl = std::max(nl, level[t] + 1);
    }
    std::vector<std::vector<int>> at(nl);
    for (int t = 0; t < D.n_steps; ++t) at[level[t]].push_back(t);
    // arena: every message kept, or ranges reused once their reader's level
    // is over (closing entries stay)
    std::vector<int32_t> off(D.n_steps);
    Reuse ar;
    for (int l = 0; l < nl; ++l) {
      for (int t : at[l]) off[t] = bwd ? st[t].off_all : ar.take(1 << st[t].w);
      if (!bwd)
        for (int t : at[l])
          for (int k = 0; k < st[t].n_in; ++k) {
            const int u = P.inputs[st[t].in_off + k].step;
            ar.give(off[u], 1 << st[u].w);
          }
    }
    si.arena = bwd ? D.arena_all : ar.top;
    si.close_off = (int32_t)out.close.size();
    for (int t = 0; t < D.n_steps; ++t)
      if (st[t].w == 0) {
        out.close.push_back(off[t]);
        out.close.push_back(t);
      }
    si.n_close = ((int32_t)out.close.size() - si.close_off) / 2;

    // passes per unit of a level: as many as leave every wave a unit
    std::vector<int> walk(nl);
    for (int l = 0; l < nl; ++l) {
      auto units_at = [&](int wk) {
        int64_t n = 0;
        for (int t : at[l]) n += std::max(1, (1 << st[t].w) >> (logE + wk));
        return n;
      };
      walk[l] = max_walk;
      while (walk[l] > 0 && units_at(walk[l]) < waves) --walk[l];
    }
    Builder B;
    B.waves = waves;
    // units of a step; scr and slot advance over the level
    auto step_units = [&](int t, int wk, SweepOp op, int32_t scr, int32_t &slot) {
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
    };
    for (int l = 0; l < nl; ++l) {
      int32_t slot = 0;
      for (int t : at[l]) step_units(t, walk[l], SWEEP_FWD, 0, slot);
      B.flush();
    }
    B.put(0, {SWEEP_LOGZ});
    for (int l = nl - 1; l >= 0 && bwd; --l) {
      int32_t scr = 0, slot = 0;
      std::vector<int32_t> scr_of, slot_of;
      for (int t : at[l]) {
        scr_of.push_back(scr);
        slot_of.push_back(slot);
        step_units(t, walk[l], SWEEP_JOINT, scr, slot);
        scr += 2 << st[t].w;
      }
      si.scr = std::max(si.scr, scr);
      si.slots = std::max(si.slots, slot);
      B.flush();
      // marginals: lanes that share a sum, and passes per unit
      struct Marg { int step, k, lc; };
      std::vector<Marg> ms;
      int64_t passes = 0;
      std::vector<int> which;
      for (size_t i = 0; i < at[l].size(); ++i) {
        const StepDesc &sd = st[at[l][i]];
        const int per = std::min(1 << sd.w, E << walk[l]);
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
          ms.push_back({at[l][i], k, lc});
          which.push_back((int)i);
          passes += std::max(1, (1 << (id.nbits + lc)) / E);
        }
      }
      int mwalk = kSweepWalk;
      while (mwalk > 0 && (passes >> mwalk) < waves) --mwalk;
      for (size_t mi = 0; mi < ms.size(); ++mi) {
        const StepDesc &sd = st[ms[mi].step];
        const InputDesc &id = P.inputs[sd.in_off + ms[mi].k];
        const int lc = ms[mi].lc;
        // output bits of an item's bits: the lanes that share a sum (free
        // output bits, lowest first), then the entry's bits
        const bool dense = sd.kind == STEP_DENSE;
        int rest = ((1 << sd.w) - 1) & ~(dense ? 0 : id.omask);
        std::vector<int> pos;
        for (int b = 0; b < lc; ++b) {
          pos.push_back(ilog2(rest & -rest));
          rest &= rest - 1;
        }
        for (int b = 0; b < id.nbits; ++b)
          pos.push_back(dense || id.src[b] < 0 ? sd.w : id.src[b]);
        const int items = 1 << (id.nbits + lc), pm = std::min(items, E << mwalk);
        std::vector<int32_t> lw(E, 0);
        for (int b = 0; b < logE && b < (int)pos.size(); ++b)
          for (int lo = 0; lo < E; ++lo)
            if ((lo >> b) & 1) lw[lo] |= 1 << pos[b];
        int32_t code = 0xfff;
        for (int b = 0; b < kSweepWalk && logE + b < (int)pos.size(); ++b)
          code = (code & ~(15 << (4 * b))) | (pos[logE + b] << (4 * b));
        const int32_t at_lanes = lane_words(lw);
        for (int i0 = 0; i0 < items; i0 += pm) {
          int32_t base = scr_of[which[mi]];
          for (size_t b = 0; b < pos.size(); ++b)
            if ((i0 >> b) & 1) base += 1 << pos[b];
          std::vector<int32_t> r = {SWEEP_MARG | (lc << 12) | (ilog2(pm) << 16), base, code,
                                    off[id.step] + (i0 >> lc), id.step, rest};
          r.resize(kSweepRec, 0);
          r[19] = at_lanes;
          B.add(8 + std::max(1, pm / E) * (4 + (1 << __builtin_popcount((unsigned)rest))), std::move(r));
        }
      }
      B.flush();
    }
    for (int k = 0; k < waves; ++k) {
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
      si.prog[k] = (int32_t)(out.prog.size() / kSweepRec);
      out.prog.insert(out.prog.end(), B.rec[k].begin(), B.rec[k].end());
    }
    out.insts.push_back(si);
  }
}

}  // namespace tnvan
