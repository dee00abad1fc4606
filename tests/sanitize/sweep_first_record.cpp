// The level schedules as the kernels take them (eight waves, tiles of 1 to 8
// samples, every mode's walk limit): small random graphs through the walk of
// sweep_harness.cpp, and over many more the words that a wave reads before
// its program runs.  Of its first record it takes a transfer table offset
// (word 2), a width and a count of entries whatever the record's operation,
// so all of them must lie in the table.  Exit status 0 when they do.
#define main sweep_harness_main
#include "sweep_harness.cpp"
#undef main

static bool draw_program(std::mt19937_64 &rng, HostProgram &P) {
  const int n = 4 + (int)(rng() % 34), d = 1 + (int)(rng() % 4);
  std::vector<std::vector<char>> adj(n, std::vector<char>(n, 0));
  std::vector<int32_t> ei, ej, W, order;
  std::vector<double> J, h(n, 0.1);
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
  const int m = (int)(rng() % (n / 2));
  for (int i = 0; i < n; ++i) (i < m ? W : order).push_back(perm[i]);
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
  std::string msg;
  P = HostProgram{};
  return compile_instance(in, 10, P, msg) == TNVAN_OK && sweep_fits(P, 0);
}

int main() {
  std::mt19937_64 rng(11);
  int done = 0, bad = 0;
  for (int trial = 0; trial < 6000; ++trial) {
    HostProgram P;
    if (!draw_program(rng, P)) continue;
    ++done;
    for (int S = 1; S <= kSweepTile; S *= 2) {
      for (int mode = 0; mode < 3; ++mode)
        for (int rs = 4; rs <= (mode ? 4 : 8); rs += 4) {
          SweepPlan pl;
          build_sweep(P, {1}, S, kSweepWaves, mode == 1, sweep_walk(mode, rs), pl);
          for (int k = 0; k < kSweepWaves; ++k) {
            const int32_t *r = &pl.prog.at((int64_t)pl.insts.at(0).prog[k] * kSweepRec);
            const int entries = std::min(64 / S, 1 << ((r[0] >> 24) & 15)), w = (r[0] >> 12) & 15;
            const int64_t last = (int64_t)r[2] + entries - 1 + (1 << w);
            if ((r[2] < 0 || last >= (int64_t)P.T.size()) && ++bad <= 10)
              std::fprintf(stderr, "program %d, tile %d, mode %d, wave %d: operation %d reads entry %lld of %zu\n",
                           trial, S, mode, k, r[0] & 15, (long long)last, P.T.size());
          }
        }
      if (done % 40 == 0)
        for (int walk : {1, 2, 3}) check(P, S, kSweepWaves, walk);
    }
  }
  if (bad || g_fail || done < 3000)
    return std::fprintf(stderr, "%d reads past the table, %d failed, %d programs\n", bad, g_fail, done), 1;
  std::printf("first records ok (%d programs)\n", done);
  return 0;
}
