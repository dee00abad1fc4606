"""Launch shapes of nets whose general instances run the level kernels
(csrc/sweep.hip), wide steps in segments (csrc/wide.hip) or FP64 chains
(csrc/chain64.hip): what get_tuning reports is what runs, a reported or tuned
shape asked for again runs the same, and a cache entry of other kernels is not
taken."""

import json

import numpy as np
import pytest

import synthetic as S
from synthetic import instances as SI

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILES = ("general_tile_fwd", "general_tile_bwd")


def _graph(n, w_u, seed=3):
    from paper_2504_12037_amd import plan_width_set
    e = SI.random_regular_edges(n, 3, np.random.default_rng(seed))
    W, order, _, _ = plan_width_set(n, e, w_u)
    rng = np.random.default_rng(seed + 1)
    return S.Instance(n, e.astype(np.int32), rng.choice([-1.0, 1.0], len(e)),
                      rng.normal(0.0, 0.3, n), 0.6, W.astype(np.int32),
                      order.astype(np.int32), None, 0, f"rrg{n}_wu{w_u}")


def _data(inst, B):
    sp = torch.from_numpy(S.uniform_spins(B, inst.n_width, 5)).cuda().reshape(-1)
    return sp, torch.full((B,), 1.0 / B, dtype=torch.float64, device="cuda"), B


def _ask(net, t):
    net.set_tuning(**{k: t[k] for k in TILES + ("chain_groups", "checkpoint_every", "launch_mode",
                                                "arena_limit_mib")})


CASES = {"level": (lambda: S.c4_rrg(), 600, "fp32", 10),
         "level64": (lambda: S.c4_rrg(), 600, "fp64", 10),
         "segments": (lambda: _graph(100, 16), 5, "fp32", 20)}


@pytest.mark.parametrize("case", sorted(CASES))
def test_reported_shapes_are_those_that_run(case):
    from paper_2504_12037_amd import Net
    make, B, prec, mw = CASES[case]
    inst = make()
    data = _data(inst, B)
    print(f"\n[tuning-level] {case}", flush=True)

    def ran(net):
        out = [x.clone() for x in net.logz_and_backward(*data)] + [net.logz(*data[::2]).clone()]
        return net.get_tuning(), out

    net = Net([inst], precision=prec, max_width=max(14, mw))
    before = net.get_tuning()
    after, want = ran(net)
    # (the level kernels choose by the batch; before one there is no tile)
    assert all(before[k] == (1 if case == "segments" else 0) for k in TILES), before
    assert all(1 <= after[k] <= 8 for k in TILES), after
    assert after["kinds"] == 1
    for shapes in (before, after):
        net = Net([inst], precision=prec, max_width=max(14, mw))
        _ask(net, shapes)
        again, out = ran(net)
        assert {k: again[k] for k in TILES} == {k: after[k] for k in TILES}
        assert all(torch.equal(x, y) for x, y in zip(out, want))
    # other batch, other tile; a tile above eight is another kernel's
    net.set_tuning(general_tile_fwd=16, general_tile_bwd=16)
    assert all(net.get_tuning()[k] == 16 for k in TILES)
    assert all(ran(net)[0][k] == 16 for k in TILES)
    net.set_tuning()
    assert all(net.get_tuning()[k] == before[k] for k in TILES)


def test_step_by_step_nets_report_their_tile_at_once():
    # (grouped dense steps below the FP64 chains' size)
    from paper_2504_12037_amd import Net
    net = Net([S.c1_small_lattice(0)], precision="fp64")
    t = net.get_tuning()
    assert t["kinds"] == 1 and all(t[k] > 0 for k in TILES)


def test_fp64_chains_have_no_general_tile(tmp_path):
    from paper_2504_12037_amd import Net
    inst = S.c2_lattice(1.0, 0)
    net = Net([inst], precision="fp64")
    sp, g, B = _data(inst, 100)
    t = net.autotune(sp, g, B, cache_path=tmp_path / "tune.json")
    assert t["kinds"] == 0 and all(t[k] == 0 for k in TILES)


def test_autotuned_shapes_apply_elsewhere_and_old_entries_do_not(tmp_path):
    from paper_2504_12037_amd import Net
    inst = S.c4_rrg()
    sp, g, B = _data(inst, 2048)
    cache = tmp_path / "tune.json"
    net = Net([inst], precision="fp32")
    chosen = net.autotune(sp, g, B, cache_path=cache)
    (key, val), = json.loads(cache.read_text()).items()
    for k in TILES:
        assert chosen[k] == val[k]          # a kept default stays the default
    # an entry keyed as for the step-by-step kernel alone
    head = key.split("|")[:2]
    old = "|".join(head + ["k1", f"w{net.info()[1]}", "n1", "B11"])
    assert old != key
    cache.write_text(json.dumps({old: dict(val, general_tile_fwd=16, general_tile_bwd=16)}))
    net = Net([inst], precision="fp32")
    net.autotune(sp, g, B, cache_path=cache)
    assert set(json.loads(cache.read_text())) == {old, key}
