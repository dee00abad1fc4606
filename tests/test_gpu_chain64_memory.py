"""Device memory of FP64 chains (csrc/chain64.hip): ln Z_R alone takes none
for the adjoint's checkpoints, and the adjoint's stay within the arena budget,
the batch running in passes with the same bits."""

import numpy as np
import pytest

import synthetic as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B = 20000
# states of every step of three strips (two of two tiles) of 1250 groups of
# 16 samples, 8 bytes each
CKPT = 3 * 1250 * 16 * 2 * 256 * 8


def _grown(call):
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    out = call()
    torch.cuda.synchronize()
    return out, free - torch.cuda.mem_get_info()[0]


def test_checkpoints_belong_to_the_adjoint_and_its_budget():
    from paper_2504_12037_amd import Net
    inst = S.c2_lattice(1.0, 0)
    sp = torch.from_numpy(S.uniform_spins(B, inst.n_width, 3)).cuda().reshape(-1)
    g = torch.from_numpy(np.random.default_rng(4).standard_normal(B)).cuda()
    outs = []
    for limit in (0, 1):
        print(f"\n[chain64-memory] limit={limit}", flush=True)
        net = Net([inst], precision="fp64")
        net.set_tuning(arena_limit_mib=limit)
        lz, grown = _grown(lambda: net.logz(sp, B))
        assert grown < CKPT // 2, grown
        both, grown = _grown(lambda: net.logz_and_backward(sp, g, B))
        assert torch.equal(both[0], lz)
        if limit:
            # (a partial row of sums per 16 samples and the outputs)
            assert grown < CKPT // 2, grown
        outs.append(both)
    assert all(torch.equal(x, y) for x, y in zip(*outs))


def test_unary_factors_stay_within_the_budget():
    # 224 remainder spins, 8 bytes each: 36 MB for the whole batch
    from paper_2504_12037_amd import Net
    inst = S.c2_lattice(1.0, 0)
    sp = torch.from_numpy(S.uniform_spins(B, inst.n_width, 3)).cuda().reshape(-1)
    net = Net([inst], precision="fp64")
    want = net.logz(sp, B).clone()
    net = Net([inst], precision="fp64")
    net.set_tuning(arena_limit_mib=1)
    lz, grown = _grown(lambda: net.logz(sp, B))
    assert torch.equal(lz, want)
    assert grown < 18 << 20, grown
    # the limit taken back: one pass again, the same bits
    net.set_tuning()
    assert torch.equal(net.logz(sp, B), want)


def test_passes_across_the_widths():
    # strips of one, two and four tiles and an empty instance beside them, one
    # MiB: passes that end among the two-tile chains, and four-tile ones alone
    from paper_2504_12037_amd import Net
    insts = [S.lattice_column_split(S.lattice_2d(L, seed=L, h_var=0.1), cols)
             for L, cols in ((8, [4]), (13, [7]), (11, [6]), (10, [4, 8]))]
    Bs = [200, 170, 333, 0]
    dev = lambda v: torch.from_numpy(np.concatenate([x.reshape(-1) for x in v])).cuda()
    sp = dev([S.uniform_spins(b, i.n_width, 9 + k) for k, (b, i) in enumerate(zip(Bs, insts))])
    g = dev([np.random.default_rng(k).standard_normal(b) for k, b in enumerate(Bs)])
    outs = []
    for limit in (0, 1):
        net = Net(insts, precision="fp64")
        net.set_tuning(arena_limit_mib=limit)
        outs.append([x.clone() for x in net.logz_and_backward(sp, g, Bs)])
        assert torch.equal(net.logz(sp, Bs), outs[-1][0])
    assert all(torch.equal(x, y) for x, y in zip(*outs))
