"""Wide steps as launches over the chip (csrc/wide.hip) with the level kernel
between them: ln Z_R bit for bit that of the step-by-step kernel (a tile of
16 asks for it), the adjoint against the oracle, a net of graphs of several
widths around the switch (scopes of 12 spins) and past the transfer tables
(14), ragged batches, one sample at a time under a small arena."""

import numpy as np
import pytest

import synthetic as S
from adjtol import check_vjp
from oracle import ising as OI
from synthetic import instances as SI

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _graph(n, w_u, seed):
    from paper_2504_12037_amd import plan_width_set
    e = SI.random_regular_edges(n, 3, np.random.default_rng(seed))
    W, order, width, _ = plan_width_set(n, e, w_u)
    assert width == w_u
    rng = np.random.default_rng(seed + 1)
    return S.Instance(n, e.astype(np.int32), rng.choice([-1.0, 1.0], len(e)),
                      rng.normal(0.0, 0.3, n), 0.6, W.astype(np.int32),
                      order.astype(np.int32), None, 0, f"rrg{n}_wu{w_u}")


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("widths,Bs", [((12, 16, 5), (3, 4, 2)), ((13, 14, 17), (1, 0, 5)),
                                       ((15,), (9,))])
def test_wide_segments(prec, widths, Bs):
    from paper_2504_12037_amd import Net
    print(f"\n[segments] {prec} {widths} {Bs}", flush=True)
    insts = [_graph(24 + 6 * w, w, 40 + w) for w in widths]
    sp = [S.uniform_spins(b, i.n_width, 7 + k) for k, (b, i) in enumerate(zip(Bs, insts))]
    g = [np.random.default_rng(k).standard_normal(b) for k, b in enumerate(Bs)]
    dev = lambda v: torch.from_numpy(np.concatenate([x.reshape(-1) for x in v])).cuda()
    outs = []
    for tune in ({}, dict(arena_limit_mib=1), dict(general_tile_fwd=16, general_tile_bwd=16)):
        net = Net(insts, precision=prec, max_width=20)
        net.set_tuning(**tune)
        lz = net.logz(dev(sp), Bs).clone()
        both = [x.clone() for x in net.logz_and_backward(dev(sp), dev(g), Bs)]
        assert torch.equal(both[0], lz)
        outs.append(both)
    assert all(torch.equal(x, y) for x, y in zip(outs[0], outs[1]))
    assert torch.equal(outs[0][0], outs[2][0])
    _, dh, dJ, db = (x.cpu().numpy() for x in outs[0])
    ho = eo = 0
    for k, (inst, b) in enumerate(zip(insts, Bs)):
        got = (dh[ho:ho + inst.n], dJ[eo:eo + inst.n_edges], db[k])
        if b:
            check_vjp(got, OI.logz_r_vjp(inst, sp[k], g[k]), inst, g[k], prec, (widths, k))
        else:
            assert not got[0].any() and not got[1].any() and got[2] == 0.0
        ho += inst.n
        eo += inst.n_edges
