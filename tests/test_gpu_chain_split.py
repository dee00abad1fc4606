"""Chains of more than 64 states on eight waves per 16 samples
(csrc/chain.hip): steps of 7 and 8 spins (some waves without a tile), long
chains with checkpoint segments, a narrow chain beside a wide one, ragged
batches around 16 samples, ln Z_R and the adjoint against the oracle."""

import numpy as np
import pytest

import synthetic as S
from adjtol import check_vjp
from oracle import ising as OI

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = {"fp32": 1e-5, "bf16": 1e-3}

CASES = {
    "sk8": ([S.sherrington_kirkpatrick(40, seed=2, beta=1.0, n_width=24, group_size=8, hidden=0),
             S.sherrington_kirkpatrick(30, seed=5, beta=0.7, n_width=16, group_size=7, hidden=0)],
            [17, 40]),
    "strips7": ([S.lattice_column_split(S.lattice_2d(12, seed=3, beta=0.9, h_var=0.1), [8])], [33]),
    "strips8": ([S.lattice_column_split(S.lattice_2d(10, seed=4, beta=1.0, h_var=0.1), [9]),
                 S.lattice_column_split(S.lattice_2d(6, seed=5, beta=1.0, h_var=0.1), [3])], [1, 16]),
}


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_wide_chains_against_the_oracle(case, prec):
    from paper_2504_12037_amd import Net
    insts, Bs = CASES[case]
    print(f"\n[chain-split] {case} {prec}", flush=True)
    sp = [S.uniform_spins(b, i.n_width, 60 + k) for k, (b, i) in enumerate(zip(Bs, insts))]
    g = [np.random.default_rng(k).standard_normal(b) for k, b in enumerate(Bs)]
    dev = lambda v: torch.from_numpy(np.concatenate([x.reshape(-1) for x in v])).cuda()
    net = Net(insts, precision=prec)
    lz = net.logz(dev(sp), Bs).cpu().numpy()
    back = [x.clone() for x in net.backward(dev(sp), dev(g), Bs)]
    assert all(torch.equal(x, y) for x, y in zip(back, net.backward(dev(sp), dev(g), Bs)))
    dh, dJ, db = (x.cpu().numpy() for x in back)
    bo = ho = eo = 0
    for k, (inst, b) in enumerate(zip(insts, Bs)):
        want = OI.logz_r_elimination(inst, sp[k])
        assert np.abs(lz[bo:bo + b] - want).max() / inst.n <= TOL[prec]
        check_vjp((dh[ho:ho + inst.n], dJ[eo:eo + inst.n_edges], db[k]),
                  OI.logz_r_vjp(inst, sp[k], g[k]), inst, g[k], prec, (case, k))
        bo += b
        ho += inst.n
        eo += inst.n_edges
