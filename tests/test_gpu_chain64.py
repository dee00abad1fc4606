"""Chains of FP64 nets on the FP64 matrix cores (csrc/chain64.hip): strips of
one, two and four tiles, ragged batches around a wave's 16 samples, an empty
instance, fields, width sets beyond the 128-bit spin mask, and mixed nets,
logZ and the adjoint against the oracle; below the size where they run the
general kernel answers."""

import numpy as np
import pytest

import synthetic as S
from adjtol import check_vjp
from oracle import ising as OI

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _lat(L, cols, seed, h_var=0.1, beta=1.0):
    return S.lattice_column_split(S.lattice_2d(L, seed=seed, beta=beta, h_var=h_var), cols)


CASES = {
    "one_tile": ([_lat(8, [4], 1)], [17]),
    "two_tiles": ([_lat(11, [6], 2, h_var=0.0, beta=2.0)], [33]),
    "four_tiles": ([_lat(13, [7], 3)], [1]),
    "uneven_strips": ([_lat(9, [2, 8], 4)], [16]),
    "mixed": ([_lat(8, [3], 5), _lat(13, [7], 6), S.c4_small_copies(limit=3)[0], _lat(4, [2], 7),
               _lat(10, [4, 8], 8)], [40, 31, 20, 25, 0]),
    "wide_set": ([_lat(20, [3, 6, 9, 12, 15, 18, 20], 9)], [19]),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_fp64_chains_against_the_oracle(case):
    from paper_2504_12037_amd import Net
    insts, Bs = CASES[case]
    print(f"\n[chain64] {case}", flush=True)
    sp = [S.uniform_spins(b, i.n_width, 70 + k) for k, (b, i) in enumerate(zip(Bs, insts))]
    g = [np.random.default_rng(k).standard_normal(b) for k, b in enumerate(Bs)]
    dev = lambda v: torch.from_numpy(np.concatenate([x.reshape(-1) for x in v])).cuda()
    net = Net(insts, precision="fp64")
    lz, dh, dJ, db = net.logz_and_backward(dev(sp), dev(g), Bs)
    assert torch.equal(net.logz(dev(sp), Bs), lz)
    again = net.backward(dev(sp), dev(g), Bs)
    assert all(torch.equal(x, y) for x, y in zip(again, (dh, dJ, db)))
    lz, dh, dJ, db = (x.cpu().numpy() for x in (lz, dh, dJ, db))
    bo = ho = eo = 0
    for k, (inst, b) in enumerate(zip(insts, Bs)):
        if b:
            want = OI.logz_r_elimination(inst, sp[k])
            assert np.abs(lz[bo:bo + b] - want).max() / inst.n <= 1e-10
        got = (dh[ho:ho + inst.n], dJ[eo:eo + inst.n_edges], db[k])
        if b:
            check_vjp(got, OI.logz_r_vjp(inst, sp[k], g[k]), inst, g[k], "fp64", (case, k))
        else:
            assert not got[0].any() and not got[1].any() and got[2] == 0.0
        bo += b
        ho += inst.n
        eo += inst.n_edges
