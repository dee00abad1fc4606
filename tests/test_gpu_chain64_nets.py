"""FP64 nets of several kinds of instances: which run as chains
(csrc/chain64.hip), on the level kernels and step by step.  A small lattice
beside random graphs or larger lattices takes part in the chain launches
(and leaves the graphs the level kernels); beside an instance that stays step
by step the chains run from 2048 of their samples on, with the same values on
both sides of that line; small lattices alone stay on the general kernel.  ln Z_R and
the adjoint against the oracle, the moments' ln Z_R beside them."""

import numpy as np
import pytest

import synthetic as S
from adjtol import check_vjp
from oracle import ising as OI

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _lat(L, cols, seed):
    return S.lattice_column_split(S.lattice_2d(L, seed=seed, h_var=0.1), cols)


def _sk():
    return S.sherrington_kirkpatrick(20, seed=3, n_width=4, group_size=8)


# instances, samples, kinds reported, whether the level kernels run
CASES = {
    "graph_and_small": ([S.c4_small_copies(limit=3)[1], _lat(4, [2], 1)], [40, 33], 1, True),
    "small_beside_large": ([_lat(4, [2], 1), _lat(6, [3], 2), _lat(8, [4], 3)], [17, 0, 50], 0, False),
    "small_alone": ([_lat(4, [2], 1), _lat(6, [3], 2)], [17, 30], 1, False),
    "dense_beside": ([_sk(), _lat(8, [4], 3)], [30, 20], 1, False),
    "dense_beside_large_batch": ([_sk(), _lat(8, [4], 3)], [20, 2048], 1, False),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_fp64_nets(case):
    from paper_2504_12037_amd import Net
    insts, Bs, kinds, level = CASES[case]
    print(f"\n[chain64-nets] {case}", flush=True)
    sp = [S.uniform_spins(b, i.n_width, 70 + k) for k, (b, i) in enumerate(zip(Bs, insts))]
    g = [np.random.default_rng(k).standard_normal(b) for k, b in enumerate(Bs)]
    dev = lambda v: torch.from_numpy(np.concatenate([x.reshape(-1) for x in v])).cuda()
    net = Net(insts, precision="fp64")
    before = net.get_tuning()
    assert before["kinds"] == kinds
    assert (before["general_tile_fwd"] == 0) == (level or kinds == 0)
    lz, dh, dJ, db = net.logz_and_backward(dev(sp), dev(g), Bs)
    assert torch.equal(net.logz(dev(sp), Bs), lz)
    mom = net.remainder_moments(dev(sp), Bs)[0]
    lz, dh, dJ, db, mom = (x.cpu().numpy() for x in (lz, dh, dJ, db, mom))
    bo = ho = eo = 0
    for k, (inst, b) in enumerate(zip(insts, Bs)):
        if b:
            n = min(b, 200)
            want = OI.logz_r_elimination(inst, sp[k][:n])
            for z in (lz, mom):
                assert np.abs(z[bo:bo + n] - want).max() / inst.n <= 1e-10
            check_vjp((dh[ho:ho + inst.n], dJ[eo:eo + inst.n_edges], db[k]),
                      OI.logz_r_vjp(inst, sp[k], g[k]), inst, g[k], "fp64", (case, k))
        bo += b
        ho += inst.n
        eo += inst.n_edges


def test_the_line_changes_no_value():
    # batches in turn on either side of it, on one net
    from paper_2504_12037_amd import Net
    insts = [_sk(), _lat(8, [4], 3)]
    net = Net(insts, precision="fp64")
    big = [100, 2100]
    sp = [S.uniform_spins(b, i.n_width, 7) for b, i in zip(big, insts)]
    dev = lambda v: torch.from_numpy(np.concatenate([x.reshape(-1) for x in v])).cuda()
    for _ in range(2):
        a = net.logz(dev(sp), big).cpu().numpy()
        b = net.logz(dev([sp[0], sp[1][:2000]]), [100, 2000]).cpu().numpy()
        for lo, hi, inst in ((0, 100, insts[0]), (100, 2100, insts[1])):
            assert np.abs(a[lo:hi] - b[lo:hi]).max() / inst.n <= 1e-12
