"""E_1 (Eq. 4) beside the unary factors of register-resident chains and in
its own launch (csrc/e1.h): |W| up to 32, up to 128 and beyond the bit mask,
none, more couplings than a block stages at once, fields, ragged and empty
batches, against the oracle.

Tolerance: a sum in FP64 of T terms +-J or +-h in four parts, so T 2^-53
times the sum of their sizes."""

import numpy as np
import pytest

import synthetic as S
from oracle import ising as OI

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _lat(L, cols, seed):
    return S.lattice_column_split(S.lattice_2d(L, seed=seed, beta=0.8, h_var=0.2), cols)


def _sk(n, nw, seed):
    return S.sherrington_kirkpatrick(n, seed=seed, n_width=nw, group_size=8, hidden=0)


CASES = {
    "chains": ([_lat(8, [4], 1), _lat(20, [4, 8, 12, 16, 20], 2),
                _lat(24, [3, 6, 9, 12, 15, 18, 21, 24], 3), _lat(4, [], 4)], [300, 1, 257, 0]),
    "sk": ([_sk(40, 24, 5), _sk(56, 40, 6)], [70, 256]),
    "general": ([S.c4_small_copies(limit=3)[0], _lat(8, [3], 7),
                 _lat(22, [2, 5, 8, 11, 14, 17, 20], 8)], [5, 513, 40]),
}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_e1(case, prec):
    from paper_2504_12037_amd import Net
    insts, Bs = CASES[case]
    print(f"\n[e1] {case} {prec}", flush=True)
    sp = [S.uniform_spins(b, i.n_width, 30 + k) for k, (b, i) in enumerate(zip(Bs, insts))]
    flat = torch.from_numpy(np.concatenate([s.reshape(-1) for s in sp])).cuda()
    net = Net(insts, precision=prec)
    lz, e1 = net.logz(flat, Bs, e1=True)
    assert torch.equal(lz, net.logz(flat, Bs))
    e1, off = e1.cpu().numpy(), 0
    for inst, b, s in zip(insts, Bs, sp):
        if b:
            size = np.abs(inst.J).sum() + np.abs(inst.h).sum()
            err = np.abs(e1[off:off + b] - OI.e1_energy(inst, s)).max()
            assert err <= (inst.n_edges + inst.n) * 2.0 ** -53 * size
        off += b
