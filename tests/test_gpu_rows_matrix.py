"""REINFORCE rows on the matrix cores (csrc/made.hip) at the edges of their
tiles: |W| and H around multiples of 16 and 4, |W| of 0 and 1, one to four
layers, chunks of 32, 16 and (FP64) 4 samples with partial last blocks,
masked entries that are not zero; the gradient of Eq. (10) against the
oracle.

Tolerance: an entry is a sum over the batch of w_b times a product of
factors of size at most about one, each a sum of fewer than 1000 terms held
to a few ulp; with the weights' rounding, 1e-4 of the largest entry in FP32
as for the other gradient tests, 1e-6 (the gradient is stored in FP32) in
FP64."""

import numpy as np
import pytest

import synthetic as S
from oracle import ising as OI
from oracle import made as OM
from oracle import objective as OO

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = {                       # (|W|, H, depth, samples)
    "one_layer": [(1, 6, 1, 10), (2, 5, 1, 33), (15, 16, 1, 47), (66, 33, 1, 100), (0, 4, 1, 5)],
    "chunks32": [(17, 15, 1, 16500), (70, 130, 1, 35)],
    "deep": [(16, 17, 2, 50), (33, 64, 4, 31), (3, 40, 3, 5), (9, 8, 1, 40)],
    "deep_wide": [(130, 96, 2, 40), (200, 250, 3, 17)],
}


def _inst(n, H, depth):
    N = n + 4                   # a ring, all but four spins in the width set
    e = np.sort(np.stack([np.arange(N), (np.arange(N) + 1) % N], 1), 1).astype(np.int32)
    i = S.Instance(N, e, np.random.default_rng(n).standard_normal(N), np.zeros(N), 0.7,
                   np.arange(n, dtype=np.int32), np.arange(n, N, dtype=np.int32), None, H, f"w{n}")
    i.depth = depth
    return i


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_gradient_rows(case, prec):
    from paper_2504_12037_amd import Net
    print(f"\n[rows] {case} {prec}", flush=True)
    insts, Bs = [_inst(*c[:3]) for c in CASES[case]], [c[3] for c in CASES[case]]
    net = Net(insts, precision=prec, seed=3)
    theta = []
    for q, (n, H, depth, _) in enumerate(CASES[case]):
        th = 0.2 * np.random.default_rng(q).standard_normal(OM.param_count(n, H, depth))
        theta.append(th.astype(np.float32))
        net.set_params(q, torch.from_numpy(theta[q]))
    spins = torch.empty(sum(b * c[0] for b, c in zip(Bs, CASES[case])), dtype=torch.int8, device="cuda")
    net.free_energy_step(Bs, 1e-3, spins_out=spins)
    sp, so = spins.cpu().numpy(), 0
    for q, (n, H, depth, b) in enumerate(CASES[case]):
        s = sp[so:so + b * n].reshape(b, n)
        so += b * n
        if n == 0:
            continue
        th = theta[q].astype(np.float64)
        f, _ = OO.free_energy_terms(insts[q], s, OM.logq(th, s, n, H, depth=depth),
                                    OI.logz_r_elimination(insts[q], s))
        g = OM.logq_backward(th, s, OO.reinforce_weights(f), n, H, depth=depth)
        got = net.get_state(q, 1).cpu().numpy().astype(np.float64)
        tol = 1e-6 if prec == "fp64" else 1e-4
        assert np.abs(got - g).max() <= 1e-7 + tol * np.abs(g).max(), q
