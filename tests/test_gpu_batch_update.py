"""Batch sums on the matrix cores and the Adam step in their second launch
(csrc/made.hip): batches around a wave's 16 rows and a slice, matrices past
one 32 x 32 tile, a width set of one spin with a second layer (whose
parameters no sum covers), an empty instance; the gradient against the
oracle's, the step against Adam of the stored gradient, from moments that are
not zero.

Tolerances as for the other gradient and optimiser tests: 1e-4 (FP32) and
1e-6 (FP64, stored in FP32) of the largest gradient entry; 1e-6 on the
parameters after the step."""

import numpy as np
import pytest

import synthetic as S
from oracle import ising as OI
from oracle import made as OM
from oracle import objective as OO

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = {                       # (|W|, H, depth, samples)
    "edges": [(33, 47, 1, 15), (66, 5, 1, 17), (70, 40, 1, 129), (12, 33, 1, 0)],
    "deep": [(1, 6, 2, 30), (20, 36, 2, 4200), (9, 64, 3, 64)],
    "no_hidden": [(80, 0, 1, 63), (70, 0, 1, 700)],
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
def test_sums_and_update(case, prec):
    from paper_2504_12037_amd import Net
    print(f"\n[update] {case} {prec}", flush=True)
    insts, Bs = [_inst(*c[:3]) for c in CASES[case]], [c[3] for c in CASES[case]]
    net = Net(insts, precision=prec, seed=4)
    theta, m0, v0 = [], [], []
    for q, (n, H, depth, _) in enumerate(CASES[case]):
        r = np.random.default_rng(q)
        k = OM.param_count(n, H, depth)
        theta.append((0.2 * r.standard_normal(k)).astype(np.float32))
        m0.append((1e-3 * r.standard_normal(k)).astype(np.float32))
        v0.append((1e-3 * r.random(k)).astype(np.float32))
        net.set_params(q, torch.from_numpy(theta[q]))
        net.set_state(q, 2, torch.from_numpy(m0[q]))
        net.set_state(q, 3, torch.from_numpy(v0[q]))
    spins = torch.empty(sum(b * c[0] for b, c in zip(Bs, CASES[case])), dtype=torch.int8, device="cuda")
    net.free_energy_step(Bs, 1e-2, spins_out=spins)
    sp, so = spins.cpu().numpy(), 0
    for q, (n, H, depth, b) in enumerate(CASES[case]):
        s = sp[so:so + b * n].reshape(b, n)
        so += b * n
        got = net.get_state(q, 1).cpu().numpy().astype(np.float64)
        th = theta[q].astype(np.float64)
        if b == 0:
            assert np.array_equal(net.get_params(q).cpu().numpy(), theta[q])
            assert np.array_equal(net.get_state(q, 2).cpu().numpy(), m0[q])
            continue
        f, _ = OO.free_energy_terms(insts[q], s, OM.logq(th, s, n, H, depth=depth),
                                    OI.logz_r_elimination(insts[q], s))
        g = OM.logq_backward(th, s, OO.reinforce_weights(f), n, H, depth=depth)
        assert np.abs(got - g).max() <= 1e-7 + (1e-6 if prec == "fp64" else 1e-4) * np.abs(g).max(), q
        want, m, v = OO.adam_step(th, got, m0[q].astype(np.float64), v0[q].astype(np.float64), 1, 1e-2)
        np.testing.assert_allclose(net.get_params(q).cpu().numpy(), want, atol=1e-6, rtol=1e-6)
        np.testing.assert_allclose(net.get_state(q, 2).cpu().numpy(), m, atol=1e-9, rtol=1e-6)
        np.testing.assert_allclose(net.get_state(q, 3).cpu().numpy(), v, atol=1e-12, rtol=1e-6)
