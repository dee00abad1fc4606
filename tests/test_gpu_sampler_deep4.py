"""The four-lane sampler of deeper networks (csrc/made.hip) at its edges:
|W| around a stage's 16 positions and its lane tables (32, 64, 128), runs of
|W| - 1 units whose lanes coincide (|W| - 1 divisible by 4, by 2, odd), two to
four layers, a one-layer and an empty instance beside them, masked entries
that are not zero, given uniforms and the Philox stream, against the oracle.

Tolerance of log q as for the other samplers: 2e-4 (FP32), 1e-10 (FP64) per 8
positions."""

import numpy as np
import pytest

import synthetic as S
from oracle import made as OM
from oracle import philox as OP

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TIE = 1e-6

CASES = {                       # (|W|, H, depth, samples)
    "small": [(2, 9, 2, 40), (3, 64, 2, 33), (5, 64, 2, 65), (7, 3, 1, 20), (0, 4, 2, 9)],
    "stage": [(16, 64, 3, 31), (17, 33, 2, 100), (32, 64, 3, 64)],
    "deep": [(33, 40, 4, 50), (36, 64, 3, 0), (64, 16, 2, 1)],
    "wide": [(65, 64, 2, 33), (128, 17, 4, 40)],
}


def _inst(n, H, depth):
    N = n + 4                   # a ring, all but four spins in the width set
    e = np.sort(np.stack([np.arange(N), (np.arange(N) + 1) % N], 1), 1).astype(np.int32)
    i = S.Instance(N, e, np.random.default_rng(n).standard_normal(N), np.zeros(N), 1.0,
                   np.arange(n, dtype=np.int32), np.arange(n, N, dtype=np.int32), None, H, f"w{n}")
    i.depth = depth
    return i


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_four_lane_deep_sampler(case, prec):
    from paper_2504_12037_amd import Net
    print(f"\n[deep4] {case} {prec}", flush=True)
    insts, Bs = [_inst(*c[:3]) for c in CASES[case]], [c[3] for c in CASES[case]]
    net = Net(insts, precision=prec, seed=8)
    theta = []
    for q, (n, H, depth, _) in enumerate(CASES[case]):
        th = 0.4 * np.random.default_rng(q).standard_normal(OM.param_count(n, H, depth))
        theta.append(th.astype(np.float32))
        net.set_params(q, torch.from_numpy(theta[q]))
    for given in (True, False):
        us = [S.uniforms(b, n, 5 + q) if given else OP.sampler_uniforms(8, 0, q, b, n)
              for q, (n, _, _, b) in enumerate(CASES[case])]
        flat = np.concatenate([u.reshape(-1) for u in us])
        sp, lq = net.sample(Bs, torch.from_numpy(flat).cuda() if given else None)
        sp, lq = sp.cpu().numpy(), lq.cpu().numpy()
        so = lo = 0
        for q, (n, H, depth, b) in enumerate(CASES[case]):
            s = sp[so:so + b * n].reshape(b, n)
            if b and n:
                th, u = theta[q].astype(np.float64), us[q].reshape(b, n)
                _, _, p = OM.sample(th, u, n, H, depth=depth)
                force = np.where(np.abs(p - u) < TIE, s, 0).astype(np.int8)
                want, _, _ = OM.sample(th, u, n, H, force=force, depth=depth)
                assert np.array_equal(want, s), q
                err = np.abs(lq[lo:lo + b] - OM.logq(th, s, n, H, depth=depth)).max()
                assert err <= (1e-10 if prec == "fp64" else 2e-4) * max(1, n / 8)
            so += b * n
            lo += b
