"""The general sampler (csrc/made.hip) at its edges: |W| of 0 to above a
stage's positions, either count of samples per lane, 8 to 64 lanes per
sample, more units than degrees and fewer, masked entries that are not zero,
given uniforms and the Philox stream, mixed and empty instances, against the
oracle.

Tolerance of log q: FP32 sums of |W| terms of a few units' ulp each, 2e-4 per
8 positions as for the other samplers; FP64 1e-10."""

import numpy as np
import pytest

import synthetic as S
from oracle import made as OM
from oracle import philox as OP

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TIE = 1e-6


def _inst(n, H):
    # a ring of n + 4 spins, all but four in the width set
    N = n + 4
    e = np.sort(np.stack([np.arange(N), (np.arange(N) + 1) % N], 1), 1).astype(np.int32)
    J = np.random.default_rng(n).standard_normal(N)
    return S.Instance(N, e, J, np.zeros(N), 1.0, np.arange(n, dtype=np.int32),
                      np.arange(n, N, dtype=np.int32), None, H, f"w{n}")


CASES = {                       # (|W|, H, samples)
    "few": [(1, 5, 40), (2, 9, 33), (3, 64, 70), (0, 4, 20), (66, 3, 1)],
    "stage": [(65, 128, 100), (128, 17, 63), (64, 1, 0), (9, 127, 31)],
    "two_per_lane": [(72, 40, 33000), (16, 8, 257)],
    "jj32": [(130, 30, 100), (256, 128, 33)],
    "lanes16": [(257, 24, 50), (20, 200, 18)],
    "lanes64": [(1030, 8, 9), (12, 700, 20)],
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_general_sampler(case, prec):
    from paper_2504_12037_amd import Net
    print(f"\n[general-sampler] {case} {prec}", flush=True)
    insts, Bs = [_inst(n, H) for n, H, _ in CASES[case]], [b for _, _, b in CASES[case]]
    net = Net(insts, precision=prec, seed=21)
    theta = []
    for q, (n, H, _) in enumerate(CASES[case]):
        r = np.random.default_rng(q)
        th = S.made_init(n, H, q)
        theta.append((th + 0.3 * r.standard_normal(th.shape)).astype(np.float32))
        net.set_params(q, torch.from_numpy(theta[q]))
    for given in (True, False):
        us = [S.uniforms(b, n, 5 + q) if given else OP.sampler_uniforms(21, 0, q, b, n)
              for q, (n, _, b) in enumerate(CASES[case])]
        flat = np.concatenate([u.reshape(-1) for u in us])
        sp, lq = net.sample(Bs, torch.from_numpy(flat).cuda() if given else None)
        sp, lq = sp.cpu().numpy(), lq.cpu().numpy()
        so = lo = 0
        for q, (n, H, b) in enumerate(CASES[case]):
            s = sp[so:so + b * n].reshape(b, n)
            if b and n:
                rows = np.unique(np.linspace(0, b - 1, 300).astype(int))
                th, u = theta[q].astype(np.float64), us[q].reshape(b, n)[rows]
                _, _, p = OM.sample(th, u, n, H)
                force = np.where(np.abs(p - u) < TIE, s[rows], 0).astype(np.int8)
                want, _, _ = OM.sample(th, u, n, H, force=force)
                assert np.array_equal(want, s[rows]), q
                err = np.abs(lq[lo:lo + b][rows] - OM.logq(th, s[rows], n, H)).max()
                assert err <= (1e-10 if prec == "fp64" else 2e-4) * max(1, n / 8)
            elif b:
                assert not lq[lo:lo + b].any()
            so += b * n
            lo += b
