"""Small deeper networks sampled on 16 lanes a sample and on four (csrc/made.hip),
which the batch size chooses between: the same spins and ln q for the samples
that a small and a large batch share, on both sides of every line of the rule
(|W| = 14, units above 32, four layers, FP64)."""

import numpy as np
import pytest

import synthetic as S
from oracle import made as OM

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (|W|, H, depth)
CASES = [(3, 64, 2), (5, 16, 3), (6, 32, 2), (9, 40, 4), (13, 33, 3), (14, 16, 4), (33, 64, 4)]


def _inst(n, H, depth):
    N = n + 4
    e = np.sort(np.stack([np.arange(N), (np.arange(N) + 1) % N], 1), 1).astype(np.int32)
    i = S.Instance(N, e, np.random.default_rng(n).standard_normal(N), np.zeros(N), 1.0,
                   np.arange(n, dtype=np.int32), np.arange(n, N, dtype=np.int32), None, H, f"w{n}")
    i.depth = depth
    return i


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_lanes_draw_the_same_spins(case, prec):
    from paper_2504_12037_amd import Net
    n, H, depth = case
    print(f"\n[lanes] {case} {prec}", flush=True)
    net = Net([_inst(n, H, depth)], precision=prec, seed=6)
    th = 0.4 * np.random.default_rng(n).standard_normal(OM.param_count(n, H, depth))
    net.set_params(0, torch.from_numpy(th.astype(np.float32)))
    B = 16400
    sp, lq = (x.clone() for x in net.sample(B))
    for b in (61, 8192):
        s, l = net.sample(b)
        assert torch.equal(s, sp[:b * n])
        # (a sum of |W| terms of order one in either order)
        assert (l - lq[:b]).abs().max().item() <= n * (1e-14 if prec == "fp64" else 1e-5)
