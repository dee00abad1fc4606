"""Graphs whose widest scope is 11 to 14 spins, the last that have full transfer
tables: forward on the level kernels (csrc/sweep.hip) at every one of them, the
adjoint there while its joint weights fit the LDS and step by step
(csrc/contract.hip) past that, on one net in turn; ln Z_R bit for bit that of a
tile of 16, which is the step-by-step kernel's, and both against the oracle."""

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
@pytest.mark.parametrize("n,w_u", [(96, 11), (96, 12), (100, 13), (108, 14), (256, 14)])
def test_widest_tables(n, w_u, prec):
    from paper_2504_12037_amd import Net
    print(f"\n[level-scopes] n={n} w_u={w_u} {prec}", flush=True)
    inst = _graph(n, w_u, 50 + w_u)
    B = 5
    sp = S.uniform_spins(B, inst.n_width, 3)
    g = np.random.default_rng(4).standard_normal(B)
    flat, gd = torch.from_numpy(sp).cuda().reshape(-1), torch.from_numpy(g).cuda()
    net = Net([inst], precision=prec)
    # a larger batch first: other tiles of the same net
    many = torch.from_numpy(S.uniform_spins(700, inst.n_width, 8)).cuda().reshape(-1)
    net.logz_and_backward(many, torch.ones(700, dtype=torch.float64, device="cuda"), 700)
    lz, *vjp = (x.clone() for x in net.logz_and_backward(flat, gd, B))
    assert torch.equal(net.logz(flat, B), lz)
    ref = Net([inst], precision=prec)
    ref.set_tuning(general_tile_fwd=16)
    assert torch.equal(ref.logz(flat, B), lz)
    want = OI.logz_r_elimination(inst, sp, chunk=1)
    assert np.abs(lz.cpu().numpy() - want).max() / inst.n <= {"fp64": 1e-10, "fp32": 1e-5}[prec]
    check_vjp(tuple(x.cpu().numpy() for x in vjp), OI.logz_r_vjp(inst, sp, g), inst, g, prec, w_u)
