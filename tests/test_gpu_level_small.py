"""Level kernels (csrc/sweep.hip) on small graphs with few leaves, where some
waves of a workgroup have no unit of their own until the marginals of the
reverse pass (the graphs behind these seeds were picked for that): ln Z_R, the
adjoint and the jets at every tile against the oracle."""

import numpy as np
import pytest

import synthetic as S
from adjtol import check_vjp
from oracle import ising as OI

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SEEDS = (77, 701, 717, 932, 1051, 1331)


def _inst(seed):
    rng = np.random.default_rng(seed)
    n = int(rng.integers(16, 36))
    m = int(rng.integers(n, 2 * n))
    e = np.sort(rng.integers(0, n, (m, 2)), 1)
    e = np.unique(e[e[:, 0] < e[:, 1]], axis=0).astype(np.int32)
    perm = rng.permutation(n)
    k = int(rng.integers(0, n // 2))
    return S.Instance(n, e, rng.standard_normal(len(e)), rng.normal(0.0, 0.3, n), 0.8,
                      np.sort(perm[:k]).astype(np.int32), perm[k:].astype(np.int32), None, 0, f"g{seed}")


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("tile", [1, 2, 4, 8])
def test_small_graphs(prec, tile):
    from paper_2504_12037_amd import Net
    B = 21
    for seed in SEEDS:
        print(f"\n[level-small] {prec} tile {tile} seed {seed}", flush=True)
        inst = _inst(seed)
        sp = S.uniform_spins(B, inst.n_width, seed)
        g = np.random.default_rng(seed).standard_normal(B)
        flat = torch.from_numpy(sp).cuda().reshape(-1)
        net = Net([inst], precision=prec)
        net.set_tuning(general_tile_fwd=tile, general_tile_bwd=tile)
        lz, *vjp = net.logz_and_backward(flat, torch.from_numpy(g).cuda(), B)
        assert torch.equal(net.logz(flat, B), lz)
        want = OI.logz_r_elimination(inst, sp)
        # (the jets round each product and sum, the forward pass once)
        for z in (lz, net.remainder_moments(flat, B)[0]):
            assert np.abs(z.cpu().numpy() - want).max() / inst.n <= {"fp64": 1e-10, "fp32": 1e-5}[prec]
        check_vjp(tuple(x.cpu().numpy() for x in vjp), OI.logz_r_vjp(inst, sp, g), inst, g, prec, seed)
