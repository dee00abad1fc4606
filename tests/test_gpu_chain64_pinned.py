"""FP64 chains (csrc/chain64.hip) with spins held by a field so strong that
exp(-2 beta |f|) is below the smallest double (beta |f| > 373): fields of both
signs, from h or from the width set at a low temperature, in strips of one,
two and four tiles, against the oracle and with the mean spin where the field
puts it.

Tolerances: as test_gpu_chain64.py (ln Z_R 1e-10 a spin; the adjoint's error
model of adjtol.py)."""

import dataclasses

import numpy as np
import pytest

import synthetic as S
from adjtol import check_vjp
from oracle import ising as OI

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

STRIPS = {"one_tile": (8, [4]), "two_tiles": (11, [6]), "four_tiles": (13, [7])}


def _inst(L, cols, how):
    base = S.lattice_column_split(S.lattice_2d(L, seed=L, h_var=0.1), cols)
    R = base.order
    if how == "fields":
        h = base.h.copy()
        h[R[::5]] = -400.0
        h[R[2::7]] = 400.0
        return dataclasses.replace(base, h=h)
    # couplings to the width set alone are strong: beta |f| = 600 beside a
    # column of it, of the sign of its spin
    J = 0.002 * base.J
    inW = np.isin(base.edges, base.width_set)
    J[inW.sum(1) == 1] = 2.0
    return dataclasses.replace(base, J=J, h=0.01 * base.h, beta=300.0)


@pytest.mark.parametrize("how", ["fields", "cold"])
@pytest.mark.parametrize("strip", sorted(STRIPS))
def test_pinned_spins(strip, how):
    from paper_2504_12037_amd import Net
    print(f"\n[chain64-pinned] {strip} {how}", flush=True)
    inst = _inst(*STRIPS[strip], how)
    B = 37
    sp = S.uniform_spins(B, inst.n_width, 3)
    g = np.random.default_rng(4).random(B) + 0.5
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda().reshape(-1)
    net = Net([inst], precision="fp64")
    lz, *vjp = net.logz_and_backward(dev(sp), dev(g), B)
    assert torch.equal(net.logz(dev(sp), B), lz)
    want = OI.logz_r_elimination(inst, sp)
    assert np.abs(lz.cpu().numpy() - want).max() / inst.n <= 1e-10
    got = tuple(x.cpu().numpy() for x in vjp)
    check_vjp(got, OI.logz_r_vjp(inst, sp, g), inst, g, "fp64", (strip, how))
    if how == "fields":
        pinned = np.flatnonzero(np.abs(inst.h) == 400.0)
        assert len(pinned) > 5
        np.testing.assert_allclose(got[0][pinned], np.sign(inst.h[pinned]) * inst.beta * g.sum(),
                                   rtol=1e-9)
