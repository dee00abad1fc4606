"""Event times of the chain launch that a net of two widths runs
(tnvan_kernel_time): the launch of both is timed as it is, and only timing a
width alone splits it; either way the same bits."""

import pytest

import synthetic as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_the_launch_of_both_widths_is_timed():
    from paper_2504_12037_amd import Net
    inst = S.c2_lattice(1.0, 0)       # strips of five, four and five columns
    B = 300
    sp = torch.from_numpy(S.uniform_spins(B, inst.n_width, 3)).cuda().reshape(-1)
    g = torch.full((B,), 1.0 / B, dtype=torch.float64, device="cuda")
    net = Net([inst], precision="fp32", flags=Net.FLAG_PROFILE)
    outs = []
    for names, counts in ((["chain_fwd_all", "chain_bwd_all"], {"chain_fwd_all": 1, "chain_bwd_all": 1}),
                          (["chain_fwd_2", "chain_bwd_1"], {"chain_fwd_2": 1, "chain_bwd_1": 1}),
                          ([], {})):
        net.profile_only(names)
        out = [net.logz(sp, B).clone(), *(x.clone() for x in net.backward(sp, g, B))]
        torch.cuda.synchronize()
        for k in Net.KERNELS:
            t, n = net.kernel_time(k)
            assert n == counts.get(k, 0), (names, k)
            assert (t > 0) == (n > 0)
        outs.append(out)
    for o in outs[1:]:
        assert all(torch.equal(x, y) for x, y in zip(o, outs[0]))
