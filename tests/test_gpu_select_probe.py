"""The probe cycles of a solve that chooses between a learned and an
operator-induced hierarchy run their coarse levels as any cycle does: a 31^2
level and those below it in one workgroup, on handles that no other call has
used, so no fused pass of that level is launched."""
import numpy as np
import pytest
import torch

from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


def test_probe_runs_small_levels_in_one_workgroup(gpu):
    n = 127
    p = inputs.jumping(n, 8, -2.0, 2.0, 11, 12)
    st, rhs = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    net = boxmg.Net(inputs.net_random(7) * np.float32(0.01), max_n=n, train=False)
    learned = boxmg.Solver(st, interp=boxmg.BMG_INTERP_LEARNED, learned_levels=1, net=net, max_cycles=200)
    plain = boxmg.Solver(st, max_cycles=200)
    with learned as a, plain as b:
        assert a.level_n(2) == 31
        for S in (a, b):
            S.trace_enable("pre", 2)
        _, info, _, _ = boxmg.solve_select(a, b, rhs, tol=1e-9, probe_cycles=4)
        assert info["status"] == boxmg.BMG_OK
        assert [S.trace_read()[0] for S in (a, b)] == [0, 0]
