"""The inner solves of the two-grid objective on the fused cycle, whose stop
test runs on the device with several cycles enqueued at a time: the loss and the
gradient planes of the separate kernels, bit for bit, where a solve ends inside
a batch of cycles, at its end, at its first cycle and at the cycle limit, on a
coarse level of one and of several levels, with sweep counts that move the
iterate twice a cycle and once."""
import numpy as np
import pytest
import torch

from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,coarsest,nu1,nu2", [(31, 15, 2, 1), (31, 3, 2, 1), (127, 15, 1, 2), (127, 3, 2, 3),
                                                (255, 15, 2, 1)])
def test_level_solves_match_separate_kernels(gpu, n, coarsest, nu1, nu2):
    p = inputs.jumping(n, max(2, (n + 1) // 16), -2.0, 2.0, n, n + 1)
    st, _ = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    r0 = torch.from_numpy(np.random.default_rng(n).standard_normal((n, n))).cuda()
    net = boxmg.Net(inputs.net_random(7) * np.float32(0.01), max_n=n, train=True)
    got = {}
    for kern in (boxmg.BMG_KERNELS_FUSED, boxmg.BMG_KERNELS_BASIC):
        with boxmg.Solver(st, interp=boxmg.BMG_INTERP_LEARNED, learned_levels=1, net=net, coarsest_n=coarsest,
                          nu1=nu1, nu2=nu2, kernels=kern) as S:
            got[kern] = []
            for tol, limit in ((1e-10, 60), (1e-4, 60), (0.9, 60), (0.0, 1), (0.0, 6), (0.0, 8)):
                loss, d = net.twogrid(S, r0, inner_tol=tol, inner_max=limit, want_grad_planes=True)
                got[kern].append((loss, d.cpu().numpy().copy()))
    for (a, da), (b, db) in zip(*got.values()):
        assert a == b and np.array_equal(da, db)
