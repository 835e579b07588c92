"""Where the coarse levels start to run in one workgroup: by default and at
every limit, with the coarsest sizes on both sides of the default's rule, the
solve of the separate kernels bit for bit."""
import numpy as np
import pytest
import torch

from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n,nc", [(15, 3), (63, 7), (127, 3), (127, 15), (255, 31)])
def test_small_level_limits(gpu, n, nc, fp32):
    p = inputs.jumping(n, max(1, (n + 1) // 16), -2, 2, 15 + n, 16 + n)
    st, rhs = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    opts = dict(coarsest_n=nc, precision=boxmg.BMG_FP32_IR if fp32 else boxmg.BMG_FP64)

    def solve(**kw):
        with boxmg.Solver(st, **opts, **kw) as S:
            x, info = S.solve(rhs, tol=1e-9)
        return info["cycles"], x.cpu().numpy()

    want = solve(kernels=boxmg.BMG_KERNELS_BASIC)
    for limit in (0, 1, 3, 7, 15, 31, 63):
        got = solve(persistent_below_n=limit)
        assert got[0] == want[0] and np.array_equal(got[1], want[1]), limit
