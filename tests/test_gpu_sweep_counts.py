"""Solves with sweep counts that one of the two fine passes does not take (the
fine iterate changes buffers once a cycle), polled several cycles at a time:
cycles enqueued past the stop must not change the result."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("refine", [0, 16])
@pytest.mark.parametrize("nu1,nu2", [(2, 3), (1, 4), (4, 1), (0, 1), (2, 0)])
def test_cycles_past_the_stop(gpu, nu1, nu2, refine):
    n = 63
    p = inputs.jumping(n, 8, -2, 2, 5, 6)
    st, rhs = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    H = ref.Hierarchy(st.cpu().numpy(), nu1=nu1, nu2=nu2)
    u, hist = H.solve(ref.pad(rhs.cpu().numpy()), tol=1e-9, max_cycles=100, refine_factor=refine)
    for every in (1, 2, 3, 8):
        with boxmg.Solver(st, nu1=nu1, nu2=nu2, check_every=every, refine_factor=refine) as S:
            x, info = S.solve(rhs, tol=1e-9)
        assert info["cycles"] == len(hist), every
        assert np.array_equal(x.cpu().numpy(), u[1:-1, 1:-1]), every
