"""The coarsest level's band substitutions on the GPU at the sizes where the
blocks of 16 and phases of 64 unknowns end raggedly: 9 unknowns (less than one
block), 49, 225 and 961 (a partial last block), 3969 (the widest band and the
largest factor), alone and inside the persistent small-level kernel.  The
oracle runs the same fused updates in the same order, so the results are equal."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc", [3, 7, 15, 31, 63])
def test_band_solve_every_coarsest_size(gpu, nc):
    n = max(2 * nc + 1, 31)
    p = inputs.jumping(n, max(1, (n + 1) // 16), -3, 3, 900 + nc, 901 + nc)
    st, rhs = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    H = ref.Hierarchy(st.cpu().numpy(), coarsest=nc)
    Lb, D = H.coarse_factor()
    rng = np.random.default_rng(nc)
    with boxmg.Solver(st, coarsest_n=nc, precision=boxmg.BMG_FP32_IR) as S:
        L = S.nlev - 1
        b = np.zeros((nc + 2, nc + 2))
        for scale in (1.0, 1e-200):          # ordinary values, and products that underflow
            b[1:-1, 1:-1] = rng.standard_normal((nc, nc)) * scale
            S.import_(L, "b", torch.from_numpy(b).cuda())
            S.step(L, "coarse")
            x = ref.band_ldlt_solve(Lb, D, b[1:-1, 1:-1].reshape(-1))
            got = S.export(L, "u").cpu().numpy()
            assert np.array_equal(got[1:-1, 1:-1].reshape(-1), x)
            got[1:-1, 1:-1] = 0.0
            assert not got.any()             # the ring stays zero
        b32 = b.copy()
        b32[1:-1, 1:-1] = rng.standard_normal((nc, nc))
        b32 = b32.astype(np.float32)
        S.import_(L, "b32", torch.from_numpy(b32).cuda())
        S.step(L, "coarse", fp32=True)
        x = ref.band_ldlt_solve(Lb, D, b32[1:-1, 1:-1].reshape(-1).astype(np.float64)).astype(np.float32)
        assert np.array_equal(S.export(L, "u32").cpu().numpy()[1:-1, 1:-1].reshape(-1), x)
    # inside whole cycles (the small-level kernel solves coarsest levels below 63^2 itself)
    with boxmg.Solver(st, coarsest_n=nc, max_cycles=3) as S:
        x, info = S.solve(rhs, tol=0.0, raise_on_noconv=False)
    u, _ = H.solve(ref.pad(rhs.cpu().numpy()), tol=0.0, max_cycles=3)
    H.close()
    assert np.array_equal(x.cpu().numpy(), u[1:-1, 1:-1])
