"""FP32 refinement steps whose fine post pass also updates the double-FP64
iterate and takes the next residual, against the oracle's separate steps:
levels of less than a strip, a strip and a few columns more and several strips,
tiles of two rows, ragged last tiles, tiles streamed both ways, one and two
sweeps on either side, three before, and steps polled one, two and three at a
time (the pair alternates between two buffers, and steps enqueued past the stop
must leave it alone), on a handle that solves twice."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows,nu1,nu2,every", [
    (7, 2, 2, 1, 1), (15, 2, 1, 1, 2), (63, 2, 2, 2, 3), (127, 0, 2, 1, 2), (127, 6, 1, 2, 1), (255, 34, 2, 1, 3),
    (255, 0, 3, 1, 2), (511, 0, 2, 1, 1),
])
def test_refinement_steps_match_oracle(gpu, n, rows, nu1, nu2, every):
    p = inputs.jumping(n, max(1, (n + 1) // 16), -2, 2, 40 + n, 41 + n)
    st, rhs = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    H = ref.Hierarchy(st.cpu().numpy(), nu1=nu1, nu2=nu2)
    b = ref.pad(rhs.cpu().numpy())
    with boxmg.Solver(st, precision=boxmg.BMG_FP32_IR, tile_rows=rows, nu1=nu1, nu2=nu2, check_every=every,
                      max_cycles=100) as S:
        for tol in (1e-12, 1e-5):
            u, hist = H.solve_ir(b, tol=tol, max_iter=100)
            x, info = S.solve(rhs, tol=tol)
            assert info["cycles"] == len(hist) - 1
            assert np.array_equal(x.cpu().numpy(), u[1:-1, 1:-1]), "high part"
            assert np.array_equal(S.export(0, "xlo").cpu().numpy(), H.xl), "low part"
            h = np.array(info["history"])
            assert np.all(np.abs(h - hist) <= 1e-12 * np.asarray(hist))
