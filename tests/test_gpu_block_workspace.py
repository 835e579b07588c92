"""A block's workspace is the caller's memory, with whatever it last held: the
solutions are those of the right-hand sides alone also when every byte of it
was set (which reads as NaN) before the block was created."""
import pytest
import torch

from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu1,nu2,refine", [(2, 1, 16), (1, 2, 0), (3, 1, 16)])
def test_block_on_memory_that_was_not_clear(gpu, nu1, nu2, refine):
    n, K = 127, 3
    p = inputs.jumping(n, 8, -2.0, 2.0, 31, 32)
    st, rhs = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    B = torch.stack([rhs, 2.0 * rhs.flip(0), torch.zeros_like(rhs)])
    with boxmg.Solver(st, nu1=nu1, nu2=nu2, refine_factor=refine, max_cycles=80) as S:
        want = [S.solve(b, tol=1e-10) for b in B]
        with boxmg.Block(S, K) as clear:
            size = clear.workspace.numel()
        with boxmg.Block(S, K, workspace=torch.full((size,), 255, dtype=torch.uint8, device="cuda")) as blk:
            x, infos = blk.solve(B, tol=1e-10)
    for k in range(K):
        assert infos[k]["cycles"] == want[k][1]["cycles"]
        assert torch.equal(x[k], want[k][0])
