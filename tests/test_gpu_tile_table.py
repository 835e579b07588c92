"""What the process-wide table of tile heights may not change: results, and the
pass that runs a cycle's fine level together with the next cycle's."""
import numpy as np
import pytest
import torch

from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu

SIZES = [(1 << m) - 1 for m in range(2, 12)]


@pytest.fixture
def table():
    yield boxmg.tile_rows_set
    for n in SIZES:
        boxmg.tile_rows_set(n, 0)


def problem(n):
    p = inputs.jumping(n, max(2, (n + 1) // 16), -2.0, 2.0, n, n + 1)
    return boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())


def solve(st, rhs, **kw):
    with boxmg.Solver(st, coarsest_n=15, max_cycles=24, **kw) as S:
        S.trace_enable("postpre", 0)
        x, info = S.solve(rhs, tol=0.0, raise_on_noconv=False)
        return x.cpu().numpy(), info["history"], S.trace_read()[0]


def test_cross_cycle_pass_keeps_its_own_height(gpu, table):
    """Heights of two rows for every level: the fine level's pass across cycles
    (whose tiles leave a partial sum each, at most 8192) still runs."""
    st, rhs = problem(2047)
    want = solve(st, rhs)
    for n in SIZES:
        table(n, 2)
    got = solve(st, rhs)
    assert got[2] == want[2] > 0 and np.array_equal(got[0], want[0])
