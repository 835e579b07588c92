"""The process-wide table of tile heights: what it may not change (results, the
pass that runs a cycle's fine level together with the next cycle's) and that
writing back what was read changes nothing."""
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


@pytest.mark.parametrize("prec", [boxmg.BMG_FP64, boxmg.BMG_FP32_IR])
def test_writing_back_what_was_read_changes_nothing(gpu, table, prec):
    """The history's sums follow the tiles of the fine post pass (two sweeps: a
    pass of its own), so equal histories to the bit are equal tiles."""
    st, rhs = problem(1023)
    want = solve(st, rhs, nu2=2, precision=prec)
    for n in SIZES:
        table(n, boxmg.tile_rows_get(n))
    got = solve(st, rhs, nu2=2, precision=prec)
    assert got[1] == want[1] and np.array_equal(got[0], want[0])
    for n in SIZES:
        table(n, 6)
    got = solve(st, rhs, nu2=2, precision=prec)
    assert np.array_equal(got[0], want[0])
