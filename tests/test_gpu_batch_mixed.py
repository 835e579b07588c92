"""Batches whose work lists are short, ragged or dominated by one problem: a
single problem, only problems that fit the per-problem sub-cycle (no tiled
level), a large one among small ones (more tiles than workgroups on its fine
level, idle workgroups elsewhere), twice on one handle.  Every problem's
solution and history are those of its own FP32-in-FP64 refinement."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(7,), (31, 7, 15), (63,), (511, 7, 31, 63, 7), (255, 255, 127)])
def test_batch_of_uneven_problems(gpu, sizes):
    rng = np.random.default_rng(sum(sizes))
    sts, rhss = [], []
    for n in sizes:
        k, f = inputs.lognormal_k(n, 1.5, rng), rng.uniform(-1.0, 1.0, (n, n))
        st, rhs = boxmg.discretize(torch.from_numpy(k).cuda(), torch.from_numpy(f).cuda())
        sts.append(st)
        rhss.append(rhs)
    with boxmg.Batch(sts, max_cycles=60) as B:
        for _ in range(2):
            x, steps, rel, status = B.solve(rhss, tol=1e-10)
            assert status == boxmg.BMG_OK
            for p in range(len(sizes)):
                H = ref.Hierarchy(sts[p].cpu().numpy())
                u, hist = H.solve_ir(ref.pad(rhss[p].cpu().numpy()), tol=1e-10, max_iter=60)
                H.close()
                assert steps[p] == len(hist) - 1
                assert np.array_equal(x[p].cpu().numpy(), u[1:-1, 1:-1]), (p, sizes[p])
                h = np.array(B.history(p))
                assert np.all(np.abs(h - hist) <= 1e-12 * hist) and rel[p] == h[-1]
