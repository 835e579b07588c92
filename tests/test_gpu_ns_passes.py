"""Nonsymmetric solves on a five-point fine level, whose cycle runs that level's
steps as two fused passes, against the oracle's separate steps: levels of less
than a strip, a strip and a few columns more and several, blocks of rows
streamed both ways, one and two sweeps on either side and counts that the
passes do not take, the separate kernels, and a handle that solves twice."""
import numpy as np
import pytest

from oracle import ref
from paper_2502_05279_amd import boxmg
from test_gpu_ns import cd_problem, dev, host, same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nu1,nu2", [(7, 2, 1), (15, 1, 1), (63, 2, 2), (127, 1, 2), (127, 2, 1), (127, 3, 1),
                                       (255, 2, 0), (255, 2, 1), (511, 2, 1)])
def test_ns_fused_cycles_match_oracle(gpu, n, nu1, nu2):
    st, rhs = cd_problem(n, 40.0, seed=n)
    H = ref.NSHierarchy(st, nu1=nu1, nu2=nu2)
    for kern in (boxmg.BMG_KERNELS_FUSED, boxmg.BMG_KERNELS_BASIC):
        with boxmg.NSSolver(dev(st), nu1=nu1, nu2=nu2, kernels=kern, max_cycles=60) as S:
            for scale, tol in ((1.0, 1e-9), (-3.0, 1e-4)):
                u, hist = H.solve(ref.pad(scale * rhs), tol=tol, max_cycles=60)
                x, info = S.solve(dev(scale * rhs), tol=tol)
                assert info["cycles"] == len(hist)
                same(host(x), u[1:-1, 1:-1], "solution")
                h = np.array(info["history"])
                assert np.all(np.abs(h - hist) <= 1e-12 * np.asarray(hist))
