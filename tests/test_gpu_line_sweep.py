"""Line relaxation in one launch per half-sweep (levels up to 1023 points) and
in separate launches (2047): sizes below, at and above one round of the
recurrence (16 pairs of rows), lines that end inside a workgroup's group of
columns, and the larger levels' route, each relaxation equal to the oracle's."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 7, 15, 31, 63, 1023, 2047])
def test_line_relaxation_matches_oracle(gpu, n):
    p = inputs.jumping(n, max(1, (n + 1) // 16), -2, 2, 40 + n, 41 + n)
    st, _ = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    H = ref.Hierarchy(st.cpu().numpy())
    rng = np.random.default_rng(n)
    with boxmg.Solver(st, smoother=boxmg.BMG_SMOOTH_LINE) as S:
        for l in range(min(2, H.nlev)):          # the five-point and the first nine-point level
            m = S.level_n(l)
            u, b = np.zeros((m + 2, m + 2)), np.zeros((m + 2, m + 2))
            u[1:-1, 1:-1] = rng.standard_normal((m, m))
            b[1:-1, 1:-1] = rng.standard_normal((m, m))
            S.import_(l, "u", torch.from_numpy(u).cuda())
            S.import_(l, "b", torch.from_numpy(b).cuda())
            S.step(l, "smooth", 2)
            planes = [S.export(l, f).cpu().numpy() if (l > 0 or f in ("O", "W", "S")) else None
                      for f in ("O", "W", "S", "SW", "NW")]
            want = ref.line_relax(*planes, ref.line_factor(*planes[:3]), b, u, 2)
            assert np.array_equal(S.export(l, "u").cpu().numpy(), want), l
    H.close()
