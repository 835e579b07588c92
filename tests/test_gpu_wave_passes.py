"""The fused passes as streams of single waves (the fine five-point level and the
nine-point level below it), against the oracle's separate steps: one and two sweeps, tiles of two rows, ragged last
tiles and strips (levels of 7 to 255 points: less than a strip, a strip and a
few columns more, several), tiles streamed upward and downward, FP64 and FP32."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2502_05279_amd import boxmg, inputs

pytestmark = pytest.mark.gpu

PLANES = ("O", "W", "S", "SW", "NW")


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n,rows", [(15, 2), (31, 6), (63, 0), (255, 2), (255, 10), (511, 34), (511, 0)])
def test_wave_passes_match_oracle(gpu, n, rows, fp32):
    p = inputs.jumping(n, max(1, (n + 1) // 16), -3, 3, 60 + n, 61 + n)
    st, _ = boxmg.discretize(torch.from_numpy(p.k).cuda(), torch.from_numpy(p.f).cuda())
    dt, sfx = (np.float32, "32") if fp32 else (np.float64, "")
    rng = np.random.default_rng(n + rows)
    prec = boxmg.BMG_FP32_IR if fp32 else boxmg.BMG_FP64
    with boxmg.Solver(st, precision=prec, tile_rows=rows, square_tiles_below_n=1, coarsest_n=3) as S:
        def level(k):
            a = np.zeros((k + 2, k + 2), dtype=dt)
            a[1:-1, 1:-1] = rng.standard_normal((k, k))
            return a

        for l in (0, 1):
            m, nc = S.level_n(l), S.level_n(l + 1)
            op = [S.export(l, f + sfx).cpu().numpy() if (l or f in ("O", "W", "S")) else None for f in PLANES]
            Ci = S.export(l, "Ci" + sfx).cpu().numpy()
            check(S, l, m, nc, op, Ci, sfx, dt, level, fp32)


def check(S, l, m, nc, op, Ci, sfx, dt, level, fp32):
    for nu in (1, 2):
        u, b = level(m), level(m)
        S.import_(l, "u" + sfx, torch.from_numpy(u).cuda())
        S.import_(l, "b" + sfx, torch.from_numpy(b).cuda())
        S.step(l, "pre", nu, fp32=fp32)
        want = ref.gs(*op, b, u, nu, dtype=dt)
        assert np.array_equal(S.export(l, "u" + sfx).cpu().numpy(), want), ("pre u", l, nu)
        bc = ref.restrict(Ci, ref.residual(*op, b, want, dtype=dt), dtype=dt)
        assert np.array_equal(S.export(l + 1, "b" + sfx).cpu().numpy(), bc), ("pre b_c", l, nu)
        u, ec = level(m), level(nc)
        S.import_(l, "u" + sfx, torch.from_numpy(u).cuda())
        S.import_(l + 1, "u" + sfx, torch.from_numpy(ec).cuda())
        S.step(l, "post", nu, fp32=fp32)
        want = ref.gs(*op, b, ref.interp_add(Ci, ec, u, dtype=dt), nu, dtype=dt)
        assert np.array_equal(S.export(l, "u" + sfx).cpu().numpy(), want), ("post", l, nu)
