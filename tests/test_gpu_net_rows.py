"""The network's first two layers in one pass, where a workgroup streams through
several rows: nine strips of columns and blocks of ten rows (the last one
ragged), five- and nine-point levels, a smaller level after a larger one in the
same arrays, and an inference network's exports; by the checks of the layers on
small levels."""
import numpy as np
import pytest

from oracle import learned
from paper_2502_05279_amd import boxmg, inputs
from test_gpu_learned import check_interval, gpu_forward, host, level_planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [5, 9])
def test_net_layers_row_blocks(gpu, kind):
    theta = inputs.net_random(3 + kind)
    p = learned.rounded(learned.unpack(theta), True)
    pa = {k: np.abs(v) for k, v in p.items()}
    net = boxmg.Net(theta, max_n=1023, train=False)
    for n in (1023, 127):
        planes, _, _ = level_planes(kind, n, 21 + n)
        nc = (n - 1) // 2
        _, X, H1, H2 = gpu_forward(net, planes)
        Xo = learned.features(*[None if a is None else host(a) for a in planes])
        assert np.array_equal(X[:, :, :9], Xo) and not X[:, :, 9:].any()
        # rows at both ends of the level and on both sides of block borders
        for first, last in ((1, 8), (nc // 2 - 8, nc // 2 + 8), (nc - 8, nc + 1)):
            J, I = np.arange(first, last + 1), np.arange(1, nc + 2)
            fj, fi = np.arange(2 * first - 1, min(2 * last, n) + 1), np.arange(1, n + 1)
            z = learned.conv(X[:, :, :9], p["W1"], p["b1"], fj, fi)
            a = learned.conv(np.abs(X[:, :, :9]), pa["W1"], pa["b1"], fj, fi)
            check_interval(H1[fj[0]:fj[-1] + 1, 1:n + 1], z, a, 81, "H1", relu=True)
            z = learned.conv(H1, p["W2"], p["b2"], 2 * J, 2 * I)
            a = learned.conv(np.abs(H1), pa["W2"], pa["b2"], 2 * J, 2 * I)
            check_interval(H2[first:last + 1, 1:nc + 2], z, a, 288, "H2", relu=True)
        for A, m in ((H1, n), (H2, nc + 1)):
            ring = A.copy()
            ring[1:m + 1, 1:m + 1] = 0
            assert not ring.any()
