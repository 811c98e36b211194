"""Large problems in the persistent launch, around the sizes where the units of partial sums change (8 tiles at
n = 23 to 25, 16 from n = 26): the same bits alone, beside other problems and under a limit on the tiles per item
that is a multiple of the unit; energies against the per-problem call."""
import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem, evaluate_many

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c128", [(23, False), (24, False), (24, True), (25, False), (25, True), (26, False), (26, True)])
def test_large_problems_alone_and_beside_others(n, c128):
    q = W.dense_integer_symmetric(n, 700 + n)
    pb = Problem(q.H, q.f, q.c0)
    small = [Problem(*(lambda i: (i.H, i.f, i.c0))(W.dense_integer_symmetric(13 + k, 720 + k))) for k in range(6)]
    x = W.random_params(2, 1, 730 + n)
    xs = [W.random_params(1 + k % 3, 2, 740 + k) for k in range(6)]
    try:
        (e,), (g,) = evaluate_many([pb], [x], grad=True, c128=c128)
        e, g = np.copy(e), np.copy(g)
        for options in (None, dict(tiles_per_chunk=16), dict(tiles_per_chunk=64, max_workgroups=128)):
            e2, g2 = evaluate_many([pb] + small, [x] + xs, grad=True, c128=c128, options=options)
            assert np.array_equal(e2[0], e) and np.array_equal(g2[0], g), options
        ref = pb.evaluate(x, c128=c128)
        # the same passes in another set order: complex128 rounding, or complex64's (header: 1e-5)
        assert abs(ref[0] - e[0]) <= (1e-11 if c128 else 1e-5) * max(abs(ref[0]), pb.info.sigma_c)
    finally:
        for p in [pb] + small:
            p.close()
