"""Complex128 phases at angles where the reduction's first step leaves a remainder beyond pi/4 (from about
2^44 on), up to the largest finite ones, against the FP64 oracle on integer instances (C and gamma C are then
the same doubles on both sides).

Tolerance.  As in test_gpu_c128.py, without the rounding of gamma C: a state is within p (3 n + 4) 2^-52 on
either side; the reduction of theta = gamma C rounds a remainder of up to |theta| 2^-52 twice, |theta| 2^-104
per layer.  Far beyond 2^52 only the norm is defined to that accuracy."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem, evaluate_many

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    N.lib()
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"


@pytest.mark.parametrize("gamma", [1e6, 3e11, 1e13, 1e15, 1e16, 1e18])
@pytest.mark.parametrize("n", [5, 12, 13, 17])
def test_large_angles(n, gamma):
    q = W.dense_integer_symmetric(n, 90 + n)
    pb = Problem(q.H, q.f, q.c0)
    p = 2
    x = W.random_params(p, 2, 91 + n)
    x[:, 0::2] *= gamma
    d = O.cost_diagonal(q.H, q.f, q.c0)
    cmax = float(np.max(np.abs(d)))
    try:
        pb.set_allocation([i % 2 for i in range(n)], 2)
        e, g = pb.evaluate(x, grad=True, c128=True)
        runs = [(e, g)]
        em, gm = evaluate_many([pb], [x], grad=True, c128=True)
        runs.append((em[0], gm[0]))
        if n > 12:  # one rotation by the sum of the two parts, exact for integers
            runs.append(pb.evaluate(x, grad=True, c128=True, partitioned=True))
        for b in range(2):
            theta = float(np.max(np.abs(x[b, 0::2]))) * cmax
            s = 2 * p * (3 * n + 4) * 2.0**-52 + p * theta * 2.0**-104
            assert np.linalg.norm(pb.state(x[b], c128=True) - O.qaoa_state(d, x[b])) <= s
            er, gr = O.gradient(d, x[b])
            for ev, gv in runs:
                assert abs(ev[b] - er) <= 2 * cmax * s
                assert np.max(np.abs(gv[b] - gr)[1::2]) <= 4 * n * cmax * s
                assert np.max(np.abs(gv[b] - gr)[0::2]) <= 4 * cmax**2 * s
    finally:
        pb.close()


@pytest.mark.parametrize("gamma", [1e25, 1e100, 1e300])
@pytest.mark.parametrize("n", [5, 13])
def test_the_norm_is_kept_at_any_angle(n, gamma):
    q = W.dense_integer_symmetric(n, 95 + n)
    pb = Problem(q.H, q.f, q.c0)
    p = 3
    x = W.random_params(p, 1, 96 + n)[0]
    x[0::2] *= gamma
    try:
        s = 2 * p * (3 * n + 4) * 2.0**-52
        assert abs(np.linalg.norm(pb.state(x, c128=True)) - 1.0) <= s
        e = pb.evaluate(x, c128=True)
        assert pb.info.cmin - 1.0 <= e[0] <= pb.info.cmax + 1.0
    finally:
        pb.close()
