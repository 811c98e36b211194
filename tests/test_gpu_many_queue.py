"""The persistent launch's queue where its segment search has far to go: thousands of one-item segments
(more than one probe spans), on three workgroups, on all, and with every automatic choice, in both
precisions.  The grid does not change a result by a bit; against per-problem calls the results differ
by the order of FP64 sums and, in complex64, by the set order's rounding (1e-5 of max(|E|, sigma_C))."""
import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem, evaluate_many

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    N.lib()
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"


@pytest.mark.parametrize("c128,tol", [(False, 1e-5), (True, 1e-11)])
def test_long_segment_lists(c128, tol):
    shapes = [(13, 1, 3000), (11, 2, 5000), (17, 3, 2)]
    pbs, xs = [], []
    for k, (n, p, B) in enumerate(shapes):
        q = W.dense_integer_symmetric(n, 800 + k)
        pbs.append(Problem(q.H, q.f, q.c0))
        xs.append(W.random_params(p, B, 810 + k))
    try:
        runs = [evaluate_many(pbs, xs, grad=True, options=o, c128=c128)
                for o in (dict(tiles_per_chunk=1, max_workgroups=3), dict(tiles_per_chunk=1), None)]
        for e, g in runs[1:2]:
            for a, b in zip(runs[0][0] + runs[0][1], e + g):
                assert np.array_equal(a, b)
        for pb, x, e, g in zip(pbs, xs, *runs[2]):
            er, gr = pb.evaluate(x, grad=True, c128=c128)
            s = pb.info.sigma_c
            assert np.max(np.abs(e - er) / np.maximum(np.abs(er), s)) <= tol
            # gradients: the complex64 bound of qq_evaluate_guarded for either side
            b = np.max(np.abs(gr), axis=1)
            lim = tol * np.maximum(b, s) if c128 else 2 * (N.QQ_GUARD_REL * b + N.QQ_GUARD_K * s * s * 2.0**-24
                                                           * 2.0 ** (-0.5 * pb.n))
            assert np.all(np.max(np.abs(g - gr), axis=1) <= lim)
    finally:
        for pb in pbs:
            pb.close()
