"""Complex128 gradients to bounds that a single-precision error anywhere in the adjoint sweep would miss: at
moderate phase angles the worst-case bounds of test_gpu_c128.py are below 1e-10 of the gradient's largest
component (asserted for every row), for every diagonal type, at one tile, one qubit above it, one partial
and one full high set, and three sets, through the per-problem call, the many-problem launch and the
partitioned phases (whose two forms carry the roundings of one cost each: twice the bound)."""
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


def instance(kind, n, seed):
    if kind == "int16":
        return W.dense_integer_symmetric(n, seed)
    if kind == "int32":
        return W.dense_integer_symmetric(n, seed, -100000, 100000)
    return W.dense_gaussian_upper(n, seed)


@pytest.mark.parametrize("kind", ["int16", "int32", "real"])
@pytest.mark.parametrize("n,p", [(3, 2), (12, 3), (13, 2), (16, 3), (17, 1), (20, 2), (21, 2)])
def test_gradients_are_double_precision_throughout(kind, n, p):
    q = instance(kind, n, 200 + n)
    d = O.cost_diagonal(q.H, q.f, q.c0)
    cmax = float(np.max(np.abs(d)))
    x = W.random_params(p, 1, 300 + n)
    x[:, 0::2] *= 0.5 / float(np.std(d))
    er, gr = O.gradient(d, x[0])
    s = 2 * p * (3 * n + 4 + n * np.max(np.abs(x[:, 0::2])) * cmax) * 2.0**-52
    be, bb, bg = 2 * cmax * s, 4 * n * cmax * s, 4 * cmax**2 * s
    assert bb <= 1e-10 * np.max(np.abs(gr[1::2])) and bg <= 1e-10 * np.max(np.abs(gr[0::2]))
    pb = Problem(q.H, q.f, q.c0)
    try:
        pb.set_allocation([i % 3 for i in range(n)], 3)
        em, gm = evaluate_many([pb], [x], grad=True, c128=True)
        for f, (e, g) in ((1, pb.evaluate(x, grad=True, c128=True)), (1, (em[0], gm[0])),
                          (2, pb.evaluate(x, grad=True, c128=True, partitioned=True))):
            assert abs(e[0] - er) <= f * be
            assert np.max(np.abs(g[0] - gr)[1::2]) <= f * bb, (g, gr)
            assert np.max(np.abs(g[0] - gr)[0::2]) <= f * bg, (g, gr)
    finally:
        pb.close()
