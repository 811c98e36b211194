"""The cost diagonal on either side of the size where its terms change from lanes to scalar loads (n = 20 / 21),
bit for bit the oracle's one-index sums: every diagonal type, dense and sparse pair lists (more than one
chunk of 64 pairs, less than one, none)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    N.lib()
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"


@pytest.mark.parametrize("kind", ["int16", "int32", "real", "sparse", "none"])
@pytest.mark.parametrize("n", [10, 20, 21])
def test_diagonal_equals_the_oracle(n, kind):
    if kind == "int16":
        q = W.dense_integer_symmetric(n, 810 + n)
    elif kind == "int32":
        q = W.dense_integer_symmetric(n, 820 + n, -100000, 100000)
    elif kind == "sparse":
        q = W.regular_graph_qubo(n - n % 2, 830 + n)
    else:
        q = W.dense_gaussian_upper(n, 840 + n)
    H = np.diag(np.diag(q.H)) if kind == "none" else q.H
    pb = Problem(H, q.f, q.c0)
    try:
        d = O.cost_diagonal(H, q.f, q.c0)
        got = pb.diagonal()
        assert np.array_equal(got.astype(np.float64), np.asarray(d, dtype=np.float64))
        assert pb.info.cmin == d.min() and pb.info.cmax == d.max() and pb.info.argmin_index == int(np.argmin(d))
    finally:
        pb.close()
