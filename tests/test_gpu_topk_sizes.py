"""Top-k against a sort of the same state's probabilities (qq_probabilities): k up to the whole state, sizes on
either side of the sweep's workgroup rule (1024 beyond n = 26), and states of equal amplitudes, where every
entry ties and the lowest indices win."""
import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    N.lib()
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"


@pytest.mark.parametrize("n,ks", [(1, (1, 2)), (4, (1, 16)), (9, (5, 16)), (14, (1, 16)), (19, (1, 3, 16)), (27, (1, 16))])
def test_topk_is_the_head_of_the_sorted_probabilities(n, ks):
    q = W.dense_integer_symmetric(n, 610 + n)
    pb = Problem(q.H, q.f, q.c0)
    try:
        x = W.random_params(2, 1, 620 + n)[0]
        flat = np.zeros(4)
        for c128 in (False, True) if n < 20 else (False,):
            P = pb.probabilities(x, c128=c128)
            k = max(ks)
            cand = np.flatnonzero(P >= np.partition(P, P.size - k)[P.size - k])
            ref = cand[np.lexsort((cand, -P[cand]))]  # by decreasing probability, ties to the lower index
            for k in ks:
                idx, prob, _ = pb.topk(x, k=k, c128=c128)
                assert np.array_equal(idx.astype(np.int64), ref[:k]) and np.array_equal(prob, P[ref[:k]]), (k, c128)
                idx, prob, _ = pb.topk(flat, k=k, c128=c128)  # the uniform superposition
                assert np.array_equal(idx, np.arange(k, dtype=np.uint64)), (k, c128)
    finally:
        pb.close()
