"""Top-k of a state that holds no number (device parameters are not checked on the host): no index is
returned and no diagonal entry is read for a rank that nothing fills."""
import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [6, 14])
def test_nan_parameters_fill_no_rank(n):
    import torch

    q = W.dense_integer_symmetric(n, 31)
    pb = Problem(q.H, q.f, q.c0)
    try:
        x = torch.full((4,), float("nan"), dtype=torch.float64, device="cuda")
        for flags in (0, N.QQ_C128):
            idx, prob, cost = N.qq_topk(pb.handle, 2, x, flags | N.QQ_PARAMS_ON_DEVICE, 5)
            assert np.all(idx == np.uint64(2**64 - 1)) and np.all(prob == -1.0) and np.all(np.isnan(cost))
    finally:
        pb.close()
