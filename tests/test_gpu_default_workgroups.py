"""The default workgroups per state: 128 at most for complex64 batches of 16 and more at n = 20 to 22, 16384 over the
batch or one per tile elsewhere.  On both sides of each edge the default's results equal those of the other
number, up to the order of the FP64 sums (the states are the same bits; 1e-12 of the largest value)."""
import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,B,c128,G", [
    (19, 64, False, 128), (20, 15, False, 256), (20, 16, False, 128), (20, 64, False, 128), (20, 200, False, 64),
    (20, 16, True, 256), (21, 15, False, 512), (21, 33, False, 128), (22, 16, False, 128), (22, 16, True, 1024),
    (23, 16, False, 1024), (24, 2, False, 4096),
])
def test_default_workgroups(n, B, c128, G):
    q = W.dense_integer_symmetric(n, 300 + n)
    pb = Problem(q.H, q.f, q.c0)
    try:
        flags = N.QQ_ENERGY | N.QQ_GRAD | (N.QQ_C128 if c128 else 0)
        got = N.qq_get_schedule(pb.handle, 2, B, flags)
        assert got["workgroups_per_state"] == G and got["pinned"] == 0
        x = W.random_params(2, B, 400 + n)
        e, g = pb.evaluate(x, grad=True, c128=c128)
        other = 256 if G == 128 else 128
        if other > 1 << (n - 12):
            other = 64
        N.qq_set_schedule(pb.handle, 2, B, flags, dict(workgroups_per_state=other, set_order=got["set_order"]))
        e2, g2 = pb.evaluate(x, grad=True, c128=c128)
        assert np.max(np.abs(e - e2)) <= 1e-12 * max(np.max(np.abs(e)), pb.info.sigma_c)
        assert np.max(np.abs(g - g2)) <= 1e-12 * max(np.max(np.abs(g)), pb.info.sigma_c)
    finally:
        pb.close()
