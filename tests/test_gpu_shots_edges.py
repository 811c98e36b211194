"""Shots at the edges of the search's blocks (4096 entries) and rows (64): one block and less, one block and
more, thousands of blocks, shots at 0, at the largest uniform below 1, around every block end and at
random; in both precisions.  A shot's entry z must satisfy cum(z - 1) <= u total < cum(z) for the state's own
probabilities, up to the rounding of the sums: at most 2^n additions, each of relative error 2^-53 in the
search and in the reference, so 2^n 2^-52 of the total (rounded up to 2^-40 for the small sizes)."""
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


@pytest.mark.parametrize("c128", [False, True])
@pytest.mark.parametrize("n", [1, 5, 6, 7, 12, 13, 18, 20])
def test_shots_at_block_and_row_edges(n, c128):
    q = W.dense_gaussian_upper(n, 80 + n)
    pb = Problem(q.H, q.f, q.c0)
    x = W.random_params(2, 1, 90 + n)[0]
    try:
        psi = pb.state(x, c128=c128).astype(np.complex128)
        cum = np.cumsum(psi.real**2 + psi.imag**2)
        ends = cum[4095::4096] / cum[-1]
        rows = cum[63::64][:500] / cum[-1]
        u = np.concatenate([[0.0, np.nextafter(1.0, 0.0)], ends, rows, np.nextafter(ends, 0.0),
                            np.nextafter(ends, 2.0), np.random.default_rng(n).random(3000)])
        u = u[(u >= 0.0) & (u < 1.0)]
        z = pb.sample(x, u, c128=c128).astype(np.int64)
        assert np.all((z >= 0) & (z < 1 << n))
        slack = max(2.0**-40, 2.0 ** (n - 52)) * cum[-1]
        t = u * cum[-1]
        before = np.where(z > 0, cum[z - 1], 0.0)
        assert np.all(before <= t + slack) and np.all(t < cum[z] + slack)
    finally:
        pb.close()
