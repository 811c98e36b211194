"""Device memory kept between calls (qq_pool): calls of different sizes on several threads and streams
return what they return alone, bit for bit, and the kept memory stays within its bound."""
import threading

import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem

pytestmark = pytest.mark.gpu

POOL_KEEP = 4 << 30


@pytest.fixture(scope="module", autouse=True)
def _lib():
    N.lib()
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"


def test_threads_and_streams_share_the_pool():
    import torch

    sizes = [(9, 2, 3), (13, 1, 5), (17, 2, 2), (20, 1, 2)]
    cases = []
    for k, (n, p, B) in enumerate(sizes):
        q = W.dense_gaussian_upper(n, 700 + k)
        x = W.random_params(p, B, 710 + k)
        pb = Problem(q.H, q.f, q.c0)
        cases.append((q, x, pb, pb.evaluate(x, grad=True), pb.topk(x[0], k=4)))
    errors = []

    def work(seed):
        try:
            rng = np.random.default_rng(seed)
            s = torch.cuda.Stream()
            for _ in range(12):
                q, x, pb, (e, g), top = cases[rng.integers(len(cases))]
                kind = rng.integers(4)
                if kind == 0:  # own stream, host buffers, memory of the call's own
                    e2, g2 = np.empty_like(e), np.empty_like(g)
                    N.qq_evaluate(pb.handle, x.shape[1] // 2, x.shape[0], x, N.QQ_ENERGY | N.QQ_GRAD, None, 0, s, e2,
                                  g2)
                elif kind == 1:
                    e2, g2 = pb.evaluate(x, grad=True)
                elif kind == 2:  # a handle built and released in between
                    pb2 = Problem(q.H, q.f, q.c0)
                    e2, g2 = pb2.evaluate(x, grad=True)
                    pb2.close()
                else:
                    t2 = pb.topk(x[0], k=4)
                    assert all(np.array_equal(a, b) for a, b in zip(t2, top))
                    continue
                assert np.array_equal(e, e2) and np.array_equal(g, g2), (pb.n, kind)
        except Exception as exc:  # noqa: BLE001
            errors.append(exc)

    threads = [threading.Thread(target=work, args=(s,)) for s in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for c in cases:
        c[2].close()
    assert not errors, errors


def test_kept_memory_is_bounded():
    import torch

    torch.cuda.synchronize()
    q = W.dense_gaussian_upper(24, 720)
    pb = Problem(q.H, q.f, q.c0)
    before = torch.cuda.mem_get_info()[0]
    for B in (1, 2, 3, 5, 8, 13, 21):  # states of 0.25 to 5.25 GiB with lambda
        pb.evaluate(W.random_params(1, B, 721 + B), grad=True)
    held = before - torch.cuda.mem_get_info()[0]
    pb.close()
    assert held <= POOL_KEEP, held
