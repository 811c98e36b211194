"""Evaluations recorded into a caller's own graph (device parameters, device results, a workspace or the fixed
scratch array): every replay, with new parameters and eager work between the replays, returns what the eager
call does, bit for bit."""
import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem

pytestmark = pytest.mark.gpu

DEV = N.QQ_ENERGY | N.QQ_GRAD | N.QQ_PARAMS_ON_DEVICE | N.QQ_OUT_ON_DEVICE


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("n,c128", [(10, False), (10, True), (15, False), (15, True)])
def test_captured_evaluations(n, c128, static):
    import torch

    q = W.dense_integer_symmetric(n, 500 + n)
    pb = Problem(q.H, q.f, q.c0)
    flags = DEV | (N.QQ_C128 if c128 else 0)
    p, B = 2, 3
    try:
        x = torch.zeros(B, 2 * p, dtype=torch.float64, device="cuda")
        block = torch.zeros(B + B * 2 * p, dtype=torch.float64, device="cuda")
        e, g = block[:B], block[B:]
        ws = torch.empty(pb.workspace_size(p, B, flags), dtype=torch.uint8, device="cuda")

        def call():
            s = torch.cuda.current_stream()
            if static:
                N.qq_evaluate_static(pb.handle, p, B, x, flags, s, e, g)
            else:
                N.qq_evaluate(pb.handle, p, B, x, flags, ws, ws.numel(), s, e, g)

        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call()
        for k in range(4):
            host = W.random_params(p, B, 510 + k)
            x.copy_(torch.from_numpy(host))
            block.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            got = block.cpu().numpy().copy()
            call()
            torch.cuda.synchronize()
            assert np.all(np.isfinite(got)) and np.array_equal(got, block.cpu().numpy()), k
            pb.evaluate(host, grad=True, c128=c128)  # eager work on the library's own memory
    finally:
        pb.close()
