"""Device results that share memory with the device parameters, or energies with gradients, are what
separate arrays receive, bit for bit: one-pass evaluations (n <= 12) read a set's parameters until its last
layer, while other sets' results are already written."""
import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem

pytestmark = pytest.mark.gpu

DEV = N.QQ_ENERGY | N.QQ_GRAD | N.QQ_PARAMS_ON_DEVICE | N.QQ_OUT_ON_DEVICE


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("c128", [False, True])
@pytest.mark.parametrize("n,p,B", [(5, 2, 1), (12, 3, 1), (12, 3, 700), (14, 2, 5)])
def test_results_may_overlap_the_parameters(n, p, B, c128, static):
    import torch

    q = W.dense_gaussian_upper(n, 400 + n)
    pb = Problem(q.H, q.f, q.c0)
    flags = DEV | (N.QQ_C128 if c128 else 0)
    host = W.random_params(p, B, 410 + n)
    try:
        ws = torch.empty(pb.workspace_size(p, B, flags), dtype=torch.uint8, device="cuda")

        def run(x, e, g):
            s = torch.cuda.current_stream()
            if static:
                N.qq_evaluate_static(pb.handle, p, B, x, flags, s, e, g)
            else:
                N.qq_evaluate(pb.handle, p, B, x, flags, ws, ws.numel(), s, e, g)
            torch.cuda.synchronize()
            return e.cpu().numpy().copy(), g.cpu().numpy().reshape(B, 2 * p).copy()

        new = lambda m: torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")  # noqa: E731
        e0, g0 = run(torch.from_numpy(host).cuda(), new(B), new(B * 2 * p))
        assert np.all(np.isfinite(e0)) and np.all(np.isfinite(g0))
        for case in ("energies", "gradients", "both"):
            x = torch.from_numpy(host).cuda()
            flat = x.view(-1)
            if case == "energies":  # into the parameters' first entries
                e, g = run(x, flat[:B], new(B * 2 * p))
            elif case == "gradients":  # in place
                e, g = run(x, new(B), flat)
            else:  # one block holding energies, then gradients; the parameters behind the first energies
                block = new(B + 2 * B * 2 * p)
                x = block[1:1 + B * 2 * p]
                x.copy_(torch.from_numpy(host.reshape(-1)))
                e, g = run(x, block[:B], block[B:B + B * 2 * p])
            assert np.array_equal(e, e0) and np.array_equal(g, g0), case
    finally:
        pb.close()
