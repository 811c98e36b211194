"""Many problems in one call: what a problem returns does not depend on what else is in the call, nor on how
many workgroups run, bit for bit, in both precisions (the launch's items grow with the batch; the partial
sums do not).  Sizes: one tile, the smallest multi-pass problem, every unit of partial sums up to n = 23, three
sets (n = 21), every diagonal type; a long chain of outputs (p = 64)."""
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


def items(spec, seed):
    out = []
    for k, (kind, n, p, B) in enumerate(spec):
        if kind == "int16":
            q = W.dense_integer_symmetric(n, seed + k)
        elif kind == "int32":
            q = W.dense_integer_symmetric(n, seed + k, -100000, 100000)
        else:
            q = W.dense_gaussian_upper(n, seed + k)
        x = W.random_params(p, B, seed + 100 + k)
        if kind == "int32":
            x[:, 0::2] /= 1000.0
        out.append((Problem(q.H, q.f, q.c0), x))
    return out


@pytest.mark.parametrize("c128", [False, True])
def test_results_do_not_depend_on_the_batch(c128):
    probe = items([("int16", 10, 2, 2), ("int16", 13, 3, 2), ("int16", 17, 2, 1), ("int16", 19, 1, 1),
                   ("int32", 20, 2, 1), ("int16", 21, 2, 1), ("real", 22, 1, 1), ("int16", 23, 1, 1)], 900)
    fill = items([("int16", 16 + k % 5, 1 + k % 4, 2) for k in range(40)] + [("real", 20, 3, 3)] * 3, 950)
    try:
        def run(which, options=None):
            e, g = evaluate_many([pb for pb, _ in which], [x for _, x in which], grad=True, options=options, c128=c128)
            return [(np.copy(a), np.copy(b)) for a, b in zip(e, g)]

        alone = [run([it])[0] for it in probe]
        for got in (run(probe), run(probe + fill), run(probe + fill, dict(max_workgroups=64))):
            for (pb, _), (ea, ga), (e, g) in zip(probe, alone, got):
                assert np.array_equal(e, ea) and np.array_equal(g, ga), pb.n
    finally:
        for pb, _ in probe + fill:
            pb.close()


@pytest.mark.parametrize("n,c128", [(11, False), (11, True), (13, False), (13, True), (21, True)])
def test_long_chains_are_summed_whole(n, c128):
    """p = 64: 129 outputs, the most slots a plan has.  Complex128 against the per-problem call (sums in another
    order: 1e-11 of max(|value|, sigma_C)), complex64 energies to 1e-5 of the same."""
    (pb, x), = items([("int16", n, 64, 1)], 990 + n)
    try:
        x = x / 8.0
        (e,), (g,) = evaluate_many([pb], [x], grad=True, c128=c128)
        er, gr = pb.evaluate(x, grad=True, c128=c128)
        s = pb.info.sigma_c
        assert np.abs(e - er)[0] <= (1e-11 if c128 else 1e-5) * max(abs(er[0]), s)
        b = np.max(np.abs(gr))
        lim = 1e-11 * max(b, s) if c128 else 2 * (N.QQ_GUARD_REL * b + N.QQ_GUARD_K * s * s * 2.0**-24 * 2.0**(-0.5 * n))
        assert np.max(np.abs(g - gr)) <= lim
    finally:
        pb.close()
