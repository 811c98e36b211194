"""Complex128 evaluations (the specialised tile passes for n > 12, the one-tile kernel for n <= 12, and
the persistent launch over both) against the FP64 oracle: energies, gradients and states at the edges of
the set geometry (n = 13: a single qubit above the tile; 20: one full high set; 21: three sets, one with
a single active qubit), at odd and even depths, for every diagonal type and for large phase angles.

Tolerance.  Each amplitude takes n p rotations, each with a relative rounding of 2^-52 in its two products
and sum, and p phases whose argument theta = gamma C carries a rounding of 2^-53 |theta| and whose sine and
cosine are good to 2^-52; with the cost sums (at most n^2 terms of the size of C's) the state is within
d = p (3 n + 4 + n |gamma| Cmax) 2^-52 of the exact one, on either side.  Then |dE| <= 2 Cmax d, a
beta-derivative 2 Im <lambda|sum X|psi>, with |lambda| <= Cmax and n terms of X, is within 2 n Cmax (2 d), and a
gamma-derivative 2 Im <lambda|C|psi> within 2 Cmax^2 (2 d)."""
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


def state_bound(n, x, d):
    p = x.size // 2
    return 2 * p * (3 * n + 4 + n * np.max(np.abs(x[0::2])) * np.max(np.abs(d))) * 2.0**-52


@pytest.mark.parametrize("kind", ["int16", "int32", "real"])
@pytest.mark.parametrize("n,p,scale", [(1, 1, 1.0), (3, 2, 1.0), (8, 3, 1.0), (11, 4, 20.0), (12, 1, 1.0), (12, 5, 1.0),
                                       (13, 2, 1.0), (16, 3, 20.0), (17, 1, 1.0), (20, 2, 1.0), (21, 3, 1.0)])
def test_c128_matches_the_oracle(kind, n, p, scale):
    q = instance(kind, n, 40 + n)
    pb = Problem(q.H, q.f, q.c0)
    x = scale * W.random_params(p, 2, 50 + n)
    x[:, 0::2] /= 1000.0 if kind == "int32" else 1.0
    try:
        e, g = pb.evaluate(x, grad=True, c128=True)
        e1 = pb.evaluate(x, c128=True)
        em, gm = evaluate_many([pb], [x], grad=True, c128=True)
        d = O.cost_diagonal(q.H, q.f, q.c0)
        cmax = np.max(np.abs(d))
        psi = pb.state(x[0], c128=True)
        assert np.linalg.norm(psi - O.qaoa_state(d, x[0])) <= state_bound(n, x[0], d)
        for b in range(2):
            er, gr = O.gradient(d, x[b])
            s = state_bound(n, x[b], d)
            for v in (e[b], e1[b], em[0][b]):
                assert abs(v - er) <= 2 * cmax * s, (v, er)
            for v in (g[b], gm[0][b]):
                assert np.max(np.abs(v - gr)[1::2]) <= 4 * n * cmax * s, (v, gr)
                assert np.max(np.abs(v - gr)[0::2]) <= 4 * float(cmax) ** 2 * s, (v, gr)
    finally:
        pb.close()


@pytest.mark.parametrize("kind", ["int16", "real"])
@pytest.mark.parametrize("n,p,qpus", [(9, 2, 2), (13, 3, 3), (17, 2, 4), (21, 2, 5)])
def test_c128_partitioned_matches_the_oracle(kind, n, p, qpus):
    """Partitioned phases (interleaved variables, so that every run of qubits spans several QPUs): the same
    unitary, within the same bound (the two forms' values carry the roundings of one each)."""
    q = instance(kind, n, 60 + n)
    pb = Problem(q.H, q.f, q.c0)
    x = W.random_params(p, 2, 70 + n)
    try:
        pb.set_allocation([i % qpus for i in range(n)], qpus)
        e, g = pb.evaluate(x, grad=True, c128=True, partitioned=True)
        d = O.cost_diagonal(q.H, q.f, q.c0)
        cmax = float(np.max(np.abs(d)))
        for b in range(2):
            er, gr = O.gradient(d, x[b])
            s = 2 * state_bound(n, x[b], d)
            assert abs(e[b] - er) <= 2 * cmax * s
            assert np.max(np.abs(g[b] - gr)[1::2]) <= 4 * n * cmax * s
            assert np.max(np.abs(g[b] - gr)[0::2]) <= 4 * cmax**2 * s
    finally:
        pb.close()
