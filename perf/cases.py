"""Performance cases: calls of the public Python API over the sizes that it is used at.

listed() and draw() describe cases, prepare() builds what a program holds before the call (the
Problem handles and the angle sets), run() makes the call and exact() gives its results in 64 bits
from plain torch (dense mixer blocks on groups of qubits, the adjoint sweep written out).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem, evaluate_many, evaluate_many_guarded, qaoa_energy


def listed():
    return [
        # The 12-variable case study in complex128: one energy per call on host arrays, the smallest
        # call a program makes (latency and launches only).
        dict(name="energy_n12_c128", kind="evaluate", inst="int", n=12, p=1, batch=1, grad=False, c128=True,
             host=True, part=0),
        # The unit-commitment-shaped batch: 256 angle sets, energies only (an angle scan).
        dict(name="scan_n20_b256", kind="evaluate", inst="uc", n=20, p=4, batch=256, grad=False, c128=False,
             host=False, part=0),
        # A torch training step through the autograd function: a few starts of an odd-sized problem.
        dict(name="train_n17_b3", kind="train", inst="gauss", n=17, p=5, batch=3, c128=False),
        # The benchmark's 3-regular 28-node instance, energy + gradient, with eight of its starts.
        dict(name="grad_n28_b8", kind="evaluate", inst="regular", n=28, p=8, batch=8, grad=True, c128=False,
             host=False, part=0),
        # The uneven batch of integer problems in one call, a quarter of it (energy + gradient).
        dict(name="uneven_128", kind="many", count=128, n_lo=10, n_hi=22, p_lo=1, p_hi=6),
        # The same kind of batch with every gradient held to a tolerance (host arrays).
        dict(name="guarded_96", kind="guarded", count=96, n_lo=10, n_hi=21, p_lo=1, p_hi=4),
        # Double-precision states on host arrays: reference gradients of a mid-sized problem.
        dict(name="grad_n22_c128", kind="evaluate", inst="gauss", n=22, p=4, batch=4, grad=True, c128=True,
             host=True, part=0),
        # The multi-QPU workload's shape (dense real QUBO, four QPUs, p = 2, two angle sets), partitioned
        # phases.
        dict(name="part_n27_b2", kind="evaluate", inst="gauss", n=27, p=2, batch=2, grad=True, c128=False,
             host=False, part=4),
        # Decoding after a search: the ten most probable bitstrings.
        dict(name="topk_n24", kind="topk", inst="regular", n=24, p=3, k=10, c128=False),
        # Shots from the final state.
        dict(name="shots_n25", kind="shots", inst="gauss", n=25, p=3, shots=200000, c128=False),
        # A QUBO seen once (an outer loop that hands over a new one each time): build, evaluate, release.
        dict(name="new_n18", kind="new", inst="int", n=18, p=2, batch=4),
        # The depth-progression search, warm, perturbed and random starts (Adam on the exact gradient).
        dict(name="search_n16", kind="search", inst="regular", n=16, p_max=3, iterations=25, random=6, perturbed=3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evaluate"] * 5 + ["train", "many", "guarded", "topk", "shots", "new", "search"])
    inst = rng.choice(["int", "uc", "gauss", "regular"])

    def size(lo, hi):
        n = rng.randint(lo, hi)
        return min(n + n % 2, hi - hi % 2) if inst == "regular" else n  # odd 3-regular graphs do not exist

    if kind == "evaluate":
        c128, host, grad = rng.random() < 0.4, rng.random() < 0.4, rng.random() < 0.6
        n = size(8, 24 if c128 else 26)
        part = rng.choice([0, 0, 0, 2, 3, 4]) if n >= 12 else 0
        p = rng.randint(1, 8)
        # amplitudes held at most: 2^27 complex64, 2^25 complex128
        batch = _log_int(rng, 1, min(512, 1 << ((25 if c128 else 27) - n)) if n < 25 else 2)
        return dict(kind=kind, inst=inst, n=n, p=p, batch=batch, grad=grad, c128=c128, host=host, part=part)
    if kind == "train":
        return dict(kind=kind, inst=inst, n=size(8, 22), p=rng.randint(1, 8), batch=_log_int(rng, 1, 32),
                    c128=rng.random() < 0.3)
    if kind in ("many", "guarded"):
        hi = rng.randint(14, 22 if kind == "many" else 21)
        return dict(kind=kind, count=_log_int(rng, 4, 128 if kind == "many" else 96), n_lo=rng.randint(8, 12), n_hi=hi,
                    p_lo=1, p_hi=rng.randint(2, 6 if kind == "many" else 4))
    if kind == "topk":
        return dict(kind=kind, inst=inst, n=size(8, 26), p=rng.randint(1, 6), k=rng.randint(1, 16),
                    c128=rng.random() < 0.3)
    if kind == "shots":
        return dict(kind=kind, inst=inst, n=size(8, 26), p=rng.randint(1, 6), shots=_log_int(rng, 1000, 500000),
                    c128=rng.random() < 0.3)
    if kind == "new":
        return dict(kind=kind, inst=inst, n=size(8, 23), p=rng.randint(1, 4), batch=_log_int(rng, 1, 16))
    return dict(kind=kind, inst=inst, n=size(8, 18), p_max=rng.randint(1, 3), iterations=rng.randint(10, 30),
                random=rng.randint(2, 8), perturbed=rng.randint(0, 4))


# ---- inputs -----------------------------------------------------------------------------------

def _instance(inst, n, seed):
    if inst == "int":
        return W.dense_integer_symmetric(n, seed)
    if inst == "uc":
        return W.unit_commitment_shaped(n, seed)
    if inst == "gauss":
        return W.dense_gaussian_upper(n, seed)
    return W.regular_graph_qubo(n, seed)


def _problem(q):
    return Problem(q.H, q.f, q.c0, device=0)


def _allocation(n, parts):
    return W.contiguous_allocation(n, [n // parts + (m < n % parts) for m in range(parts)])


def _batch_sizes(case):
    rng = np.random.default_rng(W.INSTANCE_SEEDS[4])
    return (rng.integers(case["n_lo"], case["n_hi"] + 1, size=case["count"]),
            rng.integers(case["p_lo"], case["p_hi"] + 1, size=case["count"]))


def _batch_inputs(case, seed):
    """(instances, angle sets) of an uneven batch: the sizes are the case's own, the values the seed's."""
    ns, ps = _batch_sizes(case)
    rng = np.random.default_rng(seed)
    seeds = rng.integers(0, 2**31 - 1, size=case["count"])
    qs = [W.dense_integer_symmetric(int(n), int(s)) for n, s in zip(ns, seeds)]
    return qs, [rng.uniform(0.0, np.pi, size=(1, 2 * int(p))) for p in ps]


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("many", "guarded"):
        qs, xs = _batch_inputs(case, seed)
        s["problems"] = [_problem(q) for q in qs]
        s["x"] = [torch.from_numpy(x).cuda() for x in xs] if kind == "many" else xs
        return s
    q = _instance(case["inst"], case["n"], seed)
    if kind == "new":
        s["q"] = q
    else:
        s["pb"] = _problem(q)
    if kind == "search":
        s["points"], s["offsets"] = W.optimizer_draws(case["p_max"], case["random"], case["perturbed"], seed + 1)
        return s
    x = W.random_params(case["p"], case.get("batch", 1), seed + 1)
    if kind == "train":
        x = torch.from_numpy(x).cuda()
    elif kind == "evaluate":
        if case["part"]:
            s["pb"].set_allocation(_allocation(case["n"], case["part"]), case["part"])
        if not case["host"]:
            x = torch.from_numpy(x).cuda()
    elif kind == "shots":
        s["uniforms"] = np.random.default_rng(seed + 2).random(case["shots"])
    s["x"] = x if kind not in ("topk", "shots") else x[0]
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "evaluate":
        r = s["pb"].evaluate(s["x"], grad=case["grad"], c128=case["c128"], partitioned=case["part"] > 0)
        return {"energy": r[0], "grad": r[1]} if case["grad"] else {"energy": r}
    if kind == "train":
        x = s["x"].detach().requires_grad_(True)
        e = qaoa_energy(x, s["pb"], case["c128"])
        e.sum().backward()
        return {"energy": e.detach(), "grad": x.grad}
    if kind == "many":
        e, g = evaluate_many(s["problems"], s["x"], grad=True)
        return {"energy": torch.cat(e), "grad": torch.cat([v.reshape(-1) for v in g])}
    if kind == "guarded":
        e, g, up, err = evaluate_many_guarded(s["problems"], s["x"], tol=1e-5)
        return {"energy": np.concatenate(e), "grad": np.concatenate([v.reshape(-1) for v in g]),
                "c128": np.concatenate(up), "bound": np.concatenate(err)}
    if kind == "topk":
        idx, prob, cost = s["pb"].topk(s["x"], k=case["k"], c128=case["c128"])
        return {"index": idx.astype(np.int64), "prob": prob, "cost": cost}
    if kind == "shots":
        return {"index": s["pb"].sample(s["x"], s["uniforms"], c128=case["c128"]).view(np.int64)}
    if kind == "new":
        pb = _problem(s["q"])
        e, g = pb.evaluate(s["x"], grad=True)
        info = pb.info
        r = {"energy": e, "grad": g, "argmin": info.argmin_index, "cmin": info.cmin, "cmax": info.cmax}
        pb.close()
        return r
    r = s["pb"].optimize(case["p_max"], case["iterations"], s["points"], s["offsets"], random_starts=case["random"],
                         perturbed_starts=case["perturbed"])
    return {k: r[k] for k in ("best_depth", "best_start", "best_energy", "steps", "evaluations", "depth_params",
                              "depth_energy", "start_energy")}


# ---- least work -------------------------------------------------------------------------------

def _state_work(n, p, batch, grad, c128):
    """Bytes and operations of `batch` state evaluations.  Every layer mixes every amplitude with every
    other, so a state is read and written once per layer (psi forwards; psi and lambda backwards); a
    mixer takes 4 operations per amplitude, qubit and state, <lambda|X|psi> another 4."""
    dim = float(1 << n)
    es = 16 if c128 else 8
    return {"bytes": batch * dim * es * 2 * p * (3 if grad else 1),
            "flops": batch * dim * n * p * 4 * (4 if grad else 1)}


def work(case):
    kind = case["kind"]
    if kind in ("many", "guarded"):
        ws = [_state_work(int(n), int(p), 1, True, False) for n, p in zip(*_batch_sizes(case))]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    if kind == "search":
        total = {"bytes": 0.0, "flops": 0.0}
        for p in range(1, case["p_max"] + 1):
            starts = case["random"] + (1 + case["perturbed"] if p > 1 else 0)
            for w in (_state_work(case["n"], p, starts * case["iterations"], True, False),
                      _state_work(case["n"], p, starts, False, False)):
                total = {k: total[k] + w[k] for k in total}
        return total
    w = _state_work(case["n"], case["p"], case.get("batch", 1), kind in ("train", "new") or case.get("grad", False),
                    case.get("c128", False))
    if kind == "new":  # the cost diagonal, written once, one term per coupling
        w["bytes"] += float(1 << case["n"]) * 2
        w["flops"] += float(1 << case["n"]) * 2
    if kind == "shots":
        w["bytes"] += 16.0 * case["shots"]
    return w


# ---- results in 64 bits -----------------------------------------------------------------------

def _cost(q):
    """C(z) for every z, on the GPU in float64."""
    n = q.n
    B = torch.from_numpy(np.triu(q.H, 1) + np.tril(q.H, -1).T).cuda()
    ell = torch.from_numpy(np.asarray(q.f) + np.diag(q.H)).cuda()
    z = torch.arange(1 << n, device="cuda")
    bits = [((z >> i) & 1).to(torch.bool) for i in range(n)]
    c = torch.full((1 << n,), float(q.c0), dtype=torch.float64, device="cuda")
    for i in range(n):
        row = torch.zeros_like(c)
        for j in range(i + 1, n):
            if q.H[i, j] or q.H[j, i]:
                row += B[i, j] * bits[j]
        c += torch.where(bits[i], row + ell[i], torch.zeros_like(row))
    return c


def _groups(n):
    g = -(-n // 7)
    return [n // g + (i < n % g) for i in range(g)]


def _rx(k, beta):
    """exp(-i beta X) on each of k qubits, as one 2^k x 2^k matrix."""
    one = torch.tensor([[math.cos(beta), -1j * math.sin(beta)], [-1j * math.sin(beta), math.cos(beta)]],
                       dtype=torch.complex128, device="cuda")
    m = torch.ones(1, 1, dtype=torch.complex128, device="cuda")
    for _ in range(k):
        m = torch.kron(m, one)
    return m


def _sum_x(k):
    """sum of X_q over k qubits."""
    d = 1 << k
    m = torch.zeros(d, d, dtype=torch.complex128, device="cuda")
    r = torch.arange(d, device="cuda")
    for q in range(k):
        m[r, r ^ (1 << q)] = 1
    return m


def _turn(m, v):
    """m on the highest group of qubits, which then becomes the lowest."""
    return (m @ v.view(m.shape[0], -1)).t().contiguous().view(-1)


def _state(c, n, x):
    psi = torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.complex128, device="cuda")
    for gamma, beta in zip(x[0::2], x[1::2]):
        psi = psi * torch.exp(-1j * gamma * c)
        for k in _groups(n):
            psi = _turn(_rx(k, beta), psi)
    return psi


def _evaluate(c, n, x, grad):
    """(energy, gradient or None) at the angles x (host floats)."""
    psi = _state(c, n, x)
    e = float((psi.abs().square() * c).sum())
    if not grad:
        return e, None
    mean = float(c.mean())  # <psi|psi> is constant, so the seed may be centred
    lam = (c - mean) * psi
    g = np.zeros(len(x))
    for k in range(len(x) // 2 - 1, -1, -1):
        gamma, beta = x[2 * k], x[2 * k + 1]
        for m in _groups(n):
            u = _rx(m, -beta)
            xs = (_sum_x(m) @ psi.view(1 << m, -1)).view(-1)
            g[2 * k + 1] += 2.0 * float(torch.vdot(lam, xs).imag)
            del xs
            psi, lam = _turn(u, psi), _turn(u, lam)
        g[2 * k] = 2.0 * float(((lam.conj() * psi).imag * (c - mean)).sum())
        ph = torch.exp(1j * gamma * c)
        psi, lam = psi * ph, lam * ph
    return e, g


def _evaluate_all(c, n, x, grad=True):
    r = [_evaluate(c, n, [float(v) for v in row], grad) for row in x]
    return np.array([v[0] for v in r]), np.array([v[1] for v in r]) if grad else None


def _lift(x, p):
    """Linear interpolation of a depth-p vector onto depth p + 1 (zero beyond both ends)."""
    y = np.zeros(2 * (p + 1))
    for c in range(2):
        s = np.concatenate([[0.0], x[c::2], [0.0]])
        for i in range(1, p + 2):
            y[2 * (i - 1) + c] = ((i - 1) / p) * s[i - 1] + ((p - i + 1) / p) * s[i]
    return y


def _search(c, n, case, points, offsets):
    """The depth progression with Adam on the exact gradient, in 64 bits."""
    pmax, R, P = case["p_max"], case["random"], case["perturbed"]
    a = b = 0
    prev, depth_x, depth_e, start_e = None, np.zeros((pmax, 2 * pmax)), [], []
    for p in range(1, pmax + 1):
        xs = []
        if p > 1:
            warm = _lift(prev, p - 1)
            xs = [warm] + [warm + offsets[b + 2 * p * j:b + 2 * p * (j + 1)] for j in range(P)]
            b += 2 * p * P
        xs += [points[a + 2 * p * j:a + 2 * p * (j + 1)] for j in range(R)]
        a += 2 * p * R
        x = np.array(xs)
        m, v = np.zeros_like(x), np.zeros_like(x)
        for t in range(1, case["iterations"] + 1):
            g = _evaluate_all(c, n, x)[1]
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            x = x - 0.01 * (m / (1 - 0.9**t)) / (np.sqrt(v / (1 - 0.999**t)) + 1e-8)
        e = _evaluate_all(c, n, x, False)[0]
        best = int(np.argmin(e))
        prev = x[best]
        depth_x[p - 1, :2 * p] = prev
        depth_e.append(e[best])
        start_e.append(e)
    return {"best_depth": None, "best_start": None, "best_energy": min(depth_e), "steps": None, "evaluations": None,
            "depth_params": depth_x, "depth_energy": np.array(depth_e), "start_energy": start_e}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("many", "guarded"):
        qs, xs = _batch_inputs(case, seed)
        r = [_evaluate_all(_cost(q), q.n, x) for q, x in zip(qs, xs)]
        out = {"energy": np.concatenate([v[0] for v in r]), "grad": np.concatenate([v[1].reshape(-1) for v in r])}
        return out if kind == "many" else dict(out, c128=None, bound=None)
    if kind == "shots":
        return None  # whole numbers only
    n = case["n"]
    q = _instance(case["inst"], n, seed)
    c = _cost(q)
    if kind == "search":
        points, offsets = W.optimizer_draws(case["p_max"], case["random"], case["perturbed"], seed + 1)
        return _search(c, n, case, points, offsets)
    x = W.random_params(case["p"], case.get("batch", 1), seed + 1)
    if kind == "topk":
        prob = _state(c, n, [float(v) for v in x[0]]).abs().square()
        return {"index": None, "prob": torch.topk(prob, case["k"]).values, "cost": None}
    e, g = _evaluate_all(c, n, x, kind in ("train", "new") or case["grad"])
    out = {"energy": e, "grad": g}
    if kind == "new":
        out.update(argmin=None, cmin=float(c.min()), cmax=float(c.max()))
    return {k: v for k, v in out.items() if v is not None or k != "grad"}
