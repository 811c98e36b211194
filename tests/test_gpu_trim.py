"""Kept device memory: trimming gives every kept block back to the device and changes no result, and a handle
whose allocation is replaced or released leaves nothing behind."""
import gc

import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem

pytestmark = pytest.mark.gpu


def free_bytes():
    import torch

    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_trim_and_the_last_handle():
    gc.collect()
    q = W.dense_gaussian_upper(23, 740)
    x = W.random_params(2, 4, 741)
    pb = Problem(q.H, q.f, q.c0)
    N.qq_trim_memory()
    base = free_bytes()
    e0, g0 = pb.evaluate(x, grad=True)  # 0.5 GiB of states
    held = base - free_bytes()
    assert held >= 512 << 20
    assert N.qq_trim_memory() >= 512 << 20 and N.qq_trim_memory() == 0
    assert base - free_bytes() <= 4 << 20
    pb.set_allocation([i % 3 for i in range(23)], 3)
    ep, gp = pb.evaluate(x, grad=True, partitioned=True)
    pb.set_allocation([i % 2 for i in range(23)], 2)  # the first one's memory is reused or given back
    pb.set_allocation([i % 3 for i in range(23)], 3)
    N.qq_trim_memory()
    e1, g1 = pb.evaluate(x, grad=True)
    ep1, gp1 = pb.evaluate(x, grad=True, partitioned=True)
    assert all(np.array_equal(a, b) for a, b in ((e0, e1), (g0, g1), (ep, ep1), (gp, gp1)))
    pb.close()
    N.qq_trim_memory()
    assert free_bytes() >= base - (4 << 20)


def test_unknown_devices_are_refused():
    import torch

    for d in (-1, torch.cuda.device_count()):
        with pytest.raises(N.QQError) as ei:
            N.qq_trim_memory(d)
        assert ei.value.status == N.QQ_E_INVALID
