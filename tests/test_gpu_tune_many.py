"""The many-problem tuner and its cache: what it returns leaves a small batch's items to the launch (tuned is
then the default, bit for bit, though every limit that it may return is above the items' size), entries of
other kernel revisions are tuned again, and a read-only file that holds one stays usable."""
import json
import os

import numpy as np
import pytest

from paper_2606_26297_amd import native as N
from paper_2606_26297_amd import workloads as W
from paper_2606_26297_amd.qaoa import Problem, evaluate_many

pytestmark = pytest.mark.gpu

GRAD = N.QQ_ENERGY | N.QQ_GRAD


@pytest.fixture(scope="module")
def batch():
    N.lib()
    items = [(W.dense_integer_symmetric(n, 70 + n), W.random_params(1 + n % 3, 1, 80 + n)) for n in (11, 13, 14, 16)]
    pbs = [Problem(i.H, i.f, i.c0) for i, _ in items]
    yield pbs, [x for _, x in items]
    for pb in pbs:
        pb.close()


def tune(batch, path):
    pbs, xs = batch
    return N.qq_autotune_many([pb.handle for pb in pbs], [x.shape[1] // 2 for x in xs], [1] * len(pbs), GRAD, path)


def test_limits_leave_small_batches_alone(batch):
    pbs, xs = batch
    opt, _ = tune(batch, None)
    e0, g0 = evaluate_many(pbs, xs, grad=True)
    for o in (opt, dict(tiles_per_chunk=4), dict(tiles_per_chunk=64)):
        e, g = evaluate_many(pbs, xs, grad=True, options=o)
        assert all(np.array_equal(a, b) for a, b in zip(e + g, e0 + g0)), o


def test_entries_of_other_revisions_are_tuned_again(batch, tmp_path):
    path = str(tmp_path / "many.jsonl")
    tune(batch, path)
    (line,) = open(path).read().splitlines()
    entry = json.loads(line)
    old = dict(entry, tiles_per_chunk=63, ms=1e-9)
    del old["rev"]  # as entries were before they carried one
    other = dict(old, rev=entry["rev"] + 1)
    keys = list(entry)

    def dump(e):
        return json.dumps({k: e[k] for k in keys if k in e}, separators=(",", ":"))

    with open(path, "w") as f:
        f.write(dump(old) + "\n" + dump(other) + "\n")
    opt, ms = tune(batch, path)
    assert opt["tiles_per_chunk"] != 63 and ms > 1e-6
    assert len(open(path).readlines()) == 3
    opt2, ms2 = tune(batch, path)  # now from the cache
    assert opt2 == opt and ms2 == pytest.approx(ms, rel=1e-3) and len(open(path).readlines()) == 3
    with open(path, "w") as f:
        f.write(dump(old) + "\n")
    os.chmod(path, 0o444)
    if os.access(path, os.W_OK):
        pytest.skip("this user writes to read-only files")
    opt3, _ = tune(batch, path)
    assert opt3["tiles_per_chunk"] != 63
