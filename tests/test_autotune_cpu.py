"""The autotuner's search and cache without a GPU (timings are given by a
table): what it tries at sizes of the pairwise kernel, what it keeps, and that
parameters measured on other kernels are not handed out."""
import json

import numpy as np
import pytest

from paper_1807_08116_amd import autotune
from paper_1807_08116_amd import sphgrav as sg


def tune(monkeypatch, tmp_path, precision, n, cost):
    tried = []

    def timing(st, p, params, reps=2):
        tried.append(dict(params))
        return cost(params)

    monkeypatch.setattr(autotune, "time_gravity", timing)
    path = str(tmp_path / "cache.json")
    best = autotune.tune_gravity(dict(x=np.zeros(n)), precision, path=path)
    assert autotune.lookup("grav", precision, n, path) == best
    return best, tried


@pytest.mark.parametrize("precision", [sg.SG_FP64, sg.SG_FP32C])
def test_pairwise_sizes(monkeypatch, tmp_path, precision):
    best, tried = tune(monkeypatch, tmp_path, precision, 20000,
                       lambda c: 3.0 if c["grav_variant"] else 2.0)
    assert best == autotune.AUTO
    # the pairwise kernel has no tile; every one-sided kernel has its turn
    assert not [c for c in tried if c["grav_variant"] == 0 and c["grav_tile"]]
    assert {c["grav_variant"] for c in tried} == \
        ({0, 1, 2, 3, 4} if precision == sg.SG_FP64 else {0, 1})
    # a one-sided kernel that wins gets its tile
    best, tried = tune(monkeypatch, tmp_path, precision, 20000,
                       lambda c: (1.0 if c["grav_tile"] == 512 else 1.5) if c["grav_variant"] == 1 else 2.0)
    assert best == dict(autotune.AUTO, grav_variant=1, grav_tile=512)


def test_small_sizes(monkeypatch, tmp_path):
    best, tried = tune(monkeypatch, tmp_path, sg.SG_FP32C, 12287,
                       lambda c: 1.0 if c["grav_tile"] == 128 and c["grav_split"] == 4 else 2.0 - 0.1 * (c["grav_tile"] == 128))
    assert best == dict(autotune.AUTO, grav_tile=128, grav_split=4)


def test_noise_is_not_kept(monkeypatch, tmp_path):
    k = iter(range(1000))
    best, _ = tune(monkeypatch, tmp_path, sg.SG_FP64, 2048, lambda c: 2.0 - 1e-4 * next(k))
    assert best == autotune.AUTO


def test_entries_of_other_kernels_are_not_looked_up(tmp_path):
    path = str(tmp_path / "cache.json")
    entry = dict(best=dict(autotune.AUTO, grav_variant=3), ms=1.0)
    with open(path, "w") as f:
        json.dump({"grav:0:2097152": entry}, f)
    assert autotune.lookup("grav", sg.SG_FP64, 2097152, path) is None


def test_shipped_cache_takes_the_pairwise_kernel():
    for p in (sg.SG_FP64, sg.SG_FP32C):
        best = autotune.lookup("grav", p, 2097152)
        assert best is None or best["grav_variant"] == 0
