"""What the autotuner and the benchmark time includes the call nobody tuned: tile
and grid 0, which the library may answer with kernels that no explicit width names."""
import ast
import os

import numpy as np
import pytest
import torch

import paper_2502_20392_amd.tune as tune
from launch_recorder import record

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class FakePlan:
    made = []

    def __init__(self, offsets, pairs, d, order=12, tol=None, tail_tol=None, grid=0, device=None,
                 tile=0, **kw):
        self.npairs, self.ws, self.key = len(pairs), None, (order, tile, grid)
        FakePlan.made.append(self.key)

    def run(self, pool, out=None):
        FakePlan.last = self.key


@pytest.fixture
def fake(monkeypatch):
    FakePlan.made = []
    monkeypatch.setattr(tune, "RaggedPlan", FakePlan)
    monkeypatch.setattr(tune, "counters", lambda ws: {"status": 0})
    monkeypatch.setattr(tune, "_grid_candidates", lambda order, d: [0, 512])

    def ms(fn, reps):
        fn()  # the untuned call is the fastest
        return 1.0 if FakePlan.last[1:] == (0, 0) else 2.0
    monkeypatch.setattr(tune, "_time", ms)


OFF, PAIRS = np.array([0, 10, 20, 30]), np.array([[0, 1], [1, 2]], np.int32)


def test_ragged_tuner_times_the_untuned_call(fake, tmp_path, monkeypatch):
    monkeypatch.setenv("SIGK_TUNE_CACHE", str(tmp_path / "cache.json"))
    pool = torch.zeros(30, 3, dtype=torch.float64)
    best = tune.tune_ragged(pool, OFF, PAIRS, hint=10)
    assert (best["tile"], best["grid"]) == (0, 0)
    assert {(t["tile"], t["grid"]) for t in best["trials"]} == {(0, 0), (64, 0), (64, 512),
                                                                 (32, 0), (32, 512)}
    n = len(FakePlan.made)
    assert tune.tune_ragged(pool, OFF, PAIRS, hint=10) == best and len(FakePlan.made) == n


@pytest.mark.parametrize("order,d", [(4, 3), (5, 8), (6, 3), (8, 16), (8, 3), (10, 3), (10, 16),
                                     (12, 8), (12, 32), (16, 3), (20, 16)])
def test_a_plans_own_choice_is_one_of_the_class_tuners(order, d):
    """tune_class_tiles times the two explicit widths only: whatever an untuned plan
    launches (kernel and workgroups), one of them launches too."""
    sizes = [(n, length) for n in (3, 60, 136, 256, 400, 800, 2000) for length in (60, 300, 1024)]
    jobs = [dict(call="plan", lens=[length] * (n + 1), pairs=[[i, i + 1] for i in range(n)],
                 order=order, d=d, tile=tile, steps=["run"]) for n, length in sizes
            for tile in (0, 32, 64)]
    res = [r["events"] for r in record(jobs)]
    for k, size in enumerate(sizes):
        assert res[3 * k] in res[3 * k + 1:3 * k + 3], size


def test_benchmark_times_the_untuned_call():
    text = open(os.path.join(ROOT, "bench.py")).read()
    loops = [ast.unparse(n.iter) for n in ast.walk(ast.parse(text))
             if isinstance(n, ast.For) and "tile_options" in ast.unparse(n.iter)]
    assert loops == ["[0] + sk.api.tile_options(order, X.shape[2])"]
