"""The single-problem autotuner probes what long launches run, and drops winners of
other kernels."""
import json
import os

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import autotune, pcls, synth  # noqa: E402
from gpu_util import log  # noqa: E402


def step_ms(prob, R, steps=200):
    return min(autotune._time_steps(prob, R, 0.1, steps) for _ in range(3))


@pytest.mark.parametrize("n,R", [(50, 64), (200, 64), (1000, 320)])
def test_short_constraints_are_probed_as_they_run(n, R):
    log(f"case tune n {n} R {R}")
    inst = synth.random_ksat(n, int(4.2 * n), 3, n)
    rec = autotune.tune_problem(inst, R)
    assert rec["probe_steps"] >= 8  # launches that may keep the codes on chip
    base = pcls.Problem.from_instance(inst)
    tuned = autotune.tuned_problem(inst, R, rec)
    # the default launch is among the candidates; 10% for the clock
    assert step_ms(tuned, R) <= 1.1 * step_ms(base, R)


def test_long_constraints_keep_the_asked_steps():
    log("case tune long")
    inst = synth.mixed_small(n=100, seed=3, kmax=16, count=60)
    assert autotune.tune_problem(inst, 32, probe_steps=2)["probe_steps"] == 2


def test_winner_of_other_kernels_is_not_reused(tmp_path, monkeypatch):
    log("case tune revision")
    inst = synth.random_ksat(60, 250, 3, 1)
    cache = os.path.join(str(tmp_path), "tune.json")
    assert not autotune.tune_problem(inst, 64, cache_path=cache)["cached"]
    assert autotune.tune_problem(inst, 64, cache_path=cache)["cached"]
    monkeypatch.setattr(pcls, "KERNEL_REVISION", "other")
    assert not autotune.tune_problem(inst, 64, cache_path=cache)["cached"]
    with open(cache) as f:
        assert len(json.load(f)) == 2
