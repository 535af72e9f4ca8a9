"""For one launch shape the objectives are the same bits however the steps are split
into launches, and in an evaluation: also where launches of 8 steps or more keep the
codes in LDS and shorter ones and evaluations do not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from paper_2606_06656_amd.batch import Batch  # noqa: E402
from gpu_util import log  # noqa: E402


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("case", ["sat65", "sat1025", "sat2100", "mixed", "types"])
@pytest.mark.parametrize("T", [1, 2])
def test_trace_bits(case, weighted, bits, T):
    log(f"case {case} weighted {weighted} bits {bits} T {T}")
    if case.startswith("sat"):
        m = int(case[3:])
        inst = synth.random_ksat(m // 4, m, 3, m)
    else:
        inst = synth.c2_mixed(3, 401, 1203, 121, 41) if case == "mixed" else synth.mixed_small(61, 8, 8, 700)
    if weighted:
        inst.weight = np.random.default_rng(5).uniform(0.25, 4.0, inst.m).astype(np.float32)
    R, steps = 37, 12
    prob = pcls.Problem.from_instance(inst, accumulator_bits=bits)
    prob.set_launch(T, 0)
    X = prob.new_state(R)
    prob.init_restarts(X, R, 4)
    Y = X.clone()
    first, _ = prob.evaluate(X, R)
    tr = prob.step(X, R, 0.1, steps, trace=True)
    parts = torch.cat([prob.step(Y, R, 0.1, 4, trace=True) for _ in range(steps // 4)])
    assert torch.equal(tr[0], first)
    assert torch.equal(tr, parts)
    assert torch.equal(X[:, :R], Y[:, :R])


@pytest.mark.parametrize("case", ["sat2100", "mixed"])
def test_batch_of_one_restart_tiles(case):
    """A batch whose LDS budget leaves one restart a tile: the bits of single launches."""
    log(f"case batch {case}")
    inst = synth.random_ksat(525, 2100, 3, 1) if case == "sat2100" else synth.c2_mixed(3, 401, 1203, 121, 41)
    R, steps = 37, 12
    prob = pcls.Problem.from_instance(inst, accumulator_bits=32)
    prob.set_launch(1, 0)
    X = prob.new_state(R)
    prob.init_restarts(X, R, 4)
    Y, tb = X.clone(), torch.empty((steps, R), device=X.device)
    tr = prob.step(X, R, 0.1, steps, trace=True)
    b = Batch([prob], [R], [Y], [tb])
    b.set_config(256, 6000, 0, 32)
    assert b.config()["n_items"] == R
    b.step(0.1, steps)
    assert torch.equal(tb, tr) and torch.equal(X[:, :R], Y[:, :R])
    b.close()
