"""Held variables together with the convergence test, one restart a tile: step counts,
retired states and traces against a replay one step a launch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from gpu_util import log  # noqa: E402


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("case", ["sat", "weighted", "types", "large", "loose", "long"])
def test_retired_restarts_equal_a_replay(case, bits):
    log(f"case {case} bits {bits}")
    if case == "types":
        inst = synth.mixed_small(n=61, seed=8, kmax=8, count=90)
    elif case == "long":
        inst = synth.mixed_small(n=90, seed=8, kmax=40, count=60)
    else:  # large, loose: codes do not fit LDS
        n = 4000 if case in ("large", "loose") else 300
        inst = synth.random_ksat(n, 3 * n, 3, 5)
    if case == "weighted":
        inst.weight = np.random.default_rng(5).uniform(0.25, 4.0, inst.m).astype(np.float32)
    R, steps, tol = 37, 60, 0.11 if case == "loose" else 1e-2
    prob = pcls.Problem.from_instance(inst, accumulator_bits=bits)
    prob.set_launch(1, 0)
    fixed = torch.zeros(inst.n, dtype=torch.int8, device=prob.device)
    fixed[::3], fixed[1::7] = -1, 1
    X = prob.new_state(R)
    prob.init_restarts(X, R, 4)
    Y = X.clone()
    trace, iters = prob.step_ex(X, R, 0.1, steps, trace=True, fixed=fixed, tol=tol, want_iters=True)

    held = fixed != 0
    Y[held] = fixed[held].float()[:, None]
    want = torch.full((R,), steps, dtype=torch.int32, device=prob.device)
    left = torch.ones(R, dtype=torch.bool, device=prob.device)
    end, last = Y.clone(), None
    for s in range(steps):
        before = Y.clone()
        tr, _ = prob.step_ex(Y, R, 0.1, 1, trace=True, fixed=fixed)
        row = tr[0] if s == 0 else torch.where(left, tr[0], last)  # a retired restart repeats its last objective
        assert torch.equal(trace[s], row), s
        last = row
        end[:, :R][:, left] = Y[:, :R][:, left]
        done = left & ((Y - before)[:, :R].abs().amax(0) < tol)
        want[done] = s + 1
        left &= ~done
    assert case == "large" or int((want < steps).sum()) > 0  # some retire early (none of the large ones)
    assert torch.equal(iters.to(torch.int32)[:R], want)
    assert torch.equal(X[:, :R], end[:, :R])
