"""Small problems with one restart a tile keep their literal codes in LDS for
launches of 8 steps or more.  Gradients are exact fixed-point sums, so such a
launch takes the same iterates, bit for bit, as launches too short for it; the
objectives agree to float32 rounding of their chunks' sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from gpu_util import log  # noqa: E402


def instance(case):
    if case == "one":
        return synth.random_ksat(3, 1, 3, 1)
    if case.startswith("sat"):  # constraints around whole chunks and rounds of chunks
        m = int(case[3:])
        return synth.random_ksat(max(20, m // 4), m, 3, m)
    if case == "none":
        return synth.Instance(7, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.int8), np.zeros(0, np.int32))
    if case == "mixed":
        return synth.c2_mixed(3, 401, 1203, 121, 41)
    return synth.mixed_small(n=61, seed=8, kmax=8, count=700)  # every type and length up to 8


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("case", ["one", "none", "sat63", "sat64", "sat65", "sat1023", "sat1025", "sat2100", "mixed", "types"])
def test_same_iterates_as_short_launches(case, weighted, bits):
    log(f"case {case} weighted {weighted} bits {bits}")
    inst = instance(case)
    if weighted:
        inst.weight = np.random.default_rng(5).uniform(0.25, 4.0, inst.m).astype(np.float32)
    R, steps = 37, 12
    prob = pcls.Problem.from_instance(inst, accumulator_bits=bits)
    prob.set_launch(1, 0)
    X = prob.new_state(R)
    prob.init_restarts(X, R, 4)
    Y, Z = X.clone(), X.clone()
    tr = prob.step(X, R, 0.1, steps, trace=True)
    parts = [prob.step(Y, R, 0.1, 4, trace=True) for _ in range(steps // 4)]
    assert torch.equal(X[:, :R], Y[:, :R])
    scale = 1.0 + (inst.m if inst.weight is None else float(inst.weight.sum()))
    assert torch.allclose(tr, torch.cat(parts), rtol=0, atol=1e-6 * scale)
    for block in (256, 512):  # fewer waves deal the same chunks
        prob.set_launch(1, block)
        W = Z.clone()
        assert torch.equal(prob.step(W, R, 0.1, steps, trace=True), tr) and torch.equal(W[:, :R], X[:, :R])
    # held variables and the convergence test
    fixed = torch.zeros(inst.n, dtype=torch.int8, device=X.device)
    fixed[::3] = -1
    prob.set_launch(1, 0)
    A, B = Z.clone(), Z.clone()
    _, ia = prob.step_ex(A, R, 0.1, steps, trace=True, fixed=fixed, tol=1e-2, want_iters=True)
    prob.set_launch(2, 0)
    _, ib = prob.step_ex(B, R, 0.1, steps, trace=True, fixed=fixed, tol=1e-9, want_iters=True)
    same = ia >= steps  # restarts that did not stop early took every step in both
    assert torch.equal(A[:, :R][:, same], B[:, :R][:, same])
    assert torch.all(A[::3, :R] == -1) and bool((ib <= steps).all())
