"""Workgroups of each full 256 take tiles in an order that keeps neighbouring
columns on one XCD; the last, partial 256 keep theirs.  Every restart has to be
taken once whatever the number of tiles: one restart a tile against eight (few
tiles), bit for bit, and the statistics against sums over separate launches."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from gpu_util import log  # noqa: E402


@pytest.mark.parametrize("R", [1, 255, 256, 257, 511, 513, 600, 1025, 2049])
def test_every_restart_once(R):
    log(f"R {R}")
    inst = synth.mixed_small(n=61, seed=8, kmax=8, count=200)
    prob = pcls.Problem.from_instance(inst)
    X = prob.new_state(R)
    prob.init_restarts(X, R, 4)
    Y = X.clone()
    prob.set_launch(1, 0)
    prob.step(X, R, 0.1, 3)
    prob.set_launch(8, 0)
    prob.step(Y, R, 0.1, 3)
    assert torch.equal(X[:, :R], Y[:, :R])

    # each term is rounded once to a step of at most 2^-40 whatever the launch, so
    # sums agree to the float32 rounding of the output
    whole = prob.constraint_grad_stats(X, R).double()
    parts = torch.zeros_like(whole)
    for r in range(0, R, 128):
        w = min(128, R - r)
        Z = prob.new_state(w)
        Z[:, :w] = X[:, r : r + w]
        parts += prob.constraint_grad_stats(Z, w).double()
    assert torch.allclose(whole, parts, rtol=1e-5, atol=1e-6 * R)
