"""State from rows: the transposition and range check in one kernel, at edges of its
64 x 64 tiles, and the autograd objective on inputs that take the other path."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from paper_2606_06656_amd.autograd import fe_objective  # noqa: E402
from gpu_util import log  # noqa: E402


@pytest.mark.parametrize("n,R", [(3, 1), (63, 64), (64, 65), (65, 63), (200, 130)])
def test_rows_and_range(n, R):
    log(f"case rows n {n} R {R}")
    prob = pcls.Problem.from_instance(synth.random_ksat(n, 5 if n > 3 else 1, 3, 1))
    x = torch.tensor(synth.uniform_x(n + R, R, n), device=prob.device)
    x[0, 0], x[-1, -1] = 1.0, -1.0
    X, outside = prob.state_and_range(x)
    assert torch.equal(X[:, :R], x.T) and bool((X[:, R:] == 0).all()) and int(outside) == 0
    for bad in (1.0000001, -1.5, float("nan"), float("inf")):
        for at in ((0, 0), (R - 1, n - 1)):
            y = x.clone()
            y[at] = bad
            assert int(prob.state_and_range(y)[1]) == 1
            with pytest.raises(ValueError):
                fe_objective(prob, y)
            with pytest.raises(ValueError):
                fe_objective(prob, y.double())
    for z in (x.double(), x.T.contiguous().T):  # other types and strides
        a, b = x.clone().requires_grad_(True), z.clone().requires_grad_(True)
        fa, fb = fe_objective(prob, a), fe_objective(prob, b)
        fa.sum().backward()
        fb.sum().backward()
        assert torch.equal(fa.float(), fb.float()) and torch.equal(a.grad, b.grad.float())
