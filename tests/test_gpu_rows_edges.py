"""State from rows: no restarts, and rows whose memory holds the opposite sign."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from paper_2606_06656_amd.autograd import fe_objective  # noqa: E402
from gpu_util import log  # noqa: E402


def test_no_rows_are_not_outside():
    log("case R 0")
    prob = pcls.Problem.from_instance(synth.random_ksat(9, 20, 3, 1))
    outside = torch.full((1,), 7, dtype=torch.int32, device=prob.device)
    pcls.check(pcls.load_library().pcls_state_from_rows(prob.handle, 0, None, None, ctypes.c_void_p(outside.data_ptr()),
                                                        pcls._stream()))
    assert int(outside) == 0
    X, outside = prob.state_and_range(torch.empty((0, 9), device=prob.device))
    assert tuple(X.shape) == (9, 0) and int(outside) == 0


@pytest.mark.parametrize("R,n", [(1, 1), (5, 9)])
def test_rows_with_a_pending_sign(R, n):
    """The imaginary part of a conjugate is a view that negates on reading."""
    log(f"case negated view R {R} n {n}")
    prob = pcls.Problem.from_instance(synth.random_ksat(n, 20 if n > 1 else 1, min(n, 3), 1))
    t = torch.linspace(-1, 0.5, R * n, device=prob.device).reshape(R, n)
    y = torch.complex(t, t).conj().imag if n == 1 else torch._neg_view(t)
    assert y.is_neg() and y.is_contiguous()
    X, outside = prob.state_and_range(y)
    assert torch.equal(X[:, :R], -t.T) and int(outside) == 0
    a, b = y.detach().requires_grad_(True), (-t).requires_grad_(True)
    fa, fb = fe_objective(prob, a), fe_objective(prob, b)
    fa.sum().backward()
    fb.sum().backward()
    assert torch.equal(fa, fb) and torch.equal(a.grad, b.grad)
