"""State from rows: no restarts."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
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
