"""Extraction at the edges of its launch: tiles of 32 restarts, corner rows of any
length and alignment, several splits of a tile, lengths over every plane of the
counts, and more variables than LDS holds words (the path without packing)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from gpu_util import corner_mix, log, oracle_for, rows_of  # noqa: E402


@pytest.mark.parametrize("n,kmax,count,R", [(5, 3, 1, 1), (260, 256, 900, 31), (301, 8, 1023, 33), (302, 16, 1025, 64),
                                            (400, 256, 5000, 130), (40919, 32, 300, 40), (40960, 12, 300, 3)])
def test_extract_equals_oracle(n, kmax, count, R):
    log(f"case n {n} kmax {kmax} count {count} R {R}")
    inst = synth.mixed_small(n=n, seed=n + R, kmax=kmax, count=count)
    prob = pcls.Problem.from_instance(inst)
    X = prob.state_from_rows(corner_mix(np.random.default_rng(count), R, n) if R >= 4
                             else synth.uniform_x(count, R, n))
    X[:, R:] = -1.0  # padding columns must not count
    a_ref, u_ref, b_ref = oracle_for(inst, with_coefficients=False).extract(rows_of(X, R))
    for want in (True, False):
        assign, unsat, best = prob.extract(X, R, want_assign=want)
        assert np.array_equal(unsat.cpu().numpy(), u_ref) and int(best.item()) == b_ref
        if want:
            assert np.array_equal(assign.cpu().numpy(), a_ref)
    # corners at an odd address
    raw = torch.zeros(R * n + 1, dtype=torch.int8, device=X.device)
    unsat = torch.empty(R, dtype=torch.int32, device=X.device)
    L = pcls.load_library()
    import ctypes
    pcls.check(L.pcls_extract(prob.handle, R, pcls._tptr(X), ctypes.c_void_p(raw.data_ptr() + 1), pcls._tptr(unsat),
                              None, pcls._stream()))
    assert np.array_equal(raw[1:].cpu().numpy().reshape(R, n), a_ref) and np.array_equal(unsat.cpu().numpy(), u_ref)
