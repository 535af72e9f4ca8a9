"""Extraction where its loads and counts have edges: buckets shorter than the eight
slots loaded at a time, as the image's only and last segment; a state that is not
16-byte aligned; more constraints than one split's counts hold."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from gpu_util import corner_mix, log, oracle_for, rows_of  # noqa: E402


def check(prob, inst, X, R, ptr=None):
    """Corners, violations and best restart of the state at ptr (default X) against the oracle on X."""
    a_ref, u_ref, b_ref = oracle_for(inst, with_coefficients=False).extract(rows_of(X, R))
    assign = torch.zeros((R, inst.n), dtype=torch.int8, device=X.device)
    unsat = torch.full((R,), -1, dtype=torch.int32, device=X.device)
    best = torch.full((1,), -1, dtype=torch.int32, device=X.device)
    pcls.check(pcls.load_library().pcls_extract(prob.handle, R, ptr or pcls._tptr(X), pcls._tptr(assign),
                                                pcls._tptr(unsat), pcls._tptr(best), pcls._stream()))
    assert np.array_equal(assign.cpu().numpy(), a_ref)
    assert np.array_equal(unsat.cpu().numpy(), u_ref) and int(best) == b_ref


@pytest.mark.parametrize("k", list(range(1, 10)) + [13, 17])
def test_one_segment(k):
    """Every bucket up to 24 literals alone: its block ends where the codes end."""
    for m in (1, 64, 257):
        log(f"case k {k} m {m}")
        inst = synth.random_ksat(max(k, 19), m, k, 10 * k + m)
        prob = pcls.Problem.from_instance(inst)
        X = prob.state_from_rows(corner_mix(np.random.default_rng(k), 33, inst.n))
        check(prob, inst, X, 33)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_unaligned_state(shift):
    log(f"case shift {shift}")
    inst = synth.mixed_small(n=131, seed=shift, kmax=40, count=300)
    prob = pcls.Problem.from_instance(inst)
    R = 70
    X = prob.state_from_rows(corner_mix(np.random.default_rng(shift), R, inst.n))
    raw = torch.empty(X.numel() + shift, device=X.device)
    raw[shift:].copy_(X.reshape(-1))
    check(prob, inst, X, R, ctypes.c_void_p(raw.data_ptr() + 4 * shift))


def test_more_constraints_than_a_split_counts():
    """Clauses of one literal over one variable, all violated where it is +1.  So many
    tiles of restarts that constraints alone ask for a second split: more than a
    split's counts of 16 bits hold."""
    m, R = 70000, 8192
    log(f"case m {m}")
    inst = synth.Instance(1, np.arange(m + 1, dtype=np.int32), np.ones(m, np.int32), np.zeros(m, np.int8),
                          np.zeros(m, np.int32))
    prob = pcls.Problem.from_instance(inst)
    x = np.where(np.arange(R) % 3 == 0, 0.5, -0.5).astype(np.float32)
    assign, unsat, best = prob.extract(prob.state_from_rows(x[:, None]), R)
    assert np.array_equal(assign.cpu().numpy()[:, 0], np.sign(x).astype(np.int8))
    assert np.array_equal(unsat.cpu().numpy(), np.where(x > 0, m, 0)) and int(best) == 1
