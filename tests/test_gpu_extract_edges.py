"""Extraction where its loads and counts have edges: buckets shorter than the eight
slots loaded at a time, as the image's only and last segment."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from gpu_util import corner_mix, log, oracle_for, rows_of  # noqa: E402


def check(prob, inst, X, R):
    """Corners, violations and best restart against the oracle."""
    a_ref, u_ref, b_ref = oracle_for(inst, with_coefficients=False).extract(rows_of(X, R))
    assign = torch.zeros((R, inst.n), dtype=torch.int8, device=X.device)
    unsat = torch.full((R,), -1, dtype=torch.int32, device=X.device)
    best = torch.full((1,), -1, dtype=torch.int32, device=X.device)
    pcls.check(pcls.load_library().pcls_extract(prob.handle, R, pcls._tptr(X), pcls._tptr(assign),
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
