"""Gradient statistics with several restarts a workgroup and constraints over lane
groups, against the oracle: enough restarts that every CU has a tile of two or more."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from gpu_util import corner_mix, log, oracle_for, rows_of  # noqa: E402


@pytest.mark.parametrize("kmax,R", [(16, 2049), (64, 513), (64, 1025), (64, 2049), (256, 513), (256, 1025)])
def test_grad_stats_of_wide_tiles(kmax, R):
    inst = synth.mixed_small(n=270, seed=kmax + R, kmax=kmax, count=90)
    log(f"case grad stats kmax {kmax} R {R} m {inst.m}")
    prob = pcls.Problem.from_instance(inst)
    X = prob.state_from_rows(corner_mix(np.random.default_rng(R), R, inst.n))
    X[:, R:] = float("nan")  # padding columns must not count
    got = prob.constraint_grad_stats(X, R).cpu().numpy().astype(np.float64)
    want = oracle_for(inst).constraint_grad_sq(rows_of(X, R))
    k = np.diff(inst.row_ptr)
    # FP32 terms (relative 1e-5 of each |dFE/dy| <= 1) and the 2^-s quantum
    tol = 2e-5 * np.sqrt(np.maximum(want, 0) * R * k) + 1e-5 * want + R * k * 2.0 ** -30
    assert np.all(np.abs(got - want) <= tol), np.max(np.abs(got - want) - tol)
