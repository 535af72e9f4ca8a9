"""A plan has at most as many segments as the kernels hold work counters for (72):
every type and length in one formula, under both bucket tables."""
import numpy as np
import pytest

from paper_2606_06656_amd import pcls, synth


@pytest.mark.parametrize("generic", [False, True])
@pytest.mark.parametrize("table", [0, 1])
def test_segments_of_every_class(table, generic):
    rows, ctype, param = [0], [], []
    for k in range(1, 257):
        for ty in range(7):
            if ty in (synth.CARD_GE, synth.EK):
                prs = sorted({p for p in (0, 1, 2, k // 4, k // 2, 3 * k // 4, k - 2, k - 1, k) if 0 <= p <= k})
            else:
                prs = (0, 1) if ty == synth.XOR else (0,)
            for pr in prs:
                rows.append(rows[-1] + k)
                ctype.append(ty)
                param.append(pr)
    lit = np.arange(rows[-1]) - np.repeat(np.array(rows[:-1]), np.diff(rows)) + 1
    n = pcls.Plan(256, rows, lit, ctype, param, force_generic=generic, bucket_table=table).info().n_segments
    if generic:  # one kind in every bucket of the table
        assert n == (18, 13)[table]
    else:
        assert n <= 72
