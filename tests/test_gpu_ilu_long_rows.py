"""The one-launch ILU chooses how a row is worked on row by row: 16 lanes up to 96 entries, a wavefront with the
row in LDS up to 512, beyond that with the row in memory. Rows around each bound and far beyond among short ones
against the oracle and, bit for bit, against the launches per level (forced by a limit of zero polls); a long
row sends no other row another way."""
import numpy as np
import pytest

import oracle as O
from paper_1606_00545_amd import hec
from tests.test_gpu_memory import Counting, counting  # noqa: F401  (fixture)
from tests.test_gpu_trsv_rows import _matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,n,k,inside,beyond", [
    ([91, 92, 93, 94, 95, 96, 97], 400, 0, 96, 97), ([95] * 11 + [300] * 3, 700, 0, 96, 300),
    ([507, 508, 509, 510, 511, 512, 513], 900, 0, 512, 513), ([40, 513, 600], 1100, 0, 64, 513),
    ([2000, 30, 700, 1200], 2600, 0, 64, 2000), ([120, 560], 700, 1, 64, 561)])
def test_rows_on_both_sides_of_a_bound(lens, n, k, inside, beyond, counting):  # noqa: F811
    A = _matrix(lens, n, n + len(lens))
    F = O.iluk(A.n, A.Ap, A.Aj, A.Ax, k)
    w = np.diff(F.LUp)
    assert (w <= inside).any() and w.max() >= beyond
    calls = counting.calls
    M = hec.ilu_factor(A, k=k)
    calls = counting.calls - calls
    LUp, LUj, LUx = hec.ilu_export(M)
    assert np.array_equal(LUp, F.LUp) and np.array_equal(LUj, F.LUj)
    # as in test_gpu_ilu_rows: sums of at most w products, |L||U| <= 3 max row sum entrywise
    scale = 3 * max(np.add.reduceat(np.abs(A.Ax), A.Ap[:-1]).max(), 1.0)
    assert np.max(np.abs(LUx - F.LUx)) <= 2 * (int(w.max()) + 3) ** 2 * 2.0 ** -53 * scale
    assert np.array_equal(hec.ilu_export(hec.ilu_factor(A, k=k))[2], LUx)
    hec.set_spin_limit(0)
    try:
        assert np.array_equal(hec.ilu_export(hec.ilu_factor(A, k=k))[2], LUx)
    finally:
        hec.set_spin_limit(-1)
    S = _matrix([], 50, 1)  # the same buffers as for a matrix of short rows: one launch for all rows
    short = counting.calls
    hec.ilu_factor(S)
    assert calls == counting.calls - short


def test_zero_pivot_seen_by_a_long_row():
    """Rows of every kind eliminate with row 2, whose pivot becomes zero."""
    n = 700
    D = np.diag(np.full(n, 4.0)) + np.diag(np.full(n - 1, 1.0), 1) + np.diag(np.full(n - 1, 1.0), -1)
    D[1, 1], D[2, 2] = 4.25, 0.25  # u_11 = 4, u_22 = 0.25 - 1/4 = 0
    for row, L in ((150, 120), (690, 600)):
        D[row, :L] = 1.0
    from tests._mats import from_dense
    with pytest.raises(hec.HecError) as e:
        hec.ilu_factor(from_dense(D))
    assert e.value.code == hec.ZERO_PIVOT and "row 2" in str(e.value)
