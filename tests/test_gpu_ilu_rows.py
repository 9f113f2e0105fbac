"""GPU parity of the one-launch ILU(k): row lengths at the edges of its widths (96 entries for 16 lanes
a row, 512 for 64, beyond that a launch per level) against the oracle; repeats are bit-identical."""
import numpy as np
import pytest

import oracle as O
from paper_1606_00545_amd import hec, synth
from tests.test_gpu_trsv_rows import _matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,n,k", [([], 9, 0), ([15, 16, 17, 31, 33], 150, 0), ([40, 46, 47, 48], 300, 0),
                                      ([49, 63, 64, 65], 300, 0), ([200, 250, 254, 255], 700, 0),
                                      ([256, 300], 700, 0), ([12, 20, 30], 200, 1)])
def test_row_lengths(lens, n, k):
    A = _matrix(lens, n, n + len(lens))
    F = O.iluk(A.n, A.Ap, A.Aj, A.Ax, k)
    LUp, LUj, LUx = hec.ilu_export(hec.ilu_factor(A, k=k))
    assert np.array_equal(LUp, F.LUp) and np.array_equal(LUj, F.LUj)
    # an entry's elimination is a sum of at most w products; the matrix is row diagonally dominant, so
    # the factors' growth is bounded and |L||U| <= 3 max row sum entrywise: w + 3 roundings of that
    w = int(np.diff(LUp).max())
    scale = 3 * max(np.add.reduceat(np.abs(A.Ax), A.Ap[:-1]).max(), 1.0)
    assert np.max(np.abs(LUx - F.LUx)) <= 2 * (w + 3) ** 2 * 2.0 ** -53 * scale


def test_grid_levels_repeat_bit_for_bit():
    A = synth.lognormal_tpfa((23, 19, 17), 2.0, np.random.default_rng(1))
    for k in (0, 1, 3):
        a, b = (hec.ilu_export(hec.ilu_factor(A, k=k))[2] for _ in range(2))
        assert np.array_equal(a, b)
        F = O.iluk(A.n, A.Ap, A.Aj, A.Ax, k)
        assert np.max(np.abs(a - F.LUx) / np.maximum(np.abs(F.LUx), 1e-3 * np.abs(F.LUx).max())) <= 1e-12


def test_zero_pivot_in_a_later_level():
    """The pivot of row 2 becomes zero by elimination; rows after it depend on it and still finish."""
    n = 64
    D = np.diag(np.full(n, 4.0)) + np.diag(np.full(n - 1, 1.0), 1) + np.diag(np.full(n - 1, 1.0), -1)
    D[1, 1], D[2, 2] = 4.25, 0.25  # u_11 = 4, u_22 = 0.25 - 1/4 = 0
    from tests._mats import from_dense
    with pytest.raises(hec.HecError) as e:
        hec.ilu_factor(from_dense(D))
    assert e.value.code == hec.ZERO_PIVOT and "row 2" in str(e.value)
