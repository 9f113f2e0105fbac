"""GPU parity of the row-polling triangular solve (rows of more than 32 entries): row lengths at
the edges of its items and batches, against the componentwise backward error of substitution."""
import numpy as np
import pytest

import oracle as O
from paper_1606_00545_amd import hec, synth
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu


def _rows(lens, n, rng, upper):
    """Strictly triangular pattern whose last rows (first, for the upper triangle) have the lengths
    `lens`, the others 0 to 3 entries, among the 40 nearest rows for short ones: several levels."""
    rows, cols = [], []
    for t in range(n):
        L = min(t, lens[t - (n - len(lens))] if t >= n - len(lens) else int(rng.integers(0, 4)))
        lo = 0 if L > 40 else max(0, t - 40)
        for j in rng.choice(np.arange(lo, t), size=min(L, t - lo), replace=False):
            rows.append(t)
            cols.append(int(j))
    r, c = np.array(rows), np.array(cols)
    return (n - 1 - r, n - 1 - c) if upper else (r, c)


def _matrix(lens, n, seed):
    import scipy.sparse as sp
    rng = np.random.default_rng(seed)
    S = sp.eye(n, format="lil")
    for upper in (False, True):
        r, c = _rows(lens, n, rng, upper)
        S[r, c] = rng.standard_normal(r.size)
    S = S.tocsr()
    d = 1.0 + np.asarray(abs(S).sum(axis=1)).ravel()
    S.setdiag(d)
    S.sort_indices()
    return synth.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data.astype(np.float64))


@pytest.mark.parametrize("lens,n", [([33], 34), ([64, 65], 200), ([0, 31, 32, 33, 63, 64, 65, 66, 127, 128], 400),
                                    ([511, 512, 513, 700, 64, 1025], 1200), ([65] * 9 + [40] * 17, 300)])
@pytest.mark.parametrize("f32", [False, True])
def test_row_lengths(lens, n, f32):
    import scipy.sparse as sp
    import torch
    A = _matrix(lens, n, len(lens) + n)
    F = O.iluk(A.n, A.Ap, A.Aj, A.Ax, 0)
    M = hec.ilu_factor(A, k=0, keep_f32=True)
    lv = hec.level_schedule(M)
    LUx = hec.ilu_export(M)[2]
    u, dt = (2.0 ** -24, torch.float32) if f32 else (2.0 ** -53, torch.float64)
    S = sp.csr_matrix((LUx.astype(np.float32).astype(np.float64) if f32 else LUx, F.LUj, F.LUp), shape=(n, n))
    L, U = sp.tril(S, -1).tocsr() + sp.eye(n), sp.triu(S).tocsr()
    b = dev(np.random.default_rng(n).uniform(-1, 1, n), dt)
    kind = "f32" if f32 else "f64"
    y, z, x, x2 = (empty(n, kind) for _ in range(4))
    hec.trsv_levels(M, lv, b, y, hec.LOWER)
    hec.trsv_levels(M, lv, y, z, hec.UPPER)
    hec.trsv_levels(M, lv, b, x, hec.LU)
    hec.trsv_levels(M, lv, b, x2, hec.LU)
    hec.levels_check(lv)
    b, y, z, x, x2 = (host(v).astype(np.float64) for v in (b, y, z, x, x2))
    assert np.array_equal(x, z) and np.array_equal(x, x2)  # the chain is the two solves, and repeats
    gam = 2 * (int(np.diff(F.LUp).max()) + 2) * u  # substitution in any order of the row's terms
    assert (np.abs(b - L @ y) <= gam * (abs(L) @ np.abs(y) + np.abs(b))).all()
    assert (np.abs(y - U @ z) <= gam * (abs(U) @ np.abs(z) + np.abs(y))).all()
