"""The steps of an AMG cycle on operators of every storage: rows of w entries each around a
ring, w at the edges of the ELL widths (8 entries; 20 from 16,384 rows on) and of the lanes
per CSR row (2 to 64), one cycle against the oracle's, with both smoothers. The bound is a
cycle's rounding: some 30 steps of at most w products on a diagonally dominant system."""
import numpy as np
import pytest

from oracle import amg as OA
from paper_1606_00545_amd import hec
from paper_1606_00545_amd.synth import CSR
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu


def ring(n, w):
    """Symmetric, every row with w entries: offsets +-1 .. +-(w-1)//2, and n/2 if w is even."""
    rng = np.random.default_rng(w)
    i = np.arange(n)
    cols, vals = [i], [np.zeros(n)]
    for o in range(1, (w - 1) // 2 + 1):
        v = -rng.uniform(0.5, 1.0, n)  # couples row i with row i + o
        cols += [(i + o) % n, (i - o) % n]
        vals += [v, v[(i - o) % n]]
    if w % 2 == 0:
        v = -rng.uniform(0.5, 1.0, n)
        cols.append((i + n // 2) % n)
        vals.append(np.where(i < n // 2, v, v[(i + n // 2) % n]))
    C, V = np.stack(cols, 1), np.stack(vals, 1)
    V[:, 0] = 1.0 - V.sum(axis=1)
    order = np.argsort(C, axis=1)
    C, V = np.take_along_axis(C, order, 1), np.take_along_axis(V, order, 1)
    return CSR(n, np.arange(n + 1, dtype=np.int32) * w, C.astype(np.int32).ravel(), V.ravel())


@pytest.mark.parametrize("smoother", ["jacobi", "chebyshev"])
@pytest.mark.parametrize("n,w", [(600, 2), (600, 7), (600, 8), (600, 9), (600, 24), (600, 25), (600, 97), (600, 301),
                                 (16382, 20), (16384, 20), (16384, 21)])
def test_one_cycle_on_every_storage(n, w, smoother):
    A = ring(n, w)
    opt = dict(coarse_size=8, smoother=smoother)
    H = OA.hierarchy(A, **opt)
    G = hec.amg_setup(A, **opt)
    b = np.random.default_rng(6).uniform(-1, 1, n)
    x = empty(n)
    inf = hec.amg_solve(G, dev(b), x, maxit=1, rtol=0.0, check=False)
    assert inf["iterations"] == 1
    xo = OA.vcycle(H, b, np.zeros(n))
    assert np.linalg.norm(host(x) - xo) <= 1e-12 * np.linalg.norm(xo)
    r = b - H.levels[0].A @ host(x)
    assert abs(inf["rel_res_true"] - np.linalg.norm(r) / np.linalg.norm(b)) <= 1e-13
