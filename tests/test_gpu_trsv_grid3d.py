"""GPU parity of the wavefront triangular solve on 3D grids at the edges of its tiles (8 x 8
columns), of its blocks (4 steps, slots of 8) and of the ring (32 steps), columns along each
axis, against the componentwise backward error of substitution; an infinite right-hand side
reaches exactly the rows that depend on it."""
import numpy as np
import pytest

import oracle as O
from paper_1606_00545_amd import hec, synth
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("shape", [(8, 8, 9), (9, 8, 12), (8, 16, 17), (16, 17, 18), (15, 16, 19), (17, 15, 20),
                                   (24, 25, 53), (53, 9, 10), (10, 61, 33)])
def test_tile_edges(shape, f32):
    import scipy.sparse as sp
    import torch
    A = synth.lognormal_tpfa(shape, 1.0, np.random.default_rng(shape[0]))
    M = hec.ilu_factor(A, k=0, keep_f32=True)
    lv = hec.level_schedule(M)
    assert hec.levels_grid(lv)
    LUp, LUj, LUx = hec.ilu_export(M)
    u, dt = (2.0 ** -24, torch.float32) if f32 else (2.0 ** -53, torch.float64)
    S = sp.csr_matrix((LUx.astype(np.float32).astype(np.float64) if f32 else LUx, LUj, LUp), shape=(A.n, A.n))
    L, U = sp.tril(S, -1).tocsr() + sp.eye(A.n), sp.triu(S).tocsr()
    b = dev(np.random.default_rng(A.n).uniform(-1, 1, A.n), dt)
    y, z, x, x2 = (empty(A.n, "f32" if f32 else "f64") for _ in range(4))
    hec.trsv_levels(M, lv, b, x2, hec.LU)
    hec.trsv_levels(M, lv, b, y, hec.LOWER)
    hec.trsv_levels(M, lv, y, z, hec.UPPER)
    hec.trsv_levels(M, lv, b, x, hec.LU)
    hec.levels_check(lv)
    b, y, z, x, x2 = (host(v).astype(np.float64) for v in (b, y, z, x, x2))
    assert np.array_equal(x, z) and np.array_equal(x, x2)  # the chain is the two solves, and repeats
    gam = 10 * u  # three products and subtractions, the reciprocal pivot and its product, doubled
    assert (np.abs(b - L @ y) <= gam * (abs(L) @ np.abs(y) + np.abs(b))).all()
    assert (np.abs(y - U @ z) <= gam * (abs(U) @ np.abs(z) + np.abs(y))).all()


@pytest.mark.parametrize("which", ["lower", "upper"])
@pytest.mark.parametrize("shape", [(19, 21, 30), (30, 21, 19)])
def test_infinity_stays_in_its_cone(shape, which):
    A = synth.lognormal_tpfa(shape, 1.0, np.random.default_rng(3))
    M = hec.ilu_factor(A, k=0)
    lv = hec.level_schedule(M)
    assert hec.levels_grid(lv)
    nx, ny, nz = shape
    b = np.random.default_rng(4).uniform(-1, 1, A.n)
    b[nx // 2 + nx * (ny // 2 + ny * (nz // 2))] = np.inf
    F = O.iluk(A.n, A.Ap, A.Aj, A.Ax, 0)
    y = empty(A.n)
    hec.trsv_levels(M, lv, dev(b), y, hec.LOWER if which == "lower" else hec.UPPER)
    hec.levels_check(lv)
    ref = (O.trsv_lower if which == "lower" else O.trsv_upper)(F, b)
    assert np.array_equal(np.isfinite(host(y)), np.isfinite(ref))


@pytest.mark.parametrize("f32", [False, True])
def test_nothing_is_left_behind(f32):
    """Solves whose values are infinite leave infinities and NaN in the LDS of every compute
    unit: the solves between them are not touched by them."""
    import torch
    A = synth.lognormal_tpfa((30, 30, 30), 1.0, np.random.default_rng(8))
    M = hec.ilu_factor(A, k=0, keep_f32=True)
    lv = hec.level_schedule(M)
    dt = torch.float32 if f32 else torch.float64
    b = dev(np.random.default_rng(9).uniform(-1, 1, A.n), dt)
    inf = torch.full_like(b, float("inf"))
    x, y = torch.empty_like(b), torch.empty_like(b)
    ref = None
    for _ in range(30):
        for _ in range(4):
            hec.trsv_levels(M, lv, inf, y, hec.LU)
        hec.trsv_levels(M, lv, b, x, hec.LU)
        hec.levels_check(lv)
        got = host(x)
        assert np.isfinite(got).all()
        ref = got if ref is None else ref
        assert np.array_equal(got, ref)
