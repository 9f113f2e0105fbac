"""The 3D wavefront solve hands a result to the lanes beside it through LDS, between some of them one step
later: with couplings of -1 along one axis only, unit pivots and whole right-hand sides, the solves are
prefix sums along that axis, exact in FP64 and in FP32, so that a value read a step too early or too late
is a wrong number. Full tiles and ragged ones, along each axis."""
import numpy as np
import pytest

from paper_1606_00545_amd import hec, synth
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu


def _chains(shape, axis, upper):
    """7-point pattern, 1 on the diagonal, -1 to the neighbour before (after) along `axis`, stored zeros else."""
    A = synth.lognormal_tpfa(shape, 0.5, np.random.default_rng(0))
    rows = np.repeat(np.arange(A.n), np.diff(A.Ap))
    off = (1, shape[0], shape[0] * shape[1])[axis] * (1 if upper else -1)
    Ax = np.where(A.Aj == rows, 1.0, np.where(A.Aj - rows == off, -1.0, 0.0))
    return synth.CSR(A.n, A.Ap, A.Aj, Ax)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("shape", [(8, 8, 40), (16, 24, 33), (13, 19, 50)])
def test_prefix_sums_are_exact(shape, axis, f32):
    import torch
    b = np.random.default_rng(1).integers(-9, 10, shape[::-1])  # [z][y][x]: rows in natural order
    for upper in (False, True):
        F = hec.ilu_factor(_chains(shape, axis, upper), k=0, keep_f32=f32)
        lv = hec.level_schedule(F)
        assert hec.levels_grid(lv)
        x = empty(b.size, "f32" if f32 else "f64")
        bd = dev(b.ravel().astype(np.float64), torch.float32 if f32 else torch.float64)
        want = np.flip(np.cumsum(np.flip(b, 2 - axis), 2 - axis), 2 - axis) if upper else np.cumsum(b, 2 - axis)
        for which in (hec.UPPER if upper else hec.LOWER, hec.LU):
            hec.trsv_levels(F, lv, bd, x, which)
            hec.levels_check(lv)
            assert np.array_equal(host(x), want.ravel())
