"""What a schedule with wavefront plans holds: seven coefficients and one value of the intermediate for each
padded position (claim, step, lane), two vectors of the system's size and the two face buffers, 16 values for
each step of a tile, are enough for it, with, for a system that the batched solver takes, the bytes of a
level-ordered copy of both triangles (three entries a row each, their rows, the pivots)."""
import numpy as np
import pytest

from paper_1606_00545_amd import hec, synth
from tests.test_gpu_memory import Counting, counting  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(9, 8, 10), (16, 16, 16), (17, 16, 30), (20, 20, 24), (24, 24, 24), (9, 20, 70)])
def test_schedule_bytes(shape, counting):  # noqa: F811
    A = synth.lognormal_tpfa(shape, 1.0, np.random.default_rng(0))
    F = hec.ilu_factor(A)
    before = counting.bytes
    lv = hec.level_schedule(F)
    assert hec.levels_grid(lv)
    na, nb, nc = sorted(shape)[0], sorted(shape)[1], max(shape)
    tiles = -(-na // 8) * -(-nb // 8)
    pad = 64 * tiles * (nc + 14)
    need = 8 * (7 * pad + pad + 2 * A.n + 2 * 16 * tiles * (nc + 14)) + 64
    if A.n <= hec.BATCH_MAX_N:
        need += A.n * (2 * (3 * 12 + 4) + 8)
    assert hec.footprint(None, None, lv) == counting.bytes - before <= need
