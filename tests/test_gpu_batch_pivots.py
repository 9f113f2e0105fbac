"""The batched solver divides by the pivots, as its level-order path does, whatever path a factor takes:
on grids whose longest axis has the largest stride both paths subtract a row's terms in the same order, so
that their solutions are the same bit for bit, with FP64 and with FP32 factor values (whose quotients are
formed in FP64). Shapes at the edges of the tiles and with one, several and two tiles a wavefront."""
import numpy as np
import pytest

from paper_1606_00545_amd import hec, synth
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu

SHAPES = [(16, 17), (63, 64), (64, 65), (40, 128), (70, 90), (8, 8, 100), (9, 8, 10), (17, 9, 20), (18, 17, 25)]


@pytest.mark.parametrize("mixed", [False, True])
def test_grid_and_level_order_paths_agree_bit_for_bit(mixed):
    systems = []
    for k, shape in enumerate(SHAPES):
        for grid in (True, False):
            A = synth.lognormal_tpfa(shape, 1.0, np.random.default_rng(k))
            M, F = hec.hec_from_csr(A, keep_f32=True), hec.ilu_factor(A, k=0, keep_f32=True)
            hec.set_trsv_grid(grid)
            try:
                lv = hec.level_schedule(F)
            finally:
                hec.set_trsv_grid(True)
            assert hec.levels_grid(lv) == grid
            systems.append((M, F, lv, dev(np.random.default_rng(k).uniform(-1, 1, A.n)), empty(A.n)))
    B = hec.Batch(len(systems), restart=30, max_n=max(s[0].n for s in systems))
    hec.gmres_solve_batched(B, systems, maxit=4, rtol=1e-12, precision=int(mixed), check=False)
    xs = [host(s[4]) for s in systems]
    for shape, a, b in zip(SHAPES, xs[::2], xs[1::2]):
        assert np.all(np.isfinite(a)) and np.linalg.norm(a) > 0
        assert np.array_equal(a, b), (shape, np.max(np.abs(a - b)) / np.max(np.abs(b)))
