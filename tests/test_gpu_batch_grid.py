"""GPU parity of the batched solver's grid preconditioner solves: shapes at the edges of its tiles (64
columns a wavefront in 2D, 8 x 8 in 3D, one or two tiles a wavefront), FP64 and FP32 factors, against
gmres_solve after three Arnoldi steps (the same method: only rounding differs), and the general
level-order path on the same systems."""
import numpy as np
import pytest

from paper_1606_00545_amd import hec, synth
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu

SHAPES = [(16, 17), (64, 64), (65, 64), (40, 128), (90, 91), (8, 8, 100), (9, 8, 10), (16, 16, 16), (17, 9, 20),
          (20, 20, 20), (18, 17, 25)]


@pytest.mark.parametrize("mixed", [False, True])
def test_three_steps_agree_with_the_single_solver(mixed):
    systems, ref = [], []
    for k, shape in enumerate(SHAPES):
        for grid in (True, False):
            A = synth.lognormal_tpfa(shape, 0.5, np.random.default_rng(k))
            M, F = hec.hec_from_csr(A, keep_f32=True), hec.ilu_factor(A, k=0, keep_f32=True)
            hec.set_trsv_grid(grid)
            try:
                lv = hec.level_schedule(F)
            finally:
                hec.set_trsv_grid(True)
            assert hec.levels_grid(lv) == grid
            b, x = dev(np.random.default_rng(k).uniform(-1, 1, A.n)), empty(A.n)
            hec.gmres_solve(M, F, lv, b, x, restart=30, maxit=3, rtol=1e-12, precision=int(mixed), check=False)
            ref.append(host(x))
            systems.append((M, F, lv, b, empty(A.n)))
    B = hec.Batch(len(systems), restart=30, max_n=max(s[0].n for s in systems))
    for _ in range(2):  # the recorded launch and a replay
        infos = hec.gmres_solve_batched(B, systems, maxit=3, rtol=1e-12, precision=int(mixed), check=False)
        for s, r, i in zip(systems, ref, infos):
            assert i["iterations"] == 3
            # three steps of sums over n rows in other orders; FP32 vectors of the single solver's basis
            tol = 64 * 3 * 2.0 ** (-24 if mixed else -53) * np.sqrt(r.size)
            assert np.linalg.norm(host(s[4]) - r) <= tol * np.linalg.norm(r)
    # FP64 and mixed batches share a context: each has its own recorded launch
    other = hec.gmres_solve_batched(B, systems, rtol=1e-8, precision=int(not mixed))
    assert all(i["status"] == hec.OK and i["rel_res_true"] <= 1e-8 for i in other)
