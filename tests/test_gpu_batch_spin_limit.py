"""The batched solver's waits with a limit of zero polls, on each path that a system's triangles take: the
polled dependencies of the level-order copies and the wait for the wavefront that has a grid's only tile give
up, end the launch and are reported; a grid of several tiles waits at barriers only. The same handles solve
afterwards, and a system that gave up leaves the others' results alone."""
import numpy as np
import pytest

import oracle as O
from paper_1606_00545_amd import hec, synth
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu


def _system(A, seed, grid=True):
    M, F = hec.hec_from_csr(A, keep_f32=True), hec.ilu_factor(A, k=0, keep_f32=True)
    hec.set_trsv_grid(grid)
    try:
        lv = hec.level_schedule(F)
    finally:
        hec.set_trsv_grid(True)
    assert hec.levels_grid(lv) == grid
    xt = np.random.default_rng(seed).uniform(-1, 1, A.n)
    return M, F, lv, dev(O.csr_spmv(A.n, A.Ap, A.Aj, A.Ax, xt)), empty(A.n)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("path", ["level_order", "one_tile", "tiles2d", "tiles3d"])
def test_zero_limit(path, mixed):
    A = {"tiles2d": lambda: synth.poisson2d(80), "tiles3d": lambda: synth.poisson3d(14)}.get(
        path, lambda: synth.poisson2d(64))()
    gives_up = path in ("level_order", "one_tile")
    systems = [_system(A, s, path != "level_order") for s in range(3)]
    systems.append(_system(synth.poisson2d(80), 9))  # no wait in this one
    opts = dict(rtol=1e-8, maxit=200, precision=int(mixed))
    B = hec.Batch(len(systems), restart=30, max_n=max(s[0].n for s in systems))
    want = hec.gmres_solve_batched(B, systems, **opts)
    xs = [host(s[4]) for s in systems]
    hec.set_spin_limit(0)
    try:
        if gives_up:
            with pytest.raises(hec.HecError) as e:
                hec.gmres_solve_batched(B, systems, **opts)
            assert e.value.code == hec.TIMEOUT
        else:
            hec.gmres_solve_batched(B, systems, **opts)
        assert np.array_equal(host(systems[-1][4]), xs[-1])
    finally:
        hec.set_spin_limit(-1)
    infos = hec.gmres_solve_batched(B, systems, **opts)
    for i, w, s, x in zip(infos, want, systems, xs):
        assert i["status"] == hec.OK and i["iterations"] == w["iterations"] and np.array_equal(host(s[4]), x)
