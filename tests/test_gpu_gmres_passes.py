"""One GMRES(30) cycle at sizes on both sides of where a step's partial sums are added by the
update pass itself or by a launch of their own (32 workgroups of the dot pass: 8,192 rows with
more than 16 basis vectors, 65,536 with up to 4), against the oracle's modified Gram-Schmidt.
The bound: rounding of the cycle, 1e-16 times the condition of its least-squares problem, well
under 1e7 on these systems."""
import numpy as np
import pytest

import oracle as O
from paper_1606_00545_amd import hec, synth
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(128, 64), (3, 2731), (128, 128), (5, 3277), (3, 10923), (256, 256), (3, 21846)])
def test_one_cycle(shape):
    A = synth.lognormal_tpfa(shape, 0.5, np.random.default_rng(shape[0]))
    F = O.iluk(A.n, A.Ap, A.Aj, A.Ax, 0)
    b = np.random.default_rng(shape[1]).uniform(-1, 1, A.n)
    ro = O.gmres(A, F, b, restart=30, maxit=30, rtol=1e-9)
    M, G = hec.hec_from_csr(A), hec.ilu_factor(A, k=0)
    x = empty(A.n)
    inf = hec.gmres_solve(M, G, hec.level_schedule(G), dev(b), x, restart=30, maxit=30, rtol=1e-9, check=False)
    assert inf["iterations"] == ro.iterations
    assert np.linalg.norm(host(x) - ro.x) <= 1e-9 * np.linalg.norm(ro.x)
