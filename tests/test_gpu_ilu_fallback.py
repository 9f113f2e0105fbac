"""ilu_factor's rows wait on the device for the rows they eliminate with, each wait bounded by
hec_set_spin_limit. Where one gives up, forced here with a limit of zero polls, the factorisation is done
again with a launch per level, which waits for nothing, and so it is where there is no memory for the start
values beside the factor (that way works in place): the caller gets the same values bit for bit, no status
of its own, and all temporary memory back."""
import numpy as np
import pytest

from paper_1606_00545_amd import hec, synth
from tests.test_gpu_memory import Counting, counting  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _factor(A, k, counting):
    calls = counting.calls
    F = hec.ilu_factor(A, k=k, keep_f32=True)
    assert counting.bytes == hec.footprint(None, F)
    out = hec.ilu_export(F)
    F.close()
    assert counting.bytes == 0
    return out, counting.calls - calls


MATRICES = {"grid": (lambda: synth.lognormal_tpfa((20, 17, 15), 2.0, np.random.default_rng(1)), 0),
            "fill": (lambda: synth.poisson3d(12), 3),
            "long_rows": (lambda: synth.powerlaw_random(3000, np.random.default_rng(2)), 0)}


@pytest.mark.parametrize("name", MATRICES)
def test_zero_spin_limit_leaves_the_factor_as_it_is(name, counting):  # noqa: F811
    make, k = MATRICES[name]
    A = make()
    want, calls = _factor(A, k, counting)
    hec.set_spin_limit(0)
    try:
        got, calls0 = _factor(A, k, counting)
    finally:
        hec.set_spin_limit(-1)
    assert calls0 > calls  # a wait gave up: the second way has buffers of its own
    again, calls1 = _factor(A, k, counting)
    assert calls1 == calls
    for g in (got, again):
        assert all(np.array_equal(a, b) for a, b in zip(g, want))


class Budget(Counting):
    """Refuses what would take the live bytes over a limit."""
    limit = None

    def alloc(self, nbytes, stream):
        return 0 if self.limit is not None and self.bytes + nbytes > self.limit else super().alloc(nbytes, stream)


@pytest.mark.parametrize("name", MATRICES)
def test_an_allocator_that_holds_the_factor_alone_serves_it(name):
    """No more memory than the factor, a row order and a flag word: the values are formed in place."""
    make, k = MATRICES[name]
    A = make()
    c = Budget()
    hec.set_allocator(c.alloc, c.free)
    try:
        (LUp, LUj, LUx), _ = _factor(A, k, c)
        n, nnz = A.n, LUx.size
        need = 4 * (n + 1) + 4 * nnz + 4 * n + 8 * nnz + 4 * n + 4
        c.limit = need
        F = hec.ilu_factor(A, k=k)
        out = hec.ilu_export(F)
        F.close()
        assert all(np.array_equal(a, b) for a, b in zip(out, (LUp, LUj, LUx)))
        c.limit = need - 4 * n - 4  # the factor fits, the row order does not
        with pytest.raises(hec.HecError) as e:
            hec.ilu_factor(A, k=k)
        assert e.value.code == hec.NOMEM and c.bytes == 0
    finally:
        hec.use_torch_allocator()
