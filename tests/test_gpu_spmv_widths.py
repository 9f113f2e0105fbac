"""The product with slabs whose width is known at run time only, at the edges of the batches of 10
and 4 slots that are in flight together, against the product in long double; rows shorter and
longer than the slab."""
import numpy as np
import pytest

from paper_1606_00545_amd import hec
from paper_1606_00545_amd.synth import CSR
from tests._gpu import dev, empty, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("width", [9, 10, 11, 13, 14, 15, 19, 20, 23, 24, 25, 31])
def test_run_time_widths(width, f32):
    import torch
    rng = np.random.default_rng(width)
    n = 515
    length = rng.integers(0, width + 4, n)
    length[:3] = [width, width + 3, 0]
    Ap = np.concatenate([[0], np.cumsum(length)]).astype(np.int32)
    Aj = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in length]).astype(np.int32)
    Ax = rng.uniform(-1, 1, Ap[-1]).astype(np.float32).astype(np.float64)
    x = rng.uniform(-1, 1, n).astype(np.float32).astype(np.float64)
    M = hec.hec_from_csr(CSR(n, Ap, Aj, Ax), ell_width=width, keep_f32=True)
    dt, u = (torch.float32, 2.0 ** -24) if f32 else (torch.float64, 2.0 ** -53)
    y = empty(n, "f32" if f32 else "f64")
    hec.hec_spmv(M, dev(x, dt), y)
    p = Ax.astype(np.longdouble) * x[Aj]
    row = np.repeat(np.arange(n), length)
    ref, mag = np.zeros(n, np.longdouble), np.zeros(n, np.longdouble)
    np.add.at(ref, row, p)
    np.add.at(mag, row, np.abs(p))
    bound = (length + 4) * u * mag  # a rounding per product and sum
    assert (np.abs(host(y).astype(np.longdouble) - ref) <= bound).all()
