"""Host-side checks of the row layout that triangles with rows too long for the blocked solve get
(make_row_plan, through libhecplan.so): what the row-polling kernel relies on so that its waits end, and the
solution replayed item by item in claim order, a dependency read only if an earlier item solved it."""
import ctypes as C

import numpy as np
import pytest

import oracle as O
from paper_1606_00545_amd import synth
from tests import _plan
from tests.test_gpu_trsv_rows import _matrix
from tests.test_trsv_plan import sparse_random


def _rows_plan(F, upper, lds_max=_plan.LDS_MAX, blocks=None):
    L = _plan.lib()
    ip = np.ctypeslib.ndpointer(np.int32, flags="C_CONTIGUOUS")
    L.hecplan_rows_make.restype = C.c_void_p
    L.hecplan_rows_make.argtypes = [C.c_int32, ip, ip, ip, C.c_int32, C.c_int64, C.c_void_p, C.c_int32]
    L.hecplan_rows_array.restype = C.c_int64
    L.hecplan_rows_array.argtypes = [C.c_void_p, C.c_char_p, C.c_void_p]
    L.hecplan_rows_bounds.argtypes = [ip]
    L.hecplan_rows_free.argtypes = [C.c_void_p]
    bl = None if blocks is None else np.ascontiguousarray(blocks, np.int32)
    h = L.hecplan_rows_make(F.n, _plan._i32(F.LUp), _plan._i32(F.LUj), _plan.diag_positions(F), int(upper), lds_max,
                            None if bl is None else bl.ctypes.data, 0 if bl is None else bl.size)
    if not h:
        return None
    P = {}
    try:
        for name in ("rptr", "items", "enc", "src", "grow", "pos", "psrc", "lev"):
            P[name] = np.empty(L.hecplan_rows_array(h, name.encode(), None), np.int32)
            L.hecplan_rows_array(h, name.encode(), P[name].ctypes.data_as(C.c_void_p))
    finally:
        L.hecplan_rows_free(h)
    b = np.empty(2, np.int32)
    L.hecplan_rows_bounds(b)
    P["short"], P["group"] = int(b[0]), int(b[1])
    P["items"] = P["items"].reshape(-1, 2)
    return P


CASES = {
    "powerlaw": (lambda: synth.powerlaw_random(4000, np.random.default_rng(3)), 0, {}),
    "ilu3": (lambda: synth.poisson3d(12), 3, {}),
    "edges": (lambda: _matrix([0, 31, 32, 33, 63, 64, 65, 66, 127, 128], 400, 5), 0, {}),
    "only_long": (lambda: _matrix([66 + i for i in range(40)], 300, 6), 0, {}),
    "small_lds": (lambda: sparse_random(900, 8, 8), 1, {"lds_max": 1024}),
    "blocks": (lambda: _matrix([70, 40, 80], 300, 7), 0, {"blocks": [0, 300]}),
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("upper", [False, True])
def test_rows_items_and_replay(name, upper):
    make, k, opt = CASES[name]
    A = make()
    F = O.iluk(A.n, A.Ap, A.Aj, A.Ax, k)
    n, diag = F.n, _plan.diag_positions(F)
    P = _rows_plan(F, upper, **opt)
    assert P is not None
    grow, pos, rptr, items = P["grow"], P["pos"], P["rptr"], P["items"]
    assert np.array_equal(np.sort(grow), np.arange(n)) and np.array_equal(pos[grow], np.arange(n))
    first = diag[grow] + 1 if upper else np.asarray(F.LUp)[grow]
    last = np.asarray(F.LUp)[grow + 1] if upper else diag[grow]
    assert rptr[0] == 0 and np.array_equal(np.diff(rptr), last - first)
    assert P["enc"].size == P["src"].size == rptr[n]
    if upper:
        assert np.array_equal(P["psrc"][:n], diag[grow])
    for q in range(n):  # an entry: the value's place and where its column's row is solved
        src = P["src"][rptr[q]:rptr[q + 1]]
        assert np.array_equal(src, np.arange(first[q], last[q]))
        assert np.array_equal(P["enc"][rptr[q]:rptr[q + 1]], pos[np.asarray(F.LUj)[src]])
    # items: all positions in order, once; long rows alone, short ones up to a group, one level each
    at, item_of = 0, np.empty(n, np.int64)
    for t, (q0, cnt) in enumerate(items):
        assert q0 == at and 0 <= cnt <= P["group"]
        m = max(cnt, 1)
        lens = np.diff(rptr[q0:q0 + m + 1])
        assert (lens <= P["short"]).all() if cnt else lens[0] > P["short"]
        assert np.unique(P["lev"][grow[q0:q0 + m]]).size == 1
        item_of[q0:q0 + m] = t
        at += m
    assert at == n
    # a dependency is solved by an earlier item, so the lowest unfinished item can always proceed
    assert (item_of[P["enc"]] < np.repeat(item_of, np.diff(rptr))).all()
    # replay
    b = np.random.default_rng(1).uniform(-1, 1, n)
    x = np.full(n, np.nan)
    for q0, cnt in items:
        new = [(q, b[grow[q]] - F.LUx[P["src"][rptr[q]:rptr[q + 1]]] @ x[P["enc"][rptr[q]:rptr[q + 1]]])
               for q in range(q0, q0 + max(cnt, 1))]
        for q, v in new:
            x[q] = v / F.LUx[P["psrc"][q]] if upper else v
    want = O.trsv_upper(F, b) if upper else O.trsv_lower(F, b)
    # the same rows, each a sum of at most w products in another order (diagonally dominant factors)
    w = int(np.diff(F.LUp).max())
    assert np.max(np.abs(x[pos] - want)) <= 4 * (w + 2) * 2.0 ** -53 * max(np.abs(want).max(), 1.0) * len(np.unique(P["lev"]))


def test_a_plan_that_fits_has_no_row_layout():
    F = O.iluk(*(lambda A: (A.n, A.Ap, A.Aj, A.Ax))(synth.poisson2d(20)), 0)
    assert _rows_plan(F, False) is None
