"""Workspace queries of the block solves grow with the number of columns, so that
a workspace sized for the widest block serves every narrower one, whichever
tile width the sizes choose (host-only: no call is made)."""
import ctypes as C

import numpy as np
import pytest


@pytest.fixture(scope="module")
def N():
    from paper_2012_00506_amd import _native
    return _native


def _solve_bytes(N, n, b, nsys, m, precision, resid, both):
    bs = N.fb_band(n, b, 2, b + 1, C.c_void_p(1))
    z = (C.c_double * (2 * nsys))(*([0.1] * (2 * nsys)))
    ms = (C.c_int32 * nsys)(*([m] * nsys))
    P = (C.c_void_p * nsys)(*([1] * nsys))
    ld = (C.c_int64 * nsys)(*([n] * nsys))
    res = (C.c_double * nsys)() if resid else None
    lw = C.c_size_t(0)
    o = N.fb_solve_opts(precision, 1e-10, 4, 0)
    assert N.lib().band_shifted_solve(C.byref(bs), nsys, z, ms, P, ld, P, P if both else None, ld,
                                      res, None, C.byref(o), None, C.byref(lw), None) == 0
    return lw.value


def _filter_bytes(N, n, b, cplx, nslice, m, precision, batched):
    bs = N.fb_band(n, b, 2 if cplx else 1, b + 1, C.c_void_p(1))
    lo = np.arange(nslice, dtype=np.float64)
    hi = lo + 1.0
    ms = np.full(nslice, m, np.int32)
    P = (C.c_void_p * nslice)(*([1] * nslice))
    ld = (C.c_int64 * nslice)(*([n] * nslice))
    passes = (C.c_int32 * nslice)()
    o = N.fb_feast_opts(8, 1e-10, 1, precision, 1e-10, 4, 1 if batched else 0, 1e15, 0, 0, 1.0,
                        None, 0)
    lw = C.c_size_t(0)
    assert N.lib().feast_filter(C.byref(bs), nslice, lo.ctypes.data_as(N.PD),
                                hi.ctypes.data_as(N.PD), ms.ctypes.data_as(N.PI32), P, ld, P, ld,
                                None, passes, C.byref(o), None, C.byref(lw), None) == 0
    return lw.value


def _grows(f):
    last = 0
    for m in range(1, 601):
        size = f(m)
        assert size >= last, f"{m} columns {size} bytes, {m - 1} columns {last}"
        last = size


@pytest.mark.parametrize("b", [10, 64, 100])
@pytest.mark.parametrize("precision,resid", [(0, False), (0, True), (1, True)])
@pytest.mark.parametrize("both", [False, True])
def test_shifted_solve_workspace_grows_with_the_columns(N, b, precision, resid, both):
    _grows(lambda m: _solve_bytes(N, 16384, b, 8, m, precision, resid, both))


@pytest.mark.parametrize("b", [10, 64, 100])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cplx,batched", [(False, True), (True, True), (True, False)])
def test_filter_workspace_grows_with_the_columns(N, b, precision, cplx, batched):
    for nslice in (1, 3):
        _grows(lambda m: _filter_bytes(N, 16384, b, cplx, nslice, m, precision, batched))
