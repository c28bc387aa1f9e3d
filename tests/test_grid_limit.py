"""Grids of more than 2^29 cells, whose FP64 planes the sweeps' 32-bit byte offsets do not reach, are
refused where a grid is checked; the largest within the limit is not.  No device is touched: the
permittivity's first value is invalid, which is found after the grid's check and before any other value
is read."""
import ctypes

import pytest


@pytest.mark.parametrize("n,m,refused", [(32768, 16384, False), (1 << 28, 2, False), (32768, 16386, True),
                                         (32768, 32768, True), (65536, 65536, True), (2, (1 << 28) + 2, True),
                                         (2147483646, 2147483646, True)])
def test_cell_limit(n, m, refused):
    from paper_2304_00337_amd import native
    lib = native.load()
    o = native.BlOpts()
    lib.bl_default_opts(ctypes.byref(o), 1)
    g = native.BlGrid(n, m, 1.0, 1.0)
    eps = (ctypes.c_double * 1)(-1.0)
    h = ctypes.c_void_p()
    assert lib.bl_create(ctypes.byref(g), eps, ctypes.byref(o), None, ctypes.byref(h)) == native.BL_EINVAL
    text = lib.bl_last_error()
    assert (b"2^29" in text) == refused and (b"eps must be" in text) != refused, text
