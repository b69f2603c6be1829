"""Block lists that qt_build refuses by its arguments alone, before it touches
a device: these run with and without a GPU."""
import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("n_rows,n_cols", [(0, 0), (0, 96), (96, 0)])
@pytest.mark.parametrize("leaf", [32, 256])
def test_no_position_in_the_grid(n_rows, n_cols, leaf):
    import paper_1501_07800_amd as qt
    b = 32
    I, J, V = np.zeros(1, np.int32), np.zeros(1, np.int32), np.ones((1, b, b))
    o = ctypes.c_void_p(1)
    rc = qt.lib.qt_build(n_rows, n_cols, b, leaf, 1, I.ctypes.data, J.ctypes.data, V.ctypes.data, qt.MEM_HOST, None,
                         ctypes.byref(o))
    assert rc == qt.QT_ERR_ARG, qt.lib.qt_last_error()
    assert o.value is None
