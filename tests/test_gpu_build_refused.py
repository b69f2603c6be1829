"""Block lists that a build refuses: an error and no result, whatever the shape."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows,n_cols", [(0, 0), (0, 96), (96, 0)])
@pytest.mark.parametrize("on_device", [False, True])
def test_no_position_in_the_grid(qt, n_rows, n_cols, on_device):
    import torch
    b = 32
    print("empty grid", n_rows, n_cols, on_device, flush=True)
    I, J, V = np.zeros(1, np.int32), np.zeros(1, np.int32), np.ones((1, b, b))
    if on_device:
        I, J, V = (torch.as_tensor(x, device="cuda") for x in (I, J, V))
    with pytest.raises(qt.QtError) as e:
        qt.build(n_rows, n_cols, b, 4 * b, I, J, V)
    assert e.value.status == qt.QT_ERR_ARG
    M = qt.build(n_rows, n_cols, b, 4 * b, I[:0], J[:0], V[:0])   # without blocks it stays an all-NIL matrix
    assert M.nblocks == 0
