"""Block lists that a build refuses: an error and no result, whatever the shape."""
import time

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


def _fastest(call, reps=3):
    times = []
    for _ in range(reps):
        t = time.perf_counter()
        call()
        times.append(time.perf_counter() - t)
    return min(times)


@pytest.mark.parametrize("case,status", [("one block many times", 3), ("all out of range", 1)])
def test_refusal_costs_no_more_than_a_build(qt, case, status):
    """A refused list is sorted and formed like any other and then dropped: at
    most four times an accepted list of its length and 4 ms, not a walk over
    the list by whoever starts its one leaf."""
    import torch
    b, nb, n = 16, 1024, 300000
    print("refused", case, flush=True)
    pos = torch.randperm(nb * nb, device="cuda")[:n].int()
    V = torch.zeros((n, b, b), dtype=torch.float64, device="cuda")
    I, J = pos // nb, pos % nb
    bad = torch.full_like(I, 5 if status == 3 else nb)

    def accepted():
        qt.build(nb * b, nb * b, b, 8 * b, I, J, V).free()

    def refused():
        with pytest.raises(qt.QtError) as e:
            qt.build(nb * b, nb * b, b, 8 * b, bad, bad, V)
        assert e.value.status == status

    accepted()
    refused()
    good, wrong = _fastest(accepted), _fastest(refused)
    print(f"accepted {good * 1e3:.2f} ms, refused {wrong * 1e3:.2f} ms", flush=True)
    assert wrong <= 4 * good + 4e-3
