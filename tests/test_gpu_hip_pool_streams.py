"""The library's own memory, HIP's stream-ordered pool: what was made on a
caller's stream comes back also where that stream is gone when its handle goes."""
import ctypes

import numpy as np
import pytest

from tests._util import random_pattern

pytestmark = pytest.mark.gpu


def _hip():
    """The HIP runtime of this process."""
    paths = {l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l}
    assert len(paths) == 1, paths
    return ctypes.CDLL(paths.pop())


@pytest.mark.parametrize("form", ["f32", "bf16x3", "norms"])
def test_forms_made_on_a_stream_that_is_gone(qt, form):
    import torch
    hip = _hip()
    A = random_pattern(np.random.default_rng(4), 40, 40, 0.5, 64)
    D = random_pattern(np.random.default_rng(5), 40, 40, 1 / 1600, 64)      # one block: C stays small
    home = torch.cuda.Stream()
    ref = None
    torch.cuda.synchronize()
    free = []
    qt.use_hip_pool()
    try:
        for rep in range(24):
            print("stream gone", form, rep, flush=True)
            ptr = ctypes.c_void_p()
            assert hip.hipStreamCreateWithFlags(ctypes.byref(ptr), 1) == 0      # non-blocking
            own = torch.cuda.ExternalStream(ptr.value)
            h, d = qt.from_blockmatrix(A, 256, stream=home), qt.from_blockmatrix(D, 256, stream=home)
            C = qt.multiply_tau(h, d, 1e-3, stream=own) if form == "norms" else qt.multiply(h, d, form, stream=own)
            I, J, V = C.to_blocks(stream=own)
            C.free()
            own.synchronize()
            assert hip.hipStreamDestroy(ptr) == 0
            h.free()
            d.free()
            torch.cuda.synchronize()
            if ref is None:
                ref = I, J, V
            assert all(np.array_equal(x, y) for x, y in zip(ref, (I, J, V)))
            free.append(torch.cuda.mem_get_info()[0])
    finally:
        torch.cuda.synchronize()
        if qt.ALLOCATOR is not None:
            qt.set_allocator(qt.ALLOCATOR.alloc, qt.ALLOCATOR.free)
    # lost forms would take 12 MiB (f32) and more a turn
    assert free[7] - free[-1] <= 64 << 20
