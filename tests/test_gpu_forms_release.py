"""A handle's derived forms (fp32 copy, bf16 split, norms), made on the stream of
the call that first needs them and read by calls on other streams, go back with
the handle: in order on the stream that made it."""
import numpy as np
import pytest

from tests._util import random_pattern

pytestmark = pytest.mark.gpu


class Recording:
    def __init__(self, base):
        self.base, self.live, self.freed = base, {}, []

    def alloc(self, n, stream):
        p = self.base.alloc(n, stream)
        if p:
            self.live[p] = (n, stream or 0)
        return p

    def free(self, p, stream):
        self.freed.append(self.live.pop(p) + (stream or 0,))
        self.base.free(p, stream)


@pytest.mark.parametrize("form", ["f32", "bf16x3", "norms"])
def test_forms_are_released_on_the_handles_stream(qt, form):
    import torch
    A = random_pattern(np.random.default_rng(4), 20, 20, 0.3, 32)
    s1, s2, s3 = (torch.cuda.Stream() for _ in range(3))
    rec = Recording(qt.TorchAllocator())
    torch.cuda.synchronize()
    try:
        qt.set_allocator(rec.alloc, rec.free)
        h = qt.from_blockmatrix(A, 128, stream=s1)
        before = set(rec.live)
        if form == "norms":
            qt.multiply_tau(h, h, 1e-3, stream=s2).free()
            qt.multiply_tau(h, h, 1e-3, stream=s3).free()
        else:
            qt.multiply(h, h, form, stream=s2).free()
            qt.multiply(h, h, form, stream=s3).free()
        torch.cuda.synchronize()
        made = [rec.live[p] for p in set(rec.live) - before]
        assert made and all(stream == s2.cuda_stream for _, stream in made)
        del rec.freed[:]
        h.free()
        assert len(rec.freed) >= len(made) + 1
        assert all(stream == s1.cuda_stream for _, _, stream in rec.freed)
    finally:
        torch.cuda.synchronize()
        if qt.ALLOCATOR is not None:
            qt.set_allocator(qt.ALLOCATOR.alloc, qt.ALLOCATOR.free)
        else:
            qt.use_hip_pool()
