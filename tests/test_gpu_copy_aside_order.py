"""A large copy-out whose sort has a stream of its own: where its scratch is
obtained and given back."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


class Recording:
    """Allocator over torch's that notes the stream of every call, and fails
    allocation number fail_at."""

    def __init__(self, base, fail_at=None):
        self.base, self.fail_at, self.made, self.freed = base, fail_at, [], {}

    def alloc(self, n, stream):
        if len(self.made) == self.fail_at:
            return None
        p = self.base.alloc(n, stream)
        self.made.append((p, stream or 0))
        return p

    def free(self, p, stream):
        self.freed[p] = stream or 0
        self.base.free(p, stream)


def _restore(qt):
    if qt.ALLOCATOR is not None:
        qt.set_allocator(qt.ALLOCATOR.alloc, qt.ALLOCATOR.free)
    else:
        qt.use_hip_pool()


def _matrix(qt, n, b=32, nb=300, seed=0):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pos = torch.randperm(nb * nb, generator=g, device="cuda")[:n]
    I, J = (pos // nb).int(), (pos % nb).int()
    V = torch.randn((n, b, b), generator=g, dtype=torch.float64, device="cuda")
    M = qt.build(nb * b, nb * b, b, 8 * b, I, J, V)
    o = torch.argsort(pos)
    torch.cuda.synchronize()
    return M, I[o], J[o], V[o]


@pytest.mark.parametrize("fail_at", [None, 1, 2, 3])
def test_scratch_goes_back_where_it_is_safe(qt, fail_at):
    """The sort's scratch (the first allocation) is made on the sort's stream.
    It goes back on the caller's once that runs after the sort; when the call
    fails before, on the stream it was made on."""
    import torch
    n = 16384                                       # 128 MiB of values
    M, wI, wJ, wV = _matrix(qt, n)
    rec = Recording(qt.TorchAllocator(), fail_at)
    s = torch.cuda.Stream()
    big = torch.randn(6144, 6144, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for _ in range(20):
            big @ big                               # s is busy: the sort goes to its own stream
    try:
        qt.set_allocator(rec.alloc, rec.free)
        if fail_at is None:
            I, J, V = M.to_blocks(stream=s)
        else:
            with pytest.raises(qt.QtError) as e:
                M.to_blocks(stream=s)
            assert e.value.status == qt.QT_ERR_OOM
    finally:
        _restore(qt)
        torch.cuda.synchronize()
    p, made_on = rec.made[0]
    assert made_on != s.cuda_stream
    assert len(rec.freed) == len(rec.made)
    assert rec.freed[p] == (s.cuda_stream if fail_at is None else made_on)
    if fail_at is None:
        assert np.array_equal(I, wI.cpu().numpy()) and np.array_equal(J, wJ.cpu().numpy())
        assert np.array_equal(V, wV.cpu().numpy())
