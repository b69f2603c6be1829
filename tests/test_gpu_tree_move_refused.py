"""A build whose tree would move to a buffer of its size, by an allocator with no
room for that second buffer: the matrix keeps the first one."""
import pytest

pytestmark = pytest.mark.gpu


class FailingOnce:
    """Allocator over torch's that fails allocation number fail_at only."""

    def __init__(self, base, fail_at=None):
        self.base, self.fail_at, self.count = base, fail_at, 0

    def alloc(self, n, stream):
        k, self.count = self.count, self.count + 1
        return None if k == self.fail_at else self.base.alloc(n, stream)

    def free(self, p, stream):
        self.base.free(p, stream)


def test_the_move_is_no_condition_of_a_build(qt):
    import torch
    b, nb = 16, 30000                               # a diagonal: few leaves and nodes, many positions
    I = torch.arange(nb, device="cuda").int()
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    V = torch.randn((nb, b, b), generator=g, dtype=torch.float64, device="cuda")
    want = (I.cpu().numpy(), I.cpu().numpy(), V.cpu().numpy())
    torch.cuda.synchronize()
    base = qt.TorchAllocator()

    def build(fail_at):
        """The matrix, or None where the call ran out of memory, and its allocations."""
        a = FailingOnce(base, fail_at)
        try:
            qt.set_allocator(a.alloc, a.free)
            return qt.build(nb * b, nb * b, b, 8 * b, I, I, V), a.count
        except qt.QtError as e:
            assert e.status == qt.QT_ERR_OOM
            return None, a.count
        finally:
            torch.cuda.synchronize()
            if qt.ALLOCATOR is not None:
                qt.set_allocator(qt.ALLOCATOR.alloc, qt.ALLOCATOR.free)
            else:
                qt.use_hip_pool()

    whole, count = build(None)
    built = []
    for k in range(count):
        print("fails once", k, flush=True)
        M, n = build(k)
        if M is not None:
            assert n == count
            built.append(M)
    assert len(built) == 1                          # all other buffers are needed
    for M in built:
        assert all((x == y).all() for x, y in zip(M.to_blocks(), want))
        C = qt.multiply(M, whole)
        for x, y in zip(C.to_blocks(), qt.multiply(whole, M).to_blocks()):
            assert (x == y).all()
