"""What a handle or a plan still holds when the call that made it has returned."""
import pytest

pytestmark = pytest.mark.gpu


class Counting:
    """Allocator over torch's that knows its buffers' sizes."""

    def __init__(self, base):
        self.base, self.out, self.freed = base, {}, []

    def alloc(self, n, stream):
        p = self.base.alloc(n, stream)
        if p:
            self.out[p] = n
        return p

    def free(self, p, stream):
        self.freed.append(self.out.pop(p))
        self.base.free(p, stream)

    def held(self):
        return sum(self.out.values())


@pytest.fixture
def counting(qt):
    import torch
    c = Counting(qt.TorchAllocator())
    torch.cuda.synchronize()
    qt.set_allocator(c.alloc, c.free)
    yield c
    torch.cuda.synchronize()
    if qt.ALLOCATOR is not None:
        qt.set_allocator(qt.ALLOCATOR.alloc, qt.ALLOCATOR.free)
    else:
        qt.use_hip_pool()


def _random(qt, nb, count, b, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pos = torch.unique(torch.randint(0, nb * nb, (count,), generator=g, device="cuda"))
    V = torch.randn((len(pos), b, b), generator=g, dtype=torch.float64, device="cuda")
    return qt.build(nb * b, nb * b, b, 8 * b, (pos // nb).int(), (pos % nb).int(), V), pos, V


@pytest.mark.parametrize("nb,count", [(300, 3000), (1500, 30000)])
def test_plan(qt, counting, nb, count):
    """The work prefix sums' scratch, 8 bytes per work item and more, is not
    kept beyond two megabytes."""
    A, _, _ = _random(qt, nb, count, 16, 1)
    del counting.freed[:]
    plan = qt.Plan([A], [A], "f64")
    items = plan.info()["work_items"]
    assert 8 * items <= 2 << 20 or max(counting.freed, default=0) >= 8 * items
    plan.execute(graph=False)
    plan.destroy()
