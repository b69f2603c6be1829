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


def _structure_bytes(M):
    """Child tables and keys of the nodes, bases, keys and masks of the leaves,
    block keys, and the padding of each array to 256 bytes."""
    nodes = M.levels()
    return int(24 * nodes[:-1].sum() + 36 * nodes[-1] + 8 * M.nblocks) + 256 * (2 * len(nodes) + 6)


def _allowed(M, b, values=True):
    v = 8 * M.nblocks * b * b if values else 0
    return v + _structure_bytes(M) + max(1 << 20, v // 16)


def _check(M, b, ref):
    """M's blocks are ref's (a dict of position -> values), by copy-out and by lookup; and its tree works."""
    import torch
    I, J, V = M.to_blocks()
    assert M.nblocks == len(ref)
    for i, j, v in zip(I.tolist(), J.tolist(), V):
        assert (v == ref[(i, j)]).all()
    got, found = M.get_blocks(I, J)
    assert found.all() and (got == V).all()
    torch.cuda.synchronize()


def test_truncation_to_few_blocks(qt, counting):
    import torch
    b, nb = 16, 2048
    M, pos, V = _random(qt, nb, 100000, b, 2)
    with torch.no_grad():
        V *= 1e-6
        keep = torch.tensor([5, 70000, len(pos) - 1], device="cuda")
        V[keep] = 1.0
    M = qt.build(nb * b, nb * b, b, 8 * b, (pos // nb).int(), (pos % nb).int(), V)
    before = counting.held()
    T, removed, _ = qt.truncate(M, 1.0)
    assert removed == len(pos) - 3
    assert counting.held() - before <= _allowed(T, b)
    at = pos[keep].tolist()
    _check(T, b, {(p // nb, p % nb): V[k].cpu().numpy() for p, k in zip(at, keep.tolist())})
    C = qt.multiply(T, M)                                   # the moved tree as an operand
    rows = {p % nb for p in at}
    assert C.stats()["products"] == sum(int(((pos // nb) == k).sum()) * sum(1 for p in at if p % nb == k) for k in rows)


def _band(nb, b, width, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    I = torch.arange(nb, device="cuda").repeat_interleave(width)
    J = I + torch.arange(width, device="cuda").repeat(nb)
    on = J < nb
    V = torch.randn((int(on.sum()), b, b), generator=g, dtype=torch.float64, device="cuda")
    return I[on].int(), J[on].int(), V


def test_band_of_full_leaves(qt, counting):
    """A narrow band over many block rows: few leaves and nodes, many positions.
    The matrix, its sum with itself and its symmetric structure."""
    b, nb = 16, 30000
    before = counting.held()
    lst = _band(nb, b, 3, 1)
    A = qt.build(nb * b, nb * b, b, 8 * b, *lst)
    assert counting.held() - before <= _allowed(A, b)
    before = counting.held()
    S = qt.add(A, A)
    assert counting.held() - before <= _allowed(S, b)
    I, J, V = S.to_blocks()
    assert (V == 2 * lst[2].cpu().numpy()).all() and (I == lst[0].cpu().numpy()).all() and (J == lst[1].cpu().numpy()).all()
    before = counting.held()
    C = qt.sysq(A)
    assert (C.levels() > 0).all()
    C.free()
    full = 2 * A.nblocks - nb                               # blocks of the full matrix
    assert counting.held() - before <= 12 * full + 60 * 3 * nb + (1 << 20)
    B = qt.sysq(S)                                          # 2 A: every block four times C's
    C = qt.sysq(A)
    for x, y in zip(B.to_blocks(), C.to_blocks()):
        assert (x == (4 * y if y.ndim == 3 else y)).all()


def test_empty_matrices_of_many_block_rows(qt, counting):
    """2^30 block rows and columns, no block: nothing is counted, held or summed
    over the positions, whatever is done with the matrix."""
    import numpy as np
    b, n = 16, 1 << 34
    none = (np.zeros(0, np.int32), np.zeros(0, np.int32), np.zeros((0, b, b)))
    before = counting.held()
    A = qt.build(n, n, b, 8 * b, *none)
    for C in (qt.multiply(A, A), qt.multiply_ex(A, A, trans_a=True, prec="f32"), qt.sysq(A), qt.add(A, A),
              qt.truncate(A, 1.0)[0]):
        assert C.nblocks == 0 and C.info()["n_rows"] == n
        assert qt.multiply(C, A).nblocks == 0
    plan = qt.Plan([A, A], [A, A], "f64")
    plan.execute()
    assert plan.result(1).nblocks == 0
    plan.destroy()
    assert counting.held() - before <= 1 << 20
