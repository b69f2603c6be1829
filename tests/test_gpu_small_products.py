"""Products small enough for the one-launch symbolic phase, and just too large
for it, against the level-by-level phase: the same blocks in the top-left
corner of a much larger grid take more quadtree levels than the small path has,
and must give bitwise the same blocks, the same counters and the same tree
below the added levels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
GRID = 4096    # blocks a side: nine levels above leaves of 8 x 8


@pytest.fixture(scope="module")
def qt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1501_07800_amd as q
    return q


def _positions(kind, rows, cols, seed):
    r = np.random.default_rng(seed)
    if kind == "dense":
        return np.arange(rows * cols)
    if kind == "banded":
        i, j = np.divmod(np.arange(rows * cols), cols)
        return np.flatnonzero(np.abs(i - j) <= 3)
    if kind == "corner":      # leaves whose pairs all miss: NIL leaves and nodes of C
        i, j = np.divmod(np.arange(rows * cols), cols)
        return np.flatnonzero((j % 8 == 0) & (i % 3 == 0) if seed % 2 else (i % 8 == 5) & (j % 5 == 0))
    return np.sort(r.choice(rows * cols, size=max(1, int(float(kind) * rows * cols)), replace=False))


def _pair(qt, rows, cols, kind, seed, lb, upper=False, b=16):
    import torch
    pos = _positions(kind, rows, cols, seed)
    I, J = pos // cols, pos % cols
    if upper:
        I, J = I[I <= J], J[I <= J]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    V = torch.randn((len(I), b, b), generator=g, dtype=torch.float64, device="cuda")
    I, J = (torch.as_tensor(x.astype(np.int32), device="cuda") for x in (I, J))
    return [qt.build(m * b, n * b, b, lb * b, I, J, V) for m, n in ((rows, cols), (GRID, GRID))]


def _same(a, b):
    import torch
    assert a.nblocks == b.nblocks and a.stats()["products"] == b.stats()["products"]
    la, lb = a.levels().tolist(), b.levels().tolist()
    assert la == lb[len(lb) - len(la):]
    pa, pb = a.stats()["pairs"].tolist(), b.stats()["pairs"].tolist()
    assert pa == pb[len(pb) - len(pa):]
    n = a.nblocks
    if not n:
        return
    out = []
    for M in (a, b):
        I = torch.empty(n, dtype=torch.int32, device="cuda")
        J = torch.empty_like(I)
        V = torch.empty((n, 16, 16), dtype=torch.float64, device="cuda")
        M.to_blocks_device(I, J, V)
        out.append((I, J, V))
    for x, y in zip(*out):
        assert torch.equal(x, y)


# one leaf; one to four levels; C nodes up to the 256 of the small path and
# beyond; 20000 products (dense 27 x 27 blocks have 19683, 28 x 28 21952);
# 512 pairs of a level (dense leaves of one block: 8 x 8 x 8 pairs, 9 x 9 x 9)
@pytest.mark.parametrize("kind,m,k,n,lb", [("dense", 1, 1, 1, 8), ("dense", 8, 8, 8, 8), ("dense", 9, 8, 7, 8),
                                           ("dense", 27, 27, 27, 8), ("dense", 28, 28, 28, 8), ("dense", 8, 8, 8, 1),
                                           ("dense", 9, 9, 9, 1), ("dense", 16, 2, 15, 1), ("dense", 14, 3, 13, 2),
                                           ("banded", 32, 32, 32, 8), ("banded", 100, 100, 100, 8),
                                           ("banded", 40, 40, 40, 2), ("0.1", 60, 50, 40, 8), ("0.05", 64, 64, 64, 8),
                                           ("0.03", 120, 100, 110, 8), ("0.02", 37, 300, 5, 4), ("corner", 64, 64, 64, 8),
                                           ("corner", 40, 40, 40, 4)])
def test_same_as_levels(qt, kind, m, k, n, lb):
    print("small", kind, m, k, n, lb, flush=True)
    for ta, tb in ((False, False), (True, False), (False, True), (True, True)):
        A = _pair(qt, *((k, m) if ta else (m, k)), kind, 1, lb)
        B = _pair(qt, *((n, k) if tb else (k, n)), kind, 2, lb)
        _same(*[qt.multiply_ex(x, y, trans_a=ta, trans_b=tb) for x, y in zip(A, B)])
        if not (ta or tb):
            _same(*[qt.multiply_tau(x, y, 250.0) for x, y in zip(A, B)])   # some products are below, some above


@pytest.mark.parametrize("kind,n,lb", [("dense", 1, 8), ("dense", 20, 8), ("banded", 50, 4), ("0.1", 60, 8), ("0.3", 12, 1)])
def test_symmetric_and_upper(qt, kind, n, lb):
    print("small upper", kind, n, lb, flush=True)
    A = _pair(qt, n, n, kind, 3, lb, upper=True)
    _same(*[qt.sysq(x) for x in A])
    A = _pair(qt, n, n, kind, 4, lb)
    _same(*[qt.multiply_ex(x, x, upper=True) for x in A])
