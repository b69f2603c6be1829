"""C leaves of few block products (leaves of 8 x 8 blocks, a lane per leaf pair)
against the leaf step that walks the pairs of one leaf per wave, which leaves of
4 x 4 blocks take: the block products and their order do not depend on the
leaf, so the results are bitwise the same. And C's tree against its blocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
B = 16


@pytest.fixture(scope="module")
def qt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1501_07800_amd as q
    return q


def _positions(kind, rows, cols, n, r):
    if kind == "hub":          # a few dense rows and columns, and dense leaves: leaves of over 64 products
        m = r.random((rows, cols)) < n / (rows * cols)
        m[:: rows // 3] = True
        m[:, :: cols // 3] |= r.random((rows, 1)) < 0.5
        m[16:24, 40:48] = True
        m[40:48, 16:24] = True
        return np.flatnonzero(m)
    if kind == "lanes":        # A in the columns, B in the rows 0 mod 8: many leaf pairs, all with products
        i, j = np.divmod(np.arange(rows * cols), cols)
        return np.flatnonzero((j % 8 == 0) & (i % 8 == 3)) if n else np.flatnonzero((i % 8 == 0) & (j % 8 == 5))
    if kind == "miss":         # the same with rows 1 mod 8: leaf pairs, no product but on a corner
        i, j = np.divmod(np.arange(rows * cols), cols)
        k = (j % 8 == 0) & (i % 8 == 3) if n else (i % 8 == 1) & (j % 8 == 5)
        return np.flatnonzero(k | ((i < 3) & (j < 3)))
    if kind == "rmat":
        s = max(rows, cols).bit_length()
        q = r.choice(4, size=(3 * n, s), p=[0.55, 0.15, 0.15, 0.15])
        w = 1 << np.arange(s - 1, -1, -1)
        i, j = ((q >> 1) * w).sum(1), ((q & 1) * w).sum(1)
        return np.unique((i * cols + j)[(i < rows) & (j < cols)])[:]
    return np.sort(r.choice(rows * cols, size=n, replace=False))


def _pair(qt, rows, cols, pos, seed):
    import torch
    I, J = (torch.as_tensor(x.astype(np.int32), device="cuda") for x in np.divmod(pos, cols))
    V = torch.as_tensor(np.random.default_rng(seed).standard_normal((len(pos), B, B)), device="cuda")
    return [qt.build(rows * B, cols * B, B, lb * B, I, J, V) for lb in (8, 4)]


def _blocks(M):
    import torch
    I = torch.empty(M.nblocks, dtype=torch.int32, device="cuda")
    J = torch.empty_like(I)
    V = torch.empty((M.nblocks, B, B), dtype=torch.float64, device="cuda")
    M.to_blocks_device(I, J, V)
    return I, J, V


# rows, inner, columns; blocks of A and B. Waves of one leaf and of many, leaf
# pairs up to and beyond 64 of a leaf, products up to and beyond 64 of a leaf,
# ragged edges, lifted operands
@pytest.mark.parametrize("kind,m,k,n,na,nb", [
    ("random", 200, 200, 200, 1500, 1500), ("random", 333, 1000, 257, 6000, 5000),
    ("random", 1000, 1000, 1000, 9000, 9000), ("random", 700, 3000, 650, 30000, 30000),
    ("random", 3000, 3000, 3000, 9000, 9000), ("random", 4090, 4090, 4090, 30000, 30000),
    ("random", 9, 4000, 2000, 9000, 20000), ("lanes", 640, 640, 640, 1, 0), ("miss", 640, 640, 640, 1, 0),
    ("hub", 700, 700, 700, 2000, 2000), ("rmat", 2048, 2048, 2048, 6000, 6000), ("rmat", 900, 1500, 1100, 3000, 3000)])
@pytest.mark.parametrize("ta,tb", [(False, False), (True, True)])
def test_same_as_one_leaf_per_wave(qt, kind, m, k, n, na, nb, ta, tb):
    import torch
    print("sparse", kind, m, k, n, na, nb, ta, tb, flush=True)
    r = np.random.default_rng(7)
    pa, pb = _positions(kind, m, k, na, r), _positions(kind, k, n, nb, r)
    if ta:
        pa = np.sort(pa % k * m + pa // k)
    if tb:
        pb = np.sort(pb % n * k + pb // n)
    A, Bm = _pair(qt, *((k, m) if ta else (m, k)), pa, 1), _pair(qt, *((n, k) if tb else (k, n)), pb, 2)
    C, ref = (qt.multiply_ex(a, b, trans_a=ta, trans_b=tb, prec="f64") for a, b in zip(A, Bm))
    assert C.nblocks == ref.nblocks > 0 and C.stats()["products"] == ref.stats()["products"]
    got, want = _blocks(C), _blocks(ref)
    for x, y in zip(got, want):
        assert torch.equal(x, y)
    I, J = (x.cpu().numpy().astype(np.int64) for x in got[:2])
    levels = C.levels().tolist()
    for l, nodes in enumerate(reversed(levels)):
        side = 8 << l
        assert nodes == len(np.unique((I // side) * (1 << 20) + J // side))
