"""Quadtree levels of few pairs per C node (a lane per pair) against the kernels
that take a node per wave, which the problems of a plan run: bitwise the same
blocks, trees and counters. And against exact integer products on the CPU, also
for levels wider than a plan's problems share launches for."""
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
    if kind == "rmat":
        s = max(rows, cols).bit_length()
        q = r.choice(4, size=(3 * n, s), p=[0.55, 0.15, 0.15, 0.15])
        w = 1 << np.arange(s - 1, -1, -1)
        i, j = ((q >> 1) * w).sum(1), ((q & 1) * w).sum(1)
        return np.unique((i * cols + j)[(i < rows) & (j < cols)])
    if kind == "bands":        # long runs of pairs in some nodes, one in the others
        i, j = np.divmod(np.arange(rows * cols), cols)
        return np.flatnonzero(((i // 16) % 9 == 0) & (i % 16 == 3) & (j % 4 == 1) | (i == j % rows) & (j % 16 == 0))
    return np.sort(r.choice(rows * cols, size=n, replace=False))


# rows, inner, columns; blocks of A and B: 8192 C node positions on the last
# tree level and up, nodes of one pair and of more than a wave's 64
@pytest.mark.parametrize("kind,m,k,n,na,nb,ta,tb", [
    ("random", 1450, 1450, 1450, 3000, 3000, False, False), ("random", 1500, 1500, 1500, 9000, 9000, True, False),
    ("random", 1300, 5000, 2040, 20000, 30000, False, True), ("bands", 1456, 1456, 1456, 0, 0, False, False),
    ("random", 2048, 300, 2048, 9000, 9000, False, False), ("rmat", 2040, 2040, 2040, 8000, 8000, True, True),
    ("rmat", 1500, 4000, 1900, 9000, 9000, False, False), ("random", 4090, 4090, 4090, 16000, 16000, False, False),
    ("rmat", 8192, 8192, 8192, 9000, 9000, False, False)])
def test_levels(qt, kind, m, k, n, na, nb, ta, tb):
    import scipy.sparse as sp
    import torch
    print("levels", kind, m, k, n, na, nb, ta, tb, flush=True)
    r = np.random.default_rng(11)
    mats, bsr = [], []
    for rows, cols, cnt, tr in ((m, k, na, ta), (k, n, nb, tb)):
        pos = _positions(kind, rows, cols, cnt, r)
        V = r.integers(-8, 9, size=(len(pos), B, B)).astype(np.float64)
        V[:, 0, 0] = 1e6           # no block of C cancels to zero
        I, J = np.divmod(pos, cols)
        ptr = np.searchsorted(I, np.arange(rows + 1))
        bsr.append(sp.bsr_matrix((V, J, ptr), shape=(rows * B, cols * B)))
        if tr:
            o = np.lexsort((I, J))
            I, J, V, rows, cols = J[o], I[o], V[o].transpose(0, 2, 1).copy(), cols, rows
        I, J, V = torch.as_tensor(I.astype(np.int32)), torch.as_tensor(J.astype(np.int32)), torch.as_tensor(V)
        mats.append(qt.build(rows * B, cols * B, B, 8 * B, I.cuda(), J.cuda(), V.cuda()))
    C = qt.multiply_ex(*mats, trans_a=ta, trans_b=tb, prec="f64")
    ref = (bsr[0] @ bsr[1]).tobsr((B, B))
    ref.sort_indices()
    I = torch.empty(C.nblocks, dtype=torch.int32, device="cuda")
    J = torch.empty_like(I)
    V = torch.empty((C.nblocks, B, B), dtype=torch.float64, device="cuda")
    C.to_blocks_device(I, J, V)
    gi, gj = I.cpu().numpy(), J.cpu().numpy()
    assert C.nblocks == len(ref.indices)
    assert np.array_equal(gj, ref.indices) and np.array_equal(gi, np.repeat(np.arange(m), np.diff(ref.indptr)))
    assert np.array_equal(V.cpu().numpy(), ref.data)
    if ta or tb or max(m, n) > 2048:
        return
    plan = qt.Plan([mats[0]], [mats[1]], "f64")
    plan.execute(graph=False)
    D = plan.result(0)
    a, b = C.stats(), D.stats()
    assert a["products"] == b["products"] and a["pairs"].tolist() == b["pairs"].tolist()
    assert C.levels().tolist() == D.levels().tolist() and D.nblocks == C.nblocks
    I2, J2, V2 = torch.empty_like(I), torch.empty_like(J), torch.empty_like(V)
    D.to_blocks_device(I2, J2, V2)
    assert torch.equal(I, I2) and torch.equal(J, J2) and torch.equal(V, V2)
