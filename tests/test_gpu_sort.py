"""The library's sorts (block keys at build, rows at copy-out, norms at
truncation) at the edges of their size classes, against torch's stable sorts.

Nothing is rounded on the way, so every comparison is exact.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1501_07800_amd as q
    return q


def _list(n, nbr, nbc, seed):
    """n distinct block positions of an nbr x nbc grid in random order, with
    values that name their block (entry 0: the position's number)."""
    import torch
    g = np.random.default_rng(seed)
    pos = np.array([], np.int64)
    while len(pos) < n:   # random samples until n are distinct (a full grid: all of it)
        pos = np.arange(n) if n == nbr * nbc else np.unique(np.concatenate([pos, g.integers(0, nbr * nbc, n)]))
    pos = g.permutation(pos)[:n]
    p = torch.from_numpy(pos).cuda()
    V = torch.zeros((n, 16, 16), dtype=torch.float64, device="cuda")
    V[:, 0, 0] = p.double() + 1.0
    V[:, 15, 15] = torch.rand(n, dtype=torch.float64, device="cuda")
    return p, (p // nbc).int(), (p % nbc).int(), V


# n: one wave, the one-launch sort's largest and one more, tiles' edges, two
# tile sizes; rows: one pass (up to 2048), two, three
@pytest.mark.parametrize("n,nbr,nbc", [(1, 1, 1), (2, 1, 70000), (63, 63, 1), (64, 8, 8), (65, 40, 40), (255, 3, 1000),
                                       (4095, 64, 64), (4096, 64, 64), (4097, 70, 60), (8192, 2048, 50),
                                       (8193, 2049, 50), (20000, 5000, 5), (7001, (1 << 22) + 1, 3),
                                       (448 * 1024, 1024, 1024), (448 * 1024 + 1, 700, 4096), ((1 << 19) + 1, 1024, 1024)])
def test_build_and_copy_out_order(qt, n, nbr, nbc):
    import torch
    print("sort", n, nbr, nbc, flush=True)
    p, I, J, V = _list(n, nbr, nbc, n)
    M = qt.build(nbr * 16, nbc * 16, 16, 128, I, J, V)
    assert M.nblocks == n
    order = torch.argsort(p)
    oI = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    oJ = torch.full_like(oI, -1)
    oV = torch.full((n, 16, 16), float("nan"), dtype=torch.float64, device="cuda")
    for copy in (M.to_blocks_device, M.to_blocks_noalloc):
        oI.fill_(-1), oJ.fill_(-1), oV.fill_(float("nan"))
        copy(oI, oJ, oV)
        assert torch.equal(oI, I[order]) and torch.equal(oJ, J[order]) and torch.equal(oV, V[order])
    bn, _ = M.norms()
    assert np.array_equal(bn, (V[order, 0, 0] ** 2 + V[order, 15, 15] ** 2).cpu().numpy())


@pytest.mark.parametrize("n", [2, 64, 4096, 4097, 9000])
def test_duplicate_and_range_errors(qt, n):
    p, I, J, V = _list(n, 100, 100, 5)
    I2, J2 = I.clone(), J.clone()
    I2[n - 1], J2[n - 1] = I[0], J[0]
    with pytest.raises(qt.QtError, match="duplicate"):
        qt.build(1600, 1600, 16, 128, I2, J2, V)
    I2 = I.clone()
    I2[n // 2] = 100
    with pytest.raises(qt.QtError, match="invalid argument"):
        qt.build(1600, 1600, 16, 128, I2, J, V)


def _morton(i, j):
    k = np.zeros(len(i), np.int64)
    for b in range(20):
        k |= ((i >> b) & 1) << (2 * b + 1) | ((j >> b) & 1) << (2 * b)
    return k


# blocks of few distinct norms (ties go by Morton position) and of many
@pytest.mark.parametrize("n,distinct", [(64, 3), (4096, 7), (4097, 7), (4097, 100000), (30000, 100000), (30000, 1)])
def test_truncation_order(qt, n, distinct):
    import torch
    print("truncate", n, distinct, flush=True)
    p, I, J, V = _list(n, 300, 300, n + distinct)
    V.zero_()
    w = torch.from_numpy(np.random.default_rng(1).integers(1, distinct + 1, n)).cuda()
    V[:, 3, 4] = 0.5 ** 10 * w.double()      # squares and their sums are exact in fp64
    M = qt.build(4800, 4800, 16, 128, I, J, V)
    n2 = (V[:, 3, 4] ** 2).cpu().numpy()
    i, j = I.cpu().numpy().astype(np.int64), J.cpu().numpy().astype(np.int64)
    o = np.lexsort((_morton(i, j), n2))
    sums = np.cumsum(n2[o])
    cut = n // 3
    eps = float(np.sqrt(0.5 * (sums[cut - 1] + sums[cut])))
    T, removed, lost = qt.truncate(M, eps)
    assert removed == cut and lost == sums[cut - 1]
    keep = np.sort(p.cpu().numpy()[o[cut:]])
    tI, tJ, _ = T.to_blocks()
    assert np.array_equal(tI.astype(np.int64) * 300 + tJ, keep)
