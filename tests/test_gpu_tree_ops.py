"""Sums, truncations and norms at the edges of their tiles (256 blocks per
workgroup), and the trees they form, against torch and a rebuild.

Sums of two entries, copies and kept blocks are exact; a tree is compared
through its levels and through a product with it, which a rebuilt matrix must
give bit for bit.
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


def _blocks(pos, nb, seed, b=16):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    V = torch.randn((len(pos), b, b), generator=g, dtype=torch.float64, device="cuda")
    p = torch.as_tensor(np.asarray(pos, np.int64), device="cuda")
    return (p // nb).int(), (p % nb).int(), V, p


def _out(qt, M):
    import torch
    n, b = M.nblocks, M.info()["b"]
    I = torch.empty(n, dtype=torch.int32, device="cuda")
    J = torch.empty_like(I)
    V = torch.empty((n, b, b), dtype=torch.float64, device="cuda")
    if n:
        M.to_blocks_device(I, J, V)
    return I, J, V


def _same_tree(qt, M, nb, b=16):
    """M's tree and values are those of a matrix built from its block list."""
    import torch
    I, J, V = _out(qt, M)
    R = qt.build(nb * b, nb * b, b, 8 * b, I, J, V)
    assert M.levels().tolist() == R.levels().tolist()
    for x, y in zip(_out(qt, qt.multiply(M, M)), _out(qt, qt.multiply(R, R))):
        assert torch.equal(x, y)


# blocks of A, of B, and of both: nothing in common, some, everything; tiles of
# 256 keys full, one short, one over
@pytest.mark.parametrize("na,nb,both", [(1, 1, 0), (1, 1, 1), (1, 0, 0), (0, 5, 0), (255, 10, 10), (256, 256, 100),
                                       (257, 1, 1), (512, 511, 511), (513, 700, 0), (2000, 3000, 1500),
                                       (4000, 4000, 4000)])
def test_add(qt, na, nb, both):
    import torch
    grid = 100
    print("add", na, nb, both, flush=True)
    pos = np.random.default_rng(na + nb).permutation(grid * grid)[:na + nb - both]
    pa, pb = pos[:na], pos[na - both:na - both + nb]
    Ia, Ja, Va, ka = _blocks(pa, grid, 1)
    Ib, Jb, Vb, kb = _blocks(pb, grid, 2)
    A, B = qt.build(1600, 1600, 16, 128, Ia, Ja, Va), qt.build(1600, 1600, 16, 128, Ib, Jb, Vb)
    S = qt.add(A, B)
    want = torch.zeros((grid * grid, 16, 16), dtype=torch.float64, device="cuda")
    seen = torch.zeros(grid * grid, dtype=torch.bool, device="cuda")
    for k, V in ((ka, Va), (kb, Vb)):
        want[k] += V
        seen[k] = True
    I, J, V = _out(qt, S)
    at = torch.nonzero(seen).reshape(-1)
    assert torch.equal(I.long() * grid + J, at) and torch.equal(V, want[at])
    _same_tree(qt, S, grid)


@pytest.mark.parametrize("n,cut", [(1, 0), (1, 1), (255, 17), (256, 256), (257, 256), (512, 1), (5000, 2500)])
def test_truncate(qt, n, cut):
    import torch
    grid = 100
    print("truncate", n, cut, flush=True)
    I, J, V, k = _blocks(np.random.default_rng(n).permutation(grid * grid)[:n], grid, n)
    V *= torch.logspace(0, -6, n, dtype=torch.float64, device="cuda")[:, None, None]
    n2 = V.square().sum((1, 2))
    o = torch.argsort(n2)
    sums = torch.cumsum(n2[o], 0)
    eps2 = 0.0 if cut == 0 else 2.0 * float(sums[-1]) if cut == n else 0.5 * float(sums[cut - 1] + sums[cut])
    T, removed, lost = qt.truncate(qt.build(1600, 1600, 16, 128, I, J, V), eps2 ** 0.5)
    assert removed == cut
    # each side sums cut * 256 squares, each within 2^-53 per operation of its exact value
    ref = float(sums[cut - 1]) if cut else 0.0
    assert abs(lost - ref) <= 2 * (cut * 256 + cut) * 2.0 ** -53 * ref
    keep = torch.ones(n, dtype=torch.bool, device="cuda")
    keep[o[:cut]] = False
    at = torch.argsort(k[keep])
    tI, tJ, tV = _out(qt, T)
    assert torch.equal(tI.long() * grid + tJ, k[keep][at]) and torch.equal(tV, V[keep][at])
    if cut < n:
        _same_tree(qt, T, grid)


@pytest.mark.parametrize("b", [16, 32, 64])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_norms(qt, b, prec):
    import torch
    grid = 30
    I, J, V, k = _blocks(np.random.default_rng(b).permutation(grid * grid)[:311], grid, b, b)
    M = qt.build(grid * b, grid * b, b, 8 * b, I, J, V)
    if prec == "f32":
        d = torch.arange(grid, dtype=torch.int32, device="cuda")
        M = qt.multiply(M, qt.build(grid * b, grid * b, b, 8 * b, d, d,
                                    torch.eye(b, dtype=torch.float64, device="cuda").repeat(grid, 1, 1)), "f32")
        V = V.float().double()
    bn, total = M.norms()
    n2 = V.square().sum((1, 2))[torch.argsort(k)].cpu().numpy()
    # b^2 squares on each side, added in some order
    assert (np.abs(bn - n2) <= 2 * (b * b + 1) * 2.0 ** -53 * n2).all()
    assert abs(total - n2.sum()) <= 2 * (b * b + 311) * 2.0 ** -53 * n2.sum()
