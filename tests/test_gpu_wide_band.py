"""Bands over many block rows, fewer than two products per C block: a sort of C's
blocks by inner index would gain nothing, and none is made beyond 16384 inner
blocks (the widest that is, and the next, against the definition)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [16384, 16385, 20000])
def test_band(qt, nb):
    import torch
    b = 32
    g = torch.Generator(device="cuda")
    g.manual_seed(nb)
    I = torch.arange(nb, device="cuda").repeat_interleave(3)
    J = I + torch.arange(3, device="cuda").repeat(nb)
    I, J = I[J < nb], J[J < nb]
    V = torch.randint(-3, 4, (len(I), b, b), generator=g, device="cuda").double()
    A = qt.build(nb * b, nb * b, b, 8 * b, I.int(), J.int(), V)
    C = qt.multiply(A, A)
    assert 2 * C.stats()["products"] * b * b * 8 >= 700 << 20 and C.stats()["products"] < 2 * C.nblocks
    n = C.nblocks
    oI = torch.empty(n, dtype=torch.int32, device="cuda")
    oJ = torch.empty_like(oI)
    oV = torch.empty((n, b, b), dtype=torch.float64, device="cuda")
    C.to_blocks_device(oI, oJ, oV)
    D = torch.zeros((nb + 4, 3, b, b), dtype=torch.float64, device="cuda")     # A(i, i + d)
    D[I, J - I] = V
    want = torch.zeros((nb, 5, b, b), dtype=torch.float64, device="cuda")      # C(i, i + d), whole numbers: exact
    for d in range(3):
        for e in range(3):
            want[:, d + e] += torch.bmm(D[:nb, d], D[d:nb + d, e])
    d = (oJ - oI).long()
    assert n == 5 * nb - 10 and bool(((d >= 0) & (d < 5)).all())
    same = torch.equal(oV, want[oI.long(), d])
    assert same
