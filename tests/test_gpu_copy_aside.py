"""A large copy-out whose sort runs beside work queued on the caller's stream:
the same arrays as from an idle stream, whichever stream it is given and
whatever lies queued there, the output arrays still in use by earlier work
included; and under capture."""
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


@pytest.mark.parametrize("n", [16383, 16384, 20000])    # 128 MiB of values from 16384 blocks of 32 on
@pytest.mark.parametrize("own_stream", [False, True])
def test_beside_queued_work(qt, n, own_stream):
    import torch
    b, nb = 32, 300
    r = np.random.default_rng(n)
    pos = r.choice(nb * nb, size=n, replace=False)
    I, J = (torch.as_tensor(x.astype(np.int32), device="cuda") for x in np.divmod(pos, nb))
    V = torch.randn((n, b, b), dtype=torch.float64, device="cuda")
    M = qt.build(nb * b, nb * b, b, 8 * b, I, J, V)
    o = torch.as_tensor(np.argsort(pos), device="cuda")
    wI, wJ, wV = I[o], J[o], V[o]
    big = torch.randn(6144, 6144, device="cuda")
    torch.cuda.synchronize()
    s = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    with torch.cuda.stream(s):
        for _ in range(3):
            oI, oJ = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
            oV = torch.zeros_like(V)
            for _ in range(6):
                big @ big
            before = (oI + 0, oJ + 0)          # reads the arrays before the copy-out writes them
            M.to_blocks_device(oI, oJ, oV, stream=s)
            after = (oI + 0, oJ + 0, oV + 0)
            oI.fill_(-2)
            s.synchronize()
            assert bool((before[0] == -1).all()) and bool((before[1] == -1).all())
            assert torch.equal(after[0], wI) and torch.equal(after[1], wJ) and torch.equal(after[2], wV)


def test_under_capture(qt):
    import torch
    b, nb, n = 32, 300, 20000
    r = np.random.default_rng(1)
    pos = r.choice(nb * nb, size=n, replace=False)
    I, J = (torch.as_tensor(x.astype(np.int32), device="cuda") for x in np.divmod(pos, nb))
    V = torch.randn((n, b, b), dtype=torch.float64, device="cuda")
    M = qt.build(nb * b, nb * b, b, 8 * b, I, J, V)
    o = torch.as_tensor(np.argsort(pos), device="cuda")
    oI, oJ = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    oV = torch.zeros_like(V)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        M.to_blocks_noalloc(oI, oJ, oV, stream=s)
    for k in range(3):
        oI.fill_(-1)
        oV.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(oI, I[o]) and torch.equal(oJ, J[o]) and torch.equal(oV, V[o])
