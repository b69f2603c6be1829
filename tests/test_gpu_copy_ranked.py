"""Row-major copy-out around the size up to which every block finds its place by
itself: coordinates in row-major order, values exact, whatever the alignment of
the caller's array, with and without the library's fixed scratch, pattern only."""
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


@pytest.mark.parametrize("b,nb,n", [(16, 1, 1), (16, 3, 9), (16, 64, 63), (16, 64, 257), (16, 300, 4095), (16, 300, 4096),
                                    (16, 300, 4097), (16, 2100, 4096), (16, 2100, 4097), (32, 64, 4096), (32, 70, 4097),
                                    (64, 80, 4096), (64, 80, 4097)])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_row_major(qt, b, nb, n, offset):
    import torch
    print("ranked", b, nb, n, offset, flush=True)
    r = np.random.default_rng(n + nb)
    pos = r.choice(nb * nb, size=n, replace=False)
    I, J = (torch.as_tensor(x.astype(np.int32), device="cuda") for x in np.divmod(pos, nb))
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    V = torch.randn((n, b, b), generator=g, dtype=torch.float64, device="cuda")
    M = qt.build(nb * b, nb * b, b, 8 * b, I, J, V)
    o = torch.as_tensor(np.argsort(pos), device="cuda")
    for dtype, name in ((torch.float64, "f64"), (torch.float32, "f32")):
        for copy in (M.to_blocks_device, M.to_blocks_noalloc):
            out = torch.full((n * b * b + 8,), 7.0, dtype=dtype, device="cuda")
            W = out[offset:offset + n * b * b].view(n, b, b)
            oI, oJ = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
            copy(oI, oJ, W, name)
            assert torch.equal(oI, I[o]) and torch.equal(oJ, J[o]) and torch.equal(W, V[o].to(dtype))
            assert bool((out[:offset] == 7).all()) and bool((out[offset + n * b * b:] == 7).all())
    oI, oJ = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    M.to_blocks_noalloc(oI, oJ, None)
    assert torch.equal(oI, I[o]) and torch.equal(oJ, J[o])


@pytest.mark.parametrize("b,nb", [(16, 4096), (16, 4097), (32, 4100), (64, 4097)])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_fp32_values(qt, b, nb, offset):
    """A product stored in fp32 (a block diagonal matrix times the identity), both
    output types, on both sides of the size."""
    import torch
    print("ranked fp32", b, nb, offset, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(nb)
    V = torch.randn((nb, b, b), generator=g, dtype=torch.float64, device="cuda")
    I = torch.arange(nb, dtype=torch.int32, device="cuda")
    J = torch.randperm(nb, generator=g, device="cuda").int()
    E = torch.eye(b, dtype=torch.float64, device="cuda").repeat(nb, 1, 1)
    C = qt.multiply(qt.build(nb * b, nb * b, b, 8 * b, I, J, V), qt.build(nb * b, nb * b, b, 8 * b, I, I, E), "f32")
    for dtype, name in ((torch.float64, "f64"), (torch.float32, "f32")):
        out = torch.full((nb * b * b + 8,), 7.0, dtype=dtype, device="cuda")
        W = out[offset:offset + nb * b * b].view(nb, b, b)
        oI, oJ = (torch.full((nb,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        C.to_blocks_device(oI, oJ, W, name)
        assert torch.equal(oI, I) and torch.equal(oJ, J) and torch.equal(W, V.float().to(dtype))
        assert bool((out[:offset] == 7).all()) and bool((out[offset + nb * b * b:] == 7).all())
