"""Copy-out and build with caller arrays at every alignment, both value types
in and out: copies are exact, fp64 to fp32 rounds to nearest even as torch's
cast does."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1501_07800_amd as q
    return q


@pytest.mark.parametrize("b", [16, 32, 64])
@pytest.mark.parametrize("n", [1, 3, 17, 64])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_alignments(qt, b, n, offset):
    import torch
    print("copy", b, n, offset, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    flat = torch.randn(n * b * b + 8, generator=g, dtype=torch.float64, device="cuda")
    V = flat[offset:offset + n * b * b].view(n, b, b)
    o = torch.randperm(n, generator=g, device="cuda")
    I = o.int()
    M = qt.build(n * b, n * b, b, 4 * b, I, I, V)
    identity = torch.eye(b, dtype=torch.float64, device="cuda").repeat(n, 1, 1)
    E = qt.build(n * b, n * b, b, 4 * b, I, I, identity)
    C = qt.multiply(M, E, "f32")                     # M's blocks rounded to fp32, stored in fp32
    want = torch.empty_like(V)
    want[o] = V
    for H, ref in ((M, want), (C, want.float().double())):
        for dtype, name in ((torch.float64, "f64"), (torch.float32, "f32")):
            out = torch.full((n * b * b + 8,), 7.0, dtype=dtype, device="cuda")
            W = out[offset:offset + n * b * b].view(n, b, b)
            oI = torch.empty(n, dtype=torch.int32, device="cuda")
            oJ = torch.empty_like(oI)
            H.to_blocks_device(oI, oJ, W, name)
            assert torch.equal(W, ref.to(dtype))
            assert bool((out[:offset] == 7).all()) and bool((out[offset + n * b * b:] == 7).all())
