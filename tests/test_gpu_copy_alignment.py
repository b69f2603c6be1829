"""Copy-outs beyond the one-launch size, and builds of as many blocks, with
caller arrays at every alignment of their entries (16 bytes and no more among
them, where four fp64 entries take 32): exact copies, fp64 to fp32 rounded to
nearest even as torch's cast does."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,n", [(16, 4097), (32, 4100)])
@pytest.mark.parametrize("offset", [0, 1, 2, 3, 4, 6])
def test_alignments(qt, b, n, offset):
    import torch
    print("copy", b, n, offset, flush=True)
    nb = 128
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    flat = torch.randn(n * b * b + 8, generator=g, dtype=torch.float64, device="cuda")
    V = flat[offset:offset + n * b * b].view(n, b, b)
    pos = torch.randperm(nb * nb, generator=g, device="cuda")[:n]
    M = qt.build(nb * b, nb * b, b, 4 * b, (pos // nb).int(), (pos % nb).int(), V)
    d = torch.arange(nb, device="cuda").int()
    E = qt.build(nb * b, nb * b, b, 4 * b, d, d, torch.eye(b, dtype=torch.float64, device="cuda").repeat(nb, 1, 1))
    C = qt.multiply(M, E, "f32")                     # M's blocks rounded to fp32, stored in fp32
    want = V[torch.argsort(pos)]
    for H, ref in ((M, want), (C, want.float().double())):
        for dtype, name in ((torch.float64, "f64"), (torch.float32, "f32")):
            out = torch.full((n * b * b + 8,), 7.0, dtype=dtype, device="cuda")
            W = out[offset:offset + n * b * b].view(n, b, b)
            oI = torch.empty(n, dtype=torch.int32, device="cuda")
            oJ = torch.empty_like(oI)
            H.to_blocks_device(oI, oJ, W, name)
            assert torch.equal(W, ref.to(dtype))
            assert torch.equal(oI.long() * nb + oJ, torch.sort(pos)[0])
            assert bool((out[:offset] == 7).all()) and bool((out[offset + n * b * b:] == 7).all())
