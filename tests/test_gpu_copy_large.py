"""A copy-out of more than 2^32 lanes' work at one entry per lane: 69 GB of
fp32 blocks into an array that is not aligned to 16 bytes."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.slow]


def test_unaligned_beyond_one_grid(qt):
    import torch
    b, m, n = 64, 2048, 2049                 # 4.2 M blocks of 64 x 64
    if torch.cuda.mem_get_info()[0] < (160 << 30):
        pytest.skip("needs 160 GB of free device memory")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    zm, zn = torch.zeros(m, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    am, an = torch.arange(m, dtype=torch.int32, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda")
    VA = torch.randn((m, b, b), generator=g, dtype=torch.float64, device="cuda")
    VB = torch.randn((n, b, b), generator=g, dtype=torch.float64, device="cuda")
    A = qt.build(m * b, b, b, b, am, zm, VA)
    B = qt.build(b, n * b, b, b, zn, an, VB)
    C = qt.multiply(A, B, "f32")
    N = C.nblocks
    assert N == m * n and N * b * b // 4 > 2 ** 32          # lanes of a copy of four entries each
    flat = torch.full((N * b * b + 1,), float("nan"), dtype=torch.float32, device="cuda")
    V = flat[1:].view(N, b, b)
    I = torch.full((N,), -1, dtype=torch.int32, device="cuda")
    J = torch.full_like(I, -1)
    print("copy-out of", N * b * b * 4, "bytes", flush=True)
    C.to_blocks_device(I, J, V, "f32")
    torch.cuda.synchronize()
    t = torch.arange(N, device="cuda")
    assert torch.equal(I.long(), t // n) and torch.equal(J.long(), t % n)
    for part in V.split(N // 16 + 1):
        assert not bool(torch.isnan(part).any())
    at = torch.cat([torch.tensor([0, 1, N // 2, N - 2, N - 1]), torch.randint(0, N, (400,))])
    got, found = C.get_blocks((at // n).numpy(), (at % n).numpy(), "f32")
    assert found.all()
    assert np.array_equal(got, V[at.cuda()].cpu().numpy())
    del flat, V
    C.free()
    torch.cuda.empty_cache()
