"""BF16X3 launches at b = 64 around the sizes where the run length per XCD
changes (40 C blocks and its doublings): every C block is computed once, by
the plain, the transposed and the batch kernel. Block diagonal operands of
small whole numbers, which the split holds exactly, so the result is exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 39, 40, 41, 79, 80, 81, 639, 640, 641, 5119, 5121, 10239, 10241])
def test_every_block_once(qt, n):
    import torch
    b = 64
    print("runs", n, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    d = torch.arange(n, dtype=torch.int32, device="cuda")
    V = torch.randint(-3, 4, (n, b, b), generator=g, device="cuda").double()
    A = qt.build(n * b, n * b, b, 8 * b, d, d, V)
    plan = qt.Plan([A], [A], "bf16x3")
    plan.execute(graph=False)
    for C, X in ((qt.multiply(A, A, "bf16x3"), V), (plan.result(0), V),
                 (qt.multiply_ex(A, A, trans_a=True, prec="bf16x3"), V.transpose(1, 2).contiguous())):
        I = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        J = torch.full_like(I, -1)
        W = torch.full((n, b, b), float("nan"), dtype=torch.float64, device="cuda")
        C.to_blocks_device(I, J, W)
        assert torch.equal(I, d) and torch.equal(J, d)
        same = torch.equal(W, torch.bmm(X, V))
        assert same
    plan.destroy()
