"""Counts at which one grid of a thread (or wave) per unit would pass 2^32
threads, the most a grid has: 2^26 C blocks of 16 x 16, and operands of 2^32
entries. Small whole numbers, so that fp32 (and the split) is exact."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.slow]


def _room(gib):
    import torch
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (gib << 30):
        pytest.skip(f"needs {gib} GiB of free device memory")


def _outer(qt, m, n, b, leaf):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    i = [torch.arange(x, dtype=torch.int32, device="cuda") for x in (m, n)]
    VA, VB = (torch.randint(-3, 4, (x, b, b), generator=g, device="cuda").double() for x in (m, n))
    A = qt.build(m * b, b, b, leaf, i[0], torch.zeros_like(i[0]), VA)
    B = qt.build(b, n * b, b, leaf, torch.zeros_like(i[1]), i[1], VB)
    return A, B, VA.float(), VB.float()


def _check_outer(C, VA, VB, out):
    import torch
    m, n, b = len(VA), len(VB), VA.shape[1]
    assert C.nblocks == m * n
    I, J, V = out
    V.fill_(float("nan"))
    C.to_blocks_device(I, J, V, "f32")
    t = torch.arange(m * n, device="cuda")
    placed = torch.equal(I, (t // n).int()) and torch.equal(J, (t % n).int())
    assert placed
    del t
    for i in range(m):
        same = torch.equal(V[i * n:(i + 1) * n], torch.matmul(VA[i], VB))
        assert same, i


def test_products_of_many_blocks(qt):
    """The numeric kernels, a plan's flat grid, and the block norms."""
    import torch
    _room(170)
    b, m, n = 16, 8200, 8200
    assert m * n > 2 ** 26
    A, B, VA, VB = _outer(qt, m, n, b, 8 * b)
    out = (torch.empty(m * n, dtype=torch.int32, device="cuda"), torch.empty(m * n, dtype=torch.int32, device="cuda"),
           torch.empty((m * n, b, b), dtype=torch.float32, device="cuda"))
    print("multiply", flush=True)
    C = qt.multiply(A, B, "f32")
    _check_outer(C, VA, VB, out)
    print("norms", flush=True)
    n2, _ = C.norms()
    want = torch.cat([x.double().square().sum((1, 2)) for x in out[2].split(1 << 20)])
    same = np.array_equal(n2, want.cpu().numpy())          # whole numbers: exact in any order
    assert same
    C.free()
    print("plan", flush=True)
    plan = qt.Plan([A], [B], "f32")
    plan.set_schedule("flat")
    plan.execute(graph=False)
    _check_outer(plan.result(0), VA, VB, out)
    plan.destroy()
    del out, want
    torch.cuda.empty_cache()


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
def test_operands_of_many_entries(qt, prec):
    """The fp32 copy and the bf16 split of an operand of more than 2^32 entries."""
    import torch
    _room(150)
    b, nb = 64, (1 << 20) + 1000
    assert nb * b * b > 2 ** 32
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    V = torch.empty((nb, b, b), dtype=torch.float64, device="cuda")
    for part in V.split(1 << 16):
        part.copy_(torch.randint(-3, 4, part.shape, generator=g, device="cuda"))
    d = torch.arange(nb, dtype=torch.int32, device="cuda")
    A = qt.build(nb * b, nb * b, b, b, d, d, V)
    print("square", prec, flush=True)
    C = qt.multiply(A, A, prec)
    at = torch.cat([torch.arange(3), torch.arange(nb - 1500, nb)])
    got, found = C.get_blocks(at.numpy(), at.numpy(), "f64")
    assert found.all()
    x = V[at.cuda()]
    same = np.array_equal(got, torch.bmm(x, x).cpu().numpy())
    assert same
    C.free()
    A.free()
    del V
    torch.cuda.empty_cache()


def test_more_nodes_than_waves_are_refused(qt):
    """67.2 M C leaves, of one block each: a wave per leaf is more than a grid
    holds, and the call says so before it launches anything."""
    A, B, _, _ = _outer(qt, 8200, 8200, 16, 16)
    for call in (lambda: qt.multiply(A, B, "f32"), lambda: qt.Plan([A], [B], "f32")):
        with pytest.raises(qt.QtError) as e:
            call()
        assert e.value.status == qt.QT_ERR_UNSUPPORTED
