"""Numeric launches around the sizes where the run length of tiles per XCD
changes: every C block is computed once, whatever the number of C blocks.

A is block diagonal, so C = A A has one product per C block. Both the kernel
and the reference sum b products per entry, each within b 2^-53 (|A||A|) of
the exact value, so they differ by at most twice that.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1501_07800_amd as q
    return q


def _diag(qt, n, b, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    I = torch.arange(n, dtype=torch.int32, device="cuda")
    V = torch.randn((n, b, b), generator=g, dtype=torch.float64, device="cuda")
    return qt.build(n * b, n * b, b, 8 * b, I, I, V), V


def _check(C, V, n, b):
    import torch
    I = torch.empty(n, dtype=torch.int32, device="cuda")
    J = torch.empty_like(I)
    W = torch.empty((n, b, b), dtype=torch.float64, device="cuda")
    C.to_blocks_device(I, J, W)
    assert torch.equal(I, torch.arange(n, dtype=torch.int32, device="cuda")) and torch.equal(I, J)
    bound = 2 * b * 2.0 ** -53 * torch.bmm(V.abs(), V.abs())
    assert bool(((W - torch.bmm(V, V)).abs() <= bound).all())


@pytest.mark.parametrize("b,n", [(16, n) for n in (1, 7, 8, 9, 255, 256, 257, 8191, 8193, 65535, 65537, 131071, 131073)] +
                         [(32, 511), (32, 513), (32, 16385), (64, 1), (64, 31), (64, 257), (64, 8193)])
def test_every_block_once(qt, b, n):
    print("runs", b, n, flush=True)
    A, V = _diag(qt, n, b, n)
    _check(qt.multiply(A, A), V, n, b)
    _check(qt.multiply_ex(A, A), V, n, b)


@pytest.mark.parametrize("b,sizes", [(16, (1, 130, 255)), (32, (63, 1, 64)), (64, (3, 260))])
def test_every_block_of_a_plan_once(qt, b, sizes):
    print("plan", b, sizes, flush=True)
    mats = [_diag(qt, n, b, n) for n in sizes]
    plan = qt.Plan([m for m, _ in mats], [m for m, _ in mats])
    plan.execute(graph=False)
    for i, (_, V) in enumerate(mats):
        _check(plan.result(i), V, sizes[i], b)
