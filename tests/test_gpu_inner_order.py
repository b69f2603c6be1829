"""Products with few block products per C block and enough operand bytes to be
launched grouped by inner index: bitwise what the same products give in Morton
order, which a plan can be set to, and, for transposed operands, what the
products of explicitly transposed matrices give."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1501_07800_amd as q
    return q


def _list(rows, cols, count, b, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pos = torch.unique(torch.randint(0, rows * cols, (count,), generator=g, device="cuda"))
    V = torch.randn((len(pos), b, b), generator=g, dtype=torch.float64, device="cuda")
    return (pos // cols).int(), (pos % cols).int(), V


def _build(qt, rows, cols, b, lst):
    return qt.build(rows * b, cols * b, b, 8 * b, *lst)


def _out(C, b, prec):
    import torch
    n = C.nblocks
    I = torch.empty(n, dtype=torch.int32, device="cuda")
    J = torch.empty_like(I)
    V = torch.empty((n, b, b), dtype=torch.float32 if prec == "f32" else torch.float64, device="cuda")
    C.to_blocks_device(I, J, V, "f32" if prec == "f32" else "f64")
    return I, J, V


# m, k, n in blocks; inner dimensions of one sort pass (up to 2048) and of two
@pytest.mark.parametrize("b,prec,m,k,n,count", [(64, "f64", 401, 200, 390, 1700), (64, "bf16x3", 390, 300, 410, 3100),
                                                (32, "f64", 900, 2048, 800, 16000), (32, "f32", 1000, 2049, 1003, 17000),
                                                (32, "bf16x3", 1000, 700, 1001, 11000), (16, "f64", 1300, 5000, 1500, 55000)])
def test_by_inner_index_matches_morton(qt, b, prec, m, k, n, count):
    import torch
    print("inner order", b, prec, m, k, n, count, flush=True)
    la, lb = _list(m, k, count, b, 1), _list(k, n, count, b, 2)
    A, B = _build(qt, m, k, b, la), _build(qt, k, n, b, lb)
    C = qt.multiply(A, B, prec)
    st = C.stats()
    assert st["products"] < 2 * C.nblocks                                    # grouped by inner index ...
    assert 2 * st["products"] * b * b * (8 if prec == "f64" else 4) >= 700 << 20   # ... and worth it
    plan = qt.Plan([A], [B], prec)
    plan.set_schedule("flat+morton")
    plan.execute(graph=False)
    for x, y in zip(_out(C, b, prec), _out(plan.result(0), b, prec)):
        assert torch.equal(x, y)
    if b == 64:
        return
    At = _build(qt, k, m, b, (la[1], la[0], la[2].transpose(1, 2).contiguous()))
    for x, y in zip(_out(C, b, prec), _out(qt.multiply_ex(At, B, trans_a=True, prec=prec), b, prec)):
        assert torch.equal(x, y)
