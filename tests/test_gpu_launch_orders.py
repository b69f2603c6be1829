"""Launch orders of C's blocks where they are in use: strips of block rows (b =
64, 8192 C blocks and two block products each or more) and grouped by inner
index (fewer than two products per C block, 700 MB of operand blocks or more).

Transposed, mirrored and upper-triangle products in these orders against the
dense definition in FP64, and plans of problems with orders of their own, in
every configuration, bitwise against the single multiplies.

Bounds, k the inner dimension in blocks: FP64 both sides sum k b products per
entry, 2 k b 2^-53 (|A||B|)_ij; FP32 and BF16X3 those of the parity tests,
(k b + 2) 2^-24 and 3 2^-16 + (3 b + 4) 2^-24.
"""
import pytest

pytestmark = pytest.mark.gpu


def _list(rows, cols, b, fill, seed, upper=False):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    on = torch.rand(rows, cols, generator=g, device="cuda") < fill
    if upper:
        on = torch.triu(on)
    I, J = (x.int() for x in torch.nonzero(on, as_tuple=True))
    V = torch.randn((len(I), b, b), generator=g, dtype=torch.float64, device="cuda")
    if upper:
        d = I == J
        V[d] = V[d] + V[d].transpose(1, 2)
    return I, J, V


def _dense(rows, cols, b, lst, symmetric=False):
    import torch
    I, J, V = lst
    D = torch.zeros((rows, cols, b, b), dtype=torch.float64, device="cuda")
    D[I.long(), J.long()] = V
    if symmetric:
        D[J.long(), I.long()] = V.transpose(1, 2)
    return D.permute(0, 2, 1, 3).reshape(rows * b, cols * b)


def _out(C, b, prec):
    import torch
    n = C.nblocks
    I = torch.empty(n, dtype=torch.int32, device="cuda")
    J = torch.empty_like(I)
    V = torch.empty((n, b, b), dtype=torch.float32 if prec == "f32" else torch.float64, device="cuda")
    C.to_blocks_device(I, J, V, "f32" if prec == "f32" else "f64")
    return I, J, V


def _check(C, X, Y, b, prec, upper=False):
    import torch
    I, J, V = _out(C, b, prec)
    ref, mag = X @ Y, X.abs() @ Y.abs()

    def blocks(D):
        return D.reshape(D.shape[0] // b, b, D.shape[1] // b, b).permute(0, 2, 1, 3)

    i, j = I.long(), J.long()
    there = torch.zeros((X.shape[0] // b, Y.shape[1] // b), dtype=torch.bool, device="cuda")
    there[i, j] = True
    wanted = blocks(mag).amax((2, 3)) > 0
    assert torch.equal(there, torch.triu(wanted) if upper else wanted)
    k = X.shape[1] // b
    tol = {"f64": 2 * k * b * 2.0 ** -53, "f32": (k * b + 2) * 2.0 ** -24,
           "bf16x3": 3 * 2.0 ** -16 + (3 * b + 4) * 2.0 ** -24}[prec]
    err = (V.double() - blocks(ref)[i, j]).abs()
    assert bool((err <= tol * blocks(mag)[i, j]).all())


def _order(C, b, prec):
    """Which order the rule gives this product ('' for Morton)."""
    n, p = C.nblocks, C.stats()["products"]
    if b == 64 and n >= 8192 and p >= 2 * n:
        return "strips"
    return "inner" if p < 2 * n and 2 * p * b * b * (8 if prec == "f64" else 4) >= 700 << 20 else ""


# strips of one and of eight rows; inner dimensions with and without remainders in their leaves
SHAPES = {"strips": [(95, 130, 101, 0.5, 8), (301, 8, 150, 0.48, 2)],
          "inner": [(190, 70, 191, 0.107, 8), (250, 33, 140, 0.15, 1)]}


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("ta,tb", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("order,shape", [(o, s) for o in SHAPES for s in SHAPES[o]])
def test_transposed(qt, prec, ta, tb, order, shape):
    m, k, n, fill, lb = shape
    b = 64
    print("order", order, prec, ta, tb, shape, flush=True)
    la, lB = _list(k if ta else m, m if ta else k, b, fill, 1), _list(n if tb else k, k if tb else n, b, fill, 2)
    A = qt.build((k if ta else m) * b, (m if ta else k) * b, b, lb * b, *la)
    B = qt.build((n if tb else k) * b, (k if tb else n) * b, b, lb * b, *lB)
    C = qt.multiply_ex(A, B, trans_a=ta, trans_b=tb, prec=prec)
    assert _order(C, b, prec) == order
    X, Y = _dense(*((k, m) if ta else (m, k)), b, la), _dense(*((n, k) if tb else (k, n)), b, lB)
    _check(C, X.T if ta else X, Y.T if tb else Y, b, prec)


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("fill", [0.5, 0.12])
def test_mirrored_and_upper(qt, prec, fill):
    b, nb = 64, 140
    print("strips, symmetric", prec, fill, flush=True)
    lst = _list(nb, nb, b, fill, 3, upper=True)
    C = qt.sysq(qt.build(nb * b, nb * b, b, 4 * b, *lst), prec)
    assert _order(C, b, prec) == "strips"
    S = _dense(nb, nb, b, lst, symmetric=True)
    _check(C, S, S, b, prec, upper=True)
    full = _list(nb, nb, b, fill, 4)
    M = qt.build(nb * b, nb * b, b, 4 * b, *full)
    C = qt.multiply_ex(M, M, trans_a=True, upper=True, prec=prec)
    assert _order(C, b, prec) == "strips"
    D = _dense(nb, nb, b, full)
    _check(C, D.T, D, b, prec, upper=True)


# one problem in strips (b = 64), one by inner index, one of each kind too small for an order
@pytest.mark.parametrize("b,prec,shapes", [
    (64, "f64", [(95, 130, 101, 0.3), (190, 70, 191, 0.107), (40, 31, 50, 0.3), (60, 50, 61, 0.1)]),
    (64, "f32", [(301, 8, 150, 0.48), (190, 70, 191, 0.107), (24, 24, 24, 0.04)]),
    (64, "bf16x3", [(131, 60, 120, 0.25), (250, 33, 240, 0.15), (7, 11, 5, 0.4)]),
    (32, "f64", [(280, 100, 290, 0.09), (50, 60, 70, 0.3), (300, 90, 270, 0.09)]),
    (32, "f32", [(400, 100, 401, 0.09), (128, 128, 128, 0.1)]),
    (16, "f64", [(600, 100, 610, 0.09), (100, 90, 80, 0.1)])])
def test_plans_of_problems_with_their_own_orders(qt, b, prec, shapes):
    import torch
    As, Bs = [], []
    for t, (m, k, n, fill) in enumerate(shapes):
        As.append(qt.build(m * b, k * b, b, 8 * b, *_list(m, k, b, fill, 2 * t)))
        Bs.append(qt.build(k * b, n * b, b, 8 * b, *_list(k, n, b, fill, 2 * t + 1)))
    single = [qt.multiply(x, y, prec) for x, y in zip(As, Bs)]
    orders = [_order(C, b, prec) for C in single]
    assert "inner" in orders and (b != 64 or "strips" in orders) and "" in orders
    ref = [_out(C, b, prec) for C in single]
    plan = qt.Plan(As, Bs, prec)
    for c in range(qt.PLAN_CONFIGS):
        name = qt.plan_config_name(c)
        print("plan", b, prec, orders, name, flush=True)
        plan.set_schedule(name)
        plan.execute(graph=c % 2 == 0)
        for i, want in enumerate(ref):
            for x, y in zip(want, _out(plan.result(i), b, prec)):
                assert torch.equal(x, y), (name, i)
    plan.destroy()
