"""The library's own memory, HIP's stream-ordered pool, instead of a caller's
allocator: calls queued one after another, none waited for, each with buffers of
its own or of a call whose work is done. (The pool hands memory freed on one
stream to the stream that it was made on while the first still works.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture
def hip_pool(qt):
    import torch
    torch.cuda.synchronize()
    qt.use_hip_pool()
    yield
    torch.cuda.synchronize()
    if qt.ALLOCATOR is not None:
        qt.set_allocator(qt.ALLOCATOR.alloc, qt.ALLOCATOR.free)


def _build(qt, rows, cols, count, b, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pos = torch.unique(torch.randint(0, rows * cols, (count,), generator=g, device="cuda"))
    V = torch.randn((len(pos), b, b), generator=g, dtype=torch.float64, device="cuda")
    M = qt.build(rows * b, cols * b, b, 8 * b, (pos // cols).int(), (pos % cols).int(), V)
    torch.cuda.synchronize()
    return M


def _arrays(n, b, prec):
    import torch
    return (torch.full((n,), -1, dtype=torch.int32, device="cuda"), torch.full((n,), -1, dtype=torch.int32, device="cuda"),
            torch.zeros((n, b, b), dtype=torch.float32 if prec == "f32" else torch.float64, device="cuda"))


# (rows, inner, cols, blocks of A, of B): uneven, so that one call's lists lie where another's counts would
SHAPES = [(280, 100, 290, 2500, 2600), (500, 400, 450, 3000, 3100), (300, 90, 270, 2400, 2200), (60, 50, 70, 900, 1000),
          (700, 600, 650, 5000, 5200), (250, 260, 240, 6000, 6100)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("own_stream", [False, True])
def test_products_and_copies_back_to_back(qt, hip_pool, prec, own_stream):
    import torch
    b = 32
    ops = [(_build(qt, m, k, na, b, 2 * t), _build(qt, k, n, nb, b, 2 * t + 1))
           for t, (m, k, n, na, nb) in enumerate(SHAPES)]
    ref = []
    for A, B in ops:                                    # one at a time
        C = qt.multiply(A, B, prec)
        torch.cuda.synchronize()
        out = _arrays(C.nblocks, b, prec)
        torch.cuda.synchronize()
        C.to_blocks_device(*out, prec)
        torch.cuda.synchronize()
        ref.append(out)
        C.free()
    big = torch.randn(4096, 4096, device="cuda")
    s = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    for rep in range(4):
        print("back to back", prec, own_stream, rep, flush=True)
        outs = [_arrays(len(r[0]), b, prec) for r in ref]
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            for _ in range(4):
                big @ big
        for (A, B), out in zip(ops, outs):
            C = qt.multiply(A, B, prec, stream=s)
            C.to_blocks_device(*out, prec, stream=s)
            C.free()
        torch.cuda.synchronize()
        for i, (x, y) in enumerate(zip(ref, outs)):
            assert all(torch.equal(p, q) for p, q in zip(x, y)), (rep, i)


def test_thresholds_transposes_squares_back_to_back(qt, hip_pool):
    import torch
    b = 32
    A, B = _build(qt, 300, 300, 4000, b, 1), _build(qt, 300, 300, 5000, b, 2)
    r = np.random.default_rng(3)
    I, J = np.triu_indices(200)
    u = r.random(len(I)) < 0.1
    U = qt.build(200 * b, 200 * b, b, 4 * b, I[u], J[u], r.standard_normal((int(u.sum()), b, b)))
    calls = [lambda s: qt.multiply_tau(A, B, 30.0 * b, stream=s), lambda s: qt.multiply_ex(A, B, trans_a=True, stream=s),
             lambda s: qt.sysq(U, stream=s), lambda s: qt.multiply_tau(B, A, 28.0 * b, "f32", stream=s),
             lambda s: qt.multiply_ex(B, A, upper=True, stream=s), lambda s: qt.multiply(B, B, "bf16x3", stream=s)]
    ref = []
    for call in calls:
        C = call(None)
        torch.cuda.synchronize()
        out = _arrays(C.nblocks, b, "f64")
        torch.cuda.synchronize()
        C.to_blocks_device(*out)
        torch.cuda.synchronize()
        ref.append(out)
        C.free()
    big = torch.randn(4096, 4096, device="cuda")
    s = torch.cuda.Stream()
    for rep in range(4):
        outs = [_arrays(len(x[0]), b, "f64") for x in ref]
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            for _ in range(3):
                big @ big
        for call, out in zip(calls, outs):
            C = call(s)
            C.to_blocks_device(*out, stream=s)
            C.free()
        torch.cuda.synchronize()
        for i, (x, y) in enumerate(zip(ref, outs)):
            assert all(torch.equal(p, q) for p, q in zip(x, y)), (rep, i)


def test_plans_back_to_back(qt, hip_pool):
    import torch
    b = 32
    mats = [[_build(qt, m, k, na // 2, b, 2 * t), _build(qt, k, n, nb // 2, b, 2 * t + 1)]
            for t, (m, k, n, na, nb) in enumerate(SHAPES)]
    ref = []
    for A, B in mats:
        C = qt.multiply(A, B)
        out = _arrays(C.nblocks, b, "f64")
        C.to_blocks_device(*out)
        torch.cuda.synchronize()
        ref.append(out)
    for rep in range(4):
        outs = [_arrays(len(x[0]), b, "f64") for x in ref]
        torch.cuda.synchronize()
        for half in ((0, 1, 2), (3, 4, 5)):
            plan = qt.Plan([mats[i][0] for i in half], [mats[i][1] for i in half])
            plan.execute(graph=bool(rep & 1))
            for t, i in enumerate(half):
                plan.result(t).to_blocks_device(*outs[i])
            plan.destroy()
        torch.cuda.synchronize()
        for i, (x, y) in enumerate(zip(ref, outs)):
            assert all(torch.equal(p, q) for p, q in zip(x, y)), (rep, i)


def test_memory_comes_back(qt, hip_pool):
    """Parked buffers return to the pool: a long loop holds a few products' worth."""
    import torch
    b = 32
    A, B = _build(qt, 300, 300, 4000, b, 1), _build(qt, 300, 300, 4000, b, 2)

    def loop(n):
        for _ in range(n):
            qt.multiply(A, B).free()
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    loop(20)
    before = loop(20)
    assert before - loop(300) <= 64 << 20
