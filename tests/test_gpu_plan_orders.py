"""Plans whose problems are launched by inner index below the size from which a
single product is: the order is there to choose, and every configuration gives
bitwise the single products (which are in Morton order)."""
import pytest

pytestmark = pytest.mark.gpu


def _build(qt, rows, cols, count, b, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pos = torch.unique(torch.randint(0, rows * cols, (count,), generator=g, device="cuda"))
    V = torch.randn((len(pos), b, b), generator=g, dtype=torch.float64, device="cuda")
    return qt.build(rows * b, cols * b, b, 8 * b, (pos // cols).int(), (pos % cols).int(), V)


def _out(C, b, prec):
    import torch
    n = C.nblocks
    I = torch.empty(n, dtype=torch.int32, device="cuda")
    J = torch.empty_like(I)
    V = torch.empty((n, b, b), dtype=torch.float32 if prec == "f32" else torch.float64, device="cuda")
    C.to_blocks_device(I, J, V, "f32" if prec == "f32" else "f64")
    return I, J, V


# (rows, inner, cols, blocks of A, of B): one-launch problems, problems of up to 4096 C blocks
# (sorted together) and of more (one and two digits), a dense one in Morton order, an empty one
MIXED = [(30, 40, 31, 60, 70), (300, 280, 310, 700, 900), (500, 700, 600, 3000, 2900), (400, 3000, 500, 9000, 11000),
         (20, 20, 20, 300, 300), (25, 9, 25, 1, 1), (1, 1, 1, 1, 1), (90, 5000, 80, 4000, 3500)]


@pytest.mark.parametrize("b,prec", [(16, "f64"), (32, "f32"), (32, "bf16x3"), (64, "f64"), (64, "f32")])
def test_mixed_sizes(qt, b, prec):
    import torch
    shapes = MIXED if b < 64 else MIXED[:3] + MIXED[4:7]
    As = [_build(qt, m, k, na, b, 2 * t) for t, (m, k, n, na, nb) in enumerate(shapes)]
    Bs = [_build(qt, k, n, nb, b, 2 * t + 1) for t, (m, k, n, na, nb) in enumerate(shapes)]
    single = [qt.multiply(x, y, prec) for x, y in zip(As, Bs)]
    ref = [_out(C, b, prec) for C in single]
    sizes = [C.nblocks for C in single]
    assert any(0 < C.nblocks <= 4096 and C.stats()["products"] < 2 * C.nblocks for C in single)
    assert b == 64 or any(n > 4096 for n in sizes)
    for c in range(qt.PLAN_CONFIGS):
        name = qt.plan_config_name(c)
        print("plan", b, prec, sizes, name, flush=True)
        plan = qt.Plan(As, Bs, prec)
        plan.set_schedule(name)
        for run in range(3):                 # the orders come with the first replay, the second other run
            plan.execute(graph=c % 2 == 0)
            for i, want in enumerate(ref):
                for x, y in zip(want, _out(plan.result(i), b, prec)):
                    assert torch.equal(x, y), (name, run, i)
        plan.destroy()
    plan = qt.Plan(As, Bs, prec)
    _, times = plan.tune(reps=1)
    assert "flat" in times and "flat+morton" in times
    plan.destroy()


def test_many_problems(qt):
    """More problems than share launches at once."""
    import torch
    b = 16
    hs = [_build(qt, 20 + t % 7, 20 + t % 7, 30 + t % 11, b, t) for t in range(300)]
    plan = qt.Plan(hs, hs, "f64")
    plan.execute()
    for i, h in enumerate(hs):
        for x, y in zip(_out(qt.multiply(h, h), b, "f64"), _out(plan.result(i), b, "f64")):
            assert torch.equal(x, y), i
    plan.destroy()


@pytest.mark.parametrize("first", [None, "flat+morton", "balanced", "dynamic-16"])
def test_captured_runs_and_changes_between(qt, first):
    """Runs captured by the caller before and after the orders are made, and
    configurations changed between replays."""
    import torch
    b = 32
    As = [_build(qt, m, k, na, b, 2 * t) for t, (m, k, n, na, nb) in enumerate(MIXED)]
    Bs = [_build(qt, k, n, nb, b, 2 * t + 1) for t, (m, k, n, na, nb) in enumerate(MIXED)]
    ref = [_out(qt.multiply(x, y), b, "f64") for x, y in zip(As, Bs)]
    plan = qt.Plan(As, Bs, "f64")
    big = torch.randn(1024, 1024, device="cuda")

    def check():
        for i, want in enumerate(ref):
            for x, y in zip(want, _out(plan.result(i), b, "f64")):
                assert torch.equal(x, y), i

    def captured():
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            plan.execute(stream=s, graph=False)
        return g

    if first:
        plan.set_schedule(first)
    graphs = [captured()]
    plan.execute(graph=False)
    check()
    graphs.append(captured())                # the third run, but on a captured stream
    plan.execute(graph=False)
    check()
    graphs.append(captured())
    for name in ("flat", "balanced", "flat+morton", "xcd-dynamic", "flat"):
        plan.set_schedule(name)
        for _ in range(2):
            plan.execute()
            big = big @ big
            big /= big.norm()
            check()
    for _ in range(3):
        for g in graphs:
            g.replay()
            torch.cuda.synchronize()
            check()
    plan.destroy()
