"""The problems of a plan, whose symbolic phases share launches, against the
same products one by one: bitwise the same blocks at the same positions, the
same trees and counters, whatever problems lie beside them (one-launch small
ones, several depths, lifted operands, empty ones, one too wide to share, more
than share one set of launches)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1501_07800_amd as q
    return q


def _matrix(qt, rows, cols, nblocks, seed, b=16, lb=8):
    import torch
    r = np.random.default_rng(seed)
    pos = np.sort(r.choice(rows * cols, size=min(nblocks, rows * cols), replace=False))
    I, J = (torch.as_tensor(x.astype(np.int32), device="cuda") for x in np.divmod(pos, cols))
    V = torch.as_tensor(r.standard_normal((len(pos), b, b)), device="cuda")
    return qt.build(rows * b, cols * b, b, lb * b, I, J, V)


# (rows, inner, columns, blocks of A, blocks of B)
SMALL = [(1, 1, 1, 1, 1), (9, 9, 9, 30, 30), (40, 40, 40, 160, 120), (23, 57, 31, 130, 170)]
MID = [(130, 130, 130, 900, 900), (300, 300, 300, 2500, 2000), (65, 500, 70, 1500, 1500)]
EMPTY = [(8, 8, 8, 0, 5), (64, 64, 64, 1, 1)]
LIFTED = [(40, 700, 700, 400, 20000), (700, 90, 40, 9000, 600)]     # operands of different depth
WIDE = [(2104, 2104, 2104, 14000, 14000)]                           # more nodes at a level than share a launch
DEEP = [(1500, 1500, 1500, 30000, 30000)]                           # far larger than what lies beside it
CASES = {
    "one": MID[:1],
    "small": SMALL,
    "mixed": SMALL + MID + EMPTY + LIFTED,
    "wide": MID[:2] + WIDE + SMALL[:2],
    "uneven": MID * 12 + DEEP + SMALL,
    "many": SMALL * 60 + MID * 9 + EMPTY * 4,       # 275 problems
}


@pytest.mark.parametrize("name", list(CASES))
def test_plan_equals_single_products(qt, name):
    import torch
    shapes = CASES[name]
    prec = "f64" if name != "wide" else "f32"
    made = {}
    for s in shapes:
        if s not in made:
            m, k, n, na, nb = s
            A, B = _matrix(qt, m, k, na, len(made)), _matrix(qt, k, n, nb, 100 + len(made))
            made[s] = (A, B, qt.multiply(A, B, prec))
    plan = qt.Plan([made[s][0] for s in shapes], [made[s][1] for s in shapes], prec)
    for graph in (False, True):
        plan.execute(graph=graph)
    dt = torch.float64 if prec == "f64" else torch.float32
    for i, s in enumerate(shapes):
        one, got = made[s][2], plan.result(i)
        print("plan", name, i, s, flush=True)
        assert got.nblocks == one.nblocks
        a, b = got.stats(), one.stats()
        assert a["products"] == b["products"] and a["pairs"].tolist() == b["pairs"].tolist()
        assert got.levels().tolist() == one.levels().tolist()
        if not got.nblocks:
            continue
        out = []
        for M in (got, one):
            I = torch.empty(M.nblocks, dtype=torch.int32, device="cuda")
            J = torch.empty_like(I)
            V = torch.empty((M.nblocks, 16, 16), dtype=dt, device="cuda")
            M.to_blocks_device(I, J, V, "f64" if dt == torch.float64 else "f32")
            out.append((I, J, V))
        for x, y in zip(*out):
            assert torch.equal(x, y), (name, i, s)


def test_leaf_sizes_side_by_side(qt):
    """Problems of different leaf sizes (4 x 4 and 8 x 8 blocks, one block) in one plan."""
    import torch
    mats = [_matrix(qt, 200, 200, 2000, 40 + lb, lb=lb) for lb in (8, 4, 1, 2, 8)]
    plan = qt.Plan(mats, mats, "f64")
    plan.execute(graph=False)
    for i, A in enumerate(mats):
        one, got = qt.multiply(A, A), plan.result(i)
        assert got.nblocks == one.nblocks and got.levels().tolist() == one.levels().tolist()
        out = []
        for M in (got, one):
            V = torch.empty((M.nblocks, 16, 16), dtype=torch.float64, device="cuda")
            I = torch.empty(M.nblocks, dtype=torch.int32, device="cuda")
            J = torch.empty_like(I)
            M.to_blocks_device(I, J, V)
            out.append((I, J, V))
        for x, y in zip(*out):
            assert torch.equal(x, y)
