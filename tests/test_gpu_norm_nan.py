"""Products with a norm threshold whose operands hold infinite and zero blocks:
a norm product that is not a number is dropped by the counts and the lists
alike, so C has exactly the definition's blocks and products, and every block
without an infinite factor its values.

Bound: both sides sum at most k b products per entry, each within k b 2^-53 of
the exact value relative to (|A||B|).
"""
import numpy as np
import pytest

from tests._util import norm_thresholded_by_definition, positions, random_pattern, tau_in_gap
from workloads import BlockMatrix

pytestmark = pytest.mark.gpu


# one workgroup's product, and one taken level by level; leaves of 1, 2 and 8 blocks a side
@pytest.mark.parametrize("nb,fill", [(24, 0.3), (48, 0.5)])
@pytest.mark.parametrize("lb", [1, 2, 8])
def test_infinite_times_zero(qt, nb, fill, lb):
    b = 16
    print("nan norms", nb, fill, lb, flush=True)
    rng = np.random.default_rng(nb + lb)
    A, B = random_pattern(rng, nb, nb, fill, b), random_pattern(rng, nb, nb, fill, b)
    tau = tau_in_gap(A, B, 0.4)
    inf = rng.choice(A.nnz, size=A.nnz // 12, replace=False)
    A.V[inf, 3, 5] = np.inf
    A.V[inf, 7, 1] = -np.inf
    B.V[rng.choice(B.nnz, size=B.nnz // 4, replace=False)] = 0.0
    with np.errstate(invalid="ignore"):
        ref, kept, dropped, _ = norm_thresholded_by_definition(A, B, tau)
        mag = norm_thresholded_by_definition(BlockMatrix(A.n_rows, A.n_cols, b, A.I, A.J, np.abs(A.V)),
                                             BlockMatrix(B.n_rows, B.n_cols, b, B.I, B.J, np.abs(B.V)), tau)[0]
    assert dropped > 0
    hC = qt.multiply_tau(qt.from_blockmatrix(A, lb * b), qt.from_blockmatrix(B, lb * b), tau)
    assert hC.stats()["products"] == kept
    I, J, V = hC.to_blocks()
    C = BlockMatrix(A.n_rows, B.n_cols, b, I, J, V)
    assert np.array_equal(positions(C), positions(ref))
    fin = np.isfinite(ref.V)
    assert np.array_equal(np.isfinite(C.V), fin) and fin.any() and not fin.all()
    assert np.all(np.abs(C.V[fin] - ref.V[fin]) <= 2 * nb * b * 2.0 ** -53 * mag.V[fin])
