"""Products of transposed and mirrored operands at b = 64 against numpy's
definition, over segments of one product, of several, and of mixed
transposition bits (the symmetric square).

FP64: both sides sum k 64 products per entry, so they differ by at most
2 k 64 2^-53 (|A||B|)_ij, k the most block products of a C block. FP32 and
BF16X3: the bounds of the parity tests, (64 k + 2) 2^-24 and
(3 2^-16 + (3 64 + 4) 2^-24).
"""
import numpy as np
import pytest

from tests._util import random_pattern, symmetric_from_upper, to_dense, upper_blocks

pytestmark = pytest.mark.gpu
B = 64


@pytest.fixture(scope="module")
def qt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1501_07800_amd as q
    return q


def _bound(prec, k):
    return {"f64": 2 * k * B * 2.0 ** -53, "f32": (k * B + 2) * 2.0 ** -24,
            "bf16x3": 3 * 2.0 ** -16 + (3 * B + 4) * 2.0 ** -24}[prec]


def _check(C, X, Y, prec, upper=False):
    I, J, V = C.to_blocks("f64")
    ref, mag = X @ Y, np.abs(X) @ np.abs(Y)
    got, seen = np.zeros_like(ref), np.zeros_like(ref, bool)
    for i, j, v in zip(I, J, V):
        got[i * B:(i + 1) * B, j * B:(j + 1) * B] = v
        seen[i * B:(i + 1) * B, j * B:(j + 1) * B] = True
    if upper:
        n = np.arange(ref.shape[0]) // B
        keep = n[:, None] <= n[None, :]
        assert not seen[~keep].any()
        ref, mag = np.where(keep, ref, 0.0), np.where(keep, mag, 0.0)
    assert not ref[~seen].any()
    k = X.shape[1] // B
    assert (np.abs(got - ref) <= _bound(prec, k) * mag).all()


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("ta,tb", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("m,k,n,fill", [(1, 1, 1, 1.0), (3, 1, 5, 1.0), (2, 9, 3, 0.6), (11, 10, 9, 0.3)])
def test_transposed(qt, prec, ta, tb, m, k, n, fill):
    rng = np.random.default_rng(m * 100 + k * 10 + n)
    A = random_pattern(rng, k if ta else m, m if ta else k, fill, B)
    Bm = random_pattern(rng, n if tb else k, k if tb else n, fill, B)
    print("op", prec, ta, tb, m, k, n, A.nnz, Bm.nnz, flush=True)
    hA, hB = qt.from_blockmatrix(A, 256), qt.from_blockmatrix(Bm, 256)
    C = qt.multiply_ex(hA, hB, trans_a=ta, trans_b=tb, prec=prec)
    X, Y = to_dense(A), to_dense(Bm)
    _check(C, X.T if ta else X, Y.T if tb else Y, prec)


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("n,fill", [(1, 1.0), (2, 1.0), (9, 0.5)])
def test_symmetric_square(qt, prec, n, fill):
    rng = np.random.default_rng(n)
    A = upper_blocks(random_pattern(rng, n, n, fill, B))
    for t in np.flatnonzero(A.I == A.J):
        A.V[t] = 0.5 * (A.V[t] + A.V[t].T)
    print("sysq", prec, n, A.nnz, flush=True)
    S = to_dense(symmetric_from_upper(A))
    _check(qt.sysq(qt.from_blockmatrix(A, 256), prec), S, S, prec, upper=True)
