"""A product with a norm threshold queued behind work that its operands' values
or norms still wait for: the same result as with everything finished before."""
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


def _out(C, stream):
    import torch
    with torch.cuda.stream(stream):
        I = torch.empty(C.nblocks, dtype=torch.int32, device="cuda")
        J = torch.empty_like(I)
        V = torch.empty((C.nblocks, 16, 16), dtype=torch.float64, device="cuda")
        C.to_blocks_device(I, J, V, stream=stream)
    return I, J, V


@pytest.mark.parametrize("own_stream", [False, True])
@pytest.mark.parametrize("second_stream", [False, True])
def test_behind_pending_work(qt, own_stream, second_stream):
    import torch
    r = np.random.default_rng(5)
    nb, n = 120, 1800
    pos = np.sort(r.choice(nb * nb, size=n, replace=False))
    I, J = (torch.as_tensor(x.astype(np.int32), device="cuda") for x in np.divmod(pos, nb))
    V = torch.as_tensor(r.standard_normal((n, 16, 16)) * np.exp(-6.0 * r.random((n, 1, 1))), device="cuda")
    A = qt.build(nb * 16, nb * 16, 16, 128, I, J, V)
    big = torch.randn(6144, 6144, device="cuda")
    torch.cuda.synchronize()
    s1 = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    s2 = torch.cuda.Stream() if second_stream else s1

    def steps(wait):
        with torch.cuda.stream(s1):
            for _ in range(8):
                big @ big                                   # the stream is behind
            if wait:
                torch.cuda.synchronize()
            X = qt.multiply(A, A, stream=s1)                # its values are still to come
            if wait:
                torch.cuda.synchronize()
            C = qt.multiply_tau(X, X, 30.0, stream=s1)      # and so are its norms
            if wait:
                torch.cuda.synchronize()
        s2.wait_stream(s1)
        D = qt.multiply_tau(X, A, 20.0, stream=s2)          # norms made on s1
        out = _out(C, s1) + _out(D, s2)
        torch.cuda.synchronize()
        return out, C.stats()["products"], D.stats()["products"]

    want, got = steps(True), steps(False)
    assert got[1:] == want[1:]
    full = qt.multiply(A, A)
    assert 0 < want[2] < qt.multiply(full, A).stats()["products"]    # something was dropped
    for x, y in zip(got[0], want[0]):
        assert torch.equal(x, y)
