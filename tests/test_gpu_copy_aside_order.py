"""A large copy-out whose sort has a stream of its own: where its scratch is
obtained and given back, callers on other streams, a product whose values are
still being computed, and a caller that captures the copy-out."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


class Recording:
    """Allocator over torch's that notes the stream of every call, and fails
    allocation number fail_at."""

    def __init__(self, base, fail_at=None):
        self.base, self.fail_at, self.made, self.freed = base, fail_at, [], {}

    def alloc(self, n, stream):
        if len(self.made) == self.fail_at:
            return None
        p = self.base.alloc(n, stream)
        self.made.append((p, stream or 0))
        return p

    def free(self, p, stream):
        self.freed[p] = stream or 0
        self.base.free(p, stream)


def _restore(qt):
    if qt.ALLOCATOR is not None:
        qt.set_allocator(qt.ALLOCATOR.alloc, qt.ALLOCATOR.free)
    else:
        qt.use_hip_pool()


def _matrix(qt, n, b=32, nb=300, seed=0):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pos = torch.randperm(nb * nb, generator=g, device="cuda")[:n]
    I, J = (pos // nb).int(), (pos % nb).int()
    V = torch.randn((n, b, b), generator=g, dtype=torch.float64, device="cuda")
    M = qt.build(nb * b, nb * b, b, 8 * b, I, J, V)
    o = torch.argsort(pos)
    torch.cuda.synchronize()
    return M, I[o], J[o], V[o]


@pytest.mark.parametrize("fail_at", [None, 1, 2, 3])
def test_scratch_goes_back_where_it_is_safe(qt, fail_at):
    """The sort's scratch (the first allocation) is made on the sort's stream.
    It goes back on the caller's once that runs after the sort; when the call
    fails before, on the stream it was made on."""
    import torch
    n = 16384                                       # 128 MiB of values
    M, wI, wJ, wV = _matrix(qt, n)
    rec = Recording(qt.TorchAllocator(), fail_at)
    s = torch.cuda.Stream()
    big = torch.randn(6144, 6144, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for _ in range(20):
            big @ big                               # s is busy: the sort goes to its own stream
    try:
        qt.set_allocator(rec.alloc, rec.free)
        if fail_at is None:
            I, J, V = M.to_blocks(stream=s)
        else:
            with pytest.raises(qt.QtError) as e:
                M.to_blocks(stream=s)
            assert e.value.status == qt.QT_ERR_OOM
    finally:
        _restore(qt)
        torch.cuda.synchronize()
    p, made_on = rec.made[0]
    assert made_on != s.cuda_stream
    assert len(rec.freed) == len(rec.made)
    assert rec.freed[p] == (s.cuda_stream if fail_at is None else made_on)
    if fail_at is None:
        assert np.array_equal(I, wI.cpu().numpy()) and np.array_equal(J, wJ.cpu().numpy())
        assert np.array_equal(V, wV.cpu().numpy())


def test_no_caller_waits_for_another_streams_sorts(qt):
    """While sorts for one stream are still to run, a copy-out on another
    stream sorts on its own: its scratch is made there."""
    import torch
    n = 20000
    M, wI, wJ, wV = _matrix(qt, n)
    rec = Recording(qt.TorchAllocator())
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    big = torch.randn(6144, 6144, device="cuda")
    outs = [(torch.zeros_like(wI), torch.zeros_like(wJ), torch.zeros_like(wV)) for _ in range(2)]
    torch.cuda.synchronize()
    seen = 0
    try:
        qt.set_allocator(rec.alloc, rec.free)
        for _ in range(30):
            for s in (s1, s2):
                with torch.cuda.stream(s):
                    for _ in range(4):
                        big @ big
            first = len(rec.made)
            for _ in range(6):
                M.to_blocks_device(*outs[0], stream=s1)
            aside = rec.made[first][1]
            assert aside not in (s1.cuda_stream, s2.cuda_stream)
            behind = torch.cuda.Event()
            behind.record(torch.cuda.ExternalStream(aside))
            last = len(rec.made)
            M.to_blocks_device(*outs[1], stream=s2)
            if not behind.query():                  # so the other stream's sorts were not done at that call
                seen += 1
                assert rec.made[last][1] == s2.cuda_stream
            torch.cuda.synchronize()
            for o in outs:
                assert torch.equal(o[0], wI) and torch.equal(o[1], wJ) and torch.equal(o[2], wV)
                for x in o:
                    x.zero_()
            torch.cuda.synchronize()
    finally:
        _restore(qt)
        torch.cuda.synchronize()
    print("calls beside another stream's sorts:", seen, flush=True)
    assert seen > 0


def test_threads_on_their_own_streams(qt):
    import torch
    M, wI, wJ, wV = _matrix(qt, 17000, seed=3)
    bad = []

    def work():
        s = torch.cuda.Stream()
        big = torch.randn(4096, 4096, device="cuda")
        out = (torch.zeros_like(wI), torch.zeros_like(wJ), torch.zeros_like(wV))
        torch.cuda.synchronize()
        for _ in range(8):
            with torch.cuda.stream(s):
                big @ big
            M.to_blocks_device(*out, stream=s)
            s.synchronize()
            if not (torch.equal(out[0], wI) and torch.equal(out[1], wJ) and torch.equal(out[2], wV)):
                bad.append(1)

    ts = [threading.Thread(target=work) for _ in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_product_still_running(qt, prec):
    """C's keys are sorted while C's values are computed, behind other work."""
    import torch
    b, nb = 32, 190
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    pos = torch.randperm(nb * nb, generator=g, device="cuda")[:nb * nb // 4]
    A = qt.build(nb * b, nb * b, b, 8 * b, (pos // nb).int(), (pos % nb).int(),
                 torch.randn((len(pos), b, b), generator=g, dtype=torch.float64, device="cuda"))
    dtype = torch.float64 if prec == "f64" else torch.float32
    big = torch.randn(6144, 6144, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(3):
        with torch.cuda.stream(s):
            for _ in range(6):
                big @ big
        C = qt.multiply(A, A, prec, stream=s)
        n = C.nblocks
        assert n > 4096 and n * b * b * dtype.itemsize >= 128 << 20
        I = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        J = torch.full_like(I, -1)
        V = torch.zeros((n, b, b), dtype=dtype, device="cuda")
        torch.cuda.current_stream().synchronize()       # the fills; s is still busy
        C.to_blocks_device(I, J, V, prec, stream=s)
        torch.cuda.synchronize()
        again = [torch.empty_like(x) for x in (I, J, V)]
        C.to_blocks_device(*again, prec, stream=s)      # from an idle stream
        torch.cuda.synchronize()
        at = I.long() * nb + J
        assert bool((at[1:] > at[:-1]).all()) and bool(V.any())
        assert all(torch.equal(x, y) for x, y in zip((I, J, V), again))


def test_captured_with_its_allocations(qt):
    """to_blocks itself, which allocates, on a stream that is being captured:
    all of it belongs to that stream."""
    import torch
    if qt.ALLOCATOR is None:
        pytest.skip("needs torch's allocator, whose memory a capture may use")
    M, wI, wJ, wV = _matrix(qt, 20000, seed=7)
    out = (torch.zeros_like(wI), torch.zeros_like(wJ), torch.zeros_like(wV))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        M.to_blocks_device(*out, stream=s)
    big = torch.randn(2048, 2048, device="cuda")
    for _ in range(4):
        for x in out:
            x.zero_()
        big = big @ big
        big /= big.norm()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], wI) and torch.equal(out[1], wJ) and torch.equal(out[2], wV)
