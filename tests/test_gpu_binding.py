"""The Python boundary: what it refuses, and that it keeps what it was given."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _linear(M=8, n_in=16, n_out=24, r=8):
    g = torch.Generator(device="cuda").manual_seed(1)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    return n(M, n_in), n(n_in, r), n(n_out, r), n(M, n_out)


def _zeros(*shapes):
    return [torch.zeros(s, device="cuda") for s in shapes]


@pytest.mark.parametrize("entries", [0, 1, 2, 4])
def test_grads_of_the_wrong_length_are_refused(entries):
    """Neither is a gradient left out nor an extra entry ignored."""
    import paper_2103_03936_amd as pf
    X, V, U, dY = _linear()
    grads = _zeros((24, 8), (16, 8), (24,), (24,))[:entries]
    for call in (pf.pf_lowrank_linear_bwd, pf.pf_lowrank_linear_bwd_ep):
        with pytest.raises(ValueError):
            call(X, V, U, dY, has_bias=True, grads=grads)
    with pytest.raises(ValueError):
        pf.pf_lowrank_linear_shared_bwd(X, V[None].contiguous(), U[None].contiguous(), dY[None].contiguous(), grads=grads)
    Xc, Uk, Vp, dZ = torch.ones(2, 4, 6, 6, device="cuda"), *_zeros((4, 4, 3, 3), (8, 4)), torch.ones(2, 8, 6, 6, device="cuda")
    with pytest.raises(ValueError):
        pf.pf_lowrank_conv_bwd_ep(Xc, Uk, Vp, None, dZ, pad=1, grads=grads)
    grads = _zeros((4, 4, 3, 3), (8, 4), (8,), (8,))[:3 if entries == 2 else entries]
    with pytest.raises(ValueError):
        pf.pf_lowrank_conv_bwd(Xc, Uk, Vp, dZ, pad=1, grads=grads)


def test_grads_from_an_iterator():
    """Entries that nothing else keeps alive, and one that is not wanted."""
    import paper_2103_03936_amd as pf
    X, V, U, dY = _linear()
    _, dU, dV, db = pf.pf_lowrank_linear_bwd(X, V, U, dY, has_bias=True)
    _, gU, gV, none = pf.pf_lowrank_linear_bwd(X, V, U, dY, has_bias=True, grads=(z for z in [*_zeros((24, 8), (16, 8)), None]))
    assert torch.equal(gU, dU) and torch.equal(gV, dV) and none is None and db is not None


def test_one_scratch_buffer_per_stream():
    """A call marshalled in Python (the SVD) and a native one share their stream's buffer."""
    import paper_2103_03936_amd as pf
    X, V, U, dY = _linear(64, 512, 512, 128)
    with torch.cuda.stream(torch.cuda.Stream()):
        pf.pf_svd_split(torch.randn(300, 128, device="cuda"), 8)
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        pf.pf_lowrank_linear_bwd(X, V, U, dY)
        torch.cuda.synchronize()
        assert torch.cuda.memory_allocated() == before


def test_a_call_waits_for_its_streams_buffer_without_the_interpreter():
    """While another thread has the stream's scratch buffer a call waits, and Python goes on meanwhile; on another stream it
    does not wait."""
    import threading
    import paper_2103_03936_amd as pf
    X, V, U, dY = _linear(64, 512, 512, 128)
    stream = torch.cuda.current_stream()
    pf.pf_lowrank_linear_bwd(X, V, U, dY)
    done = threading.Event()

    def call():
        with torch.cuda.stream(stream):
            pf.pf_lowrank_linear_bwd(X, V, U, dY)
        done.set()

    thread = threading.Thread(target=call)
    with pf._workspace(256, X):
        thread.start()
        assert not done.wait(0.2)
        with torch.cuda.stream(torch.cuda.Stream()):
            pf.pf_lowrank_linear_bwd(X, V, U, dY)
    assert done.wait(60)
    thread.join()


@pytest.mark.parametrize("own_stream", [False, True])
def test_threads(own_stream):
    """Four threads' calls, on one stream (which share its scratch buffer) and on their own, give what one thread gets."""
    import threading
    import paper_2103_03936_amd as pf
    shapes = [(64, 512, 512, 128), (300, 200, 100, 30), (129, 65, 127, 33), (1000, 130, 72, 17)]
    inputs = [_linear(*s) for s in shapes]
    want = [pf.pf_lowrank_linear_bwd(*a, has_bias=True) for a in inputs]
    torch.cuda.synchronize()
    main, wrong = torch.cuda.current_stream(), []

    def work(i):
        s = torch.cuda.Stream() if own_stream else main
        with torch.cuda.stream(s):
            for _ in range(100):
                got = pf.pf_lowrank_linear_bwd(*inputs[i], has_bias=True)
            s.synchronize()
            wrong.extend(k for k, (g, w) in enumerate(zip(got, want[i])) if not torch.equal(g, w))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
