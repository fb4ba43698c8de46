"""Sequences whose exchange buffers have more elements than 32 bits count: a whole run against the same run in two parts (the
oracle would take minutes).  Nothing but the order of a few float sums differs between the two."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(T, B, d, h, r, L, groups):
    g = torch.Generator(device="cuda").manual_seed(7)
    u = lambda *s: (torch.rand(s, generator=g, device="cuda") - 0.5) * 0.2
    din = [d] + [h] * (L - 1)
    return dict(x=u(T, B, d), h0=[u(B, h) for _ in range(L)], c0=[u(B, h) for _ in range(L)],
                Vx=[u(i, groups * r) for i in din], Ux=[u(4 * h, r) for _ in range(L)],
                Vh=[u(h, groups * r) for _ in range(L)], Uh=[u(4 * h, r) for _ in range(L)],
                bias=[u(4 * h) for _ in range(L)])


def _rel(a, b):
    return float((a - b).double().norm() / b.double().norm())


@pytest.fixture(autouse=True)
def _give_memory_back():
    yield
    torch.cuda.empty_cache()


def test_forward():
    """A factor pair per gate, rank 384, batch 20: T x of 69906 steps and more are beyond 2^31 elements."""
    import paper_2103_03936_amd as pf
    T, half = 70400, 35200
    assert T * 4 * 384 * 20 > 2 ** 31 > half * 4 * 384 * 20
    a = _inputs(T, 20, 16, 32, 384, 1, 4)
    f = [a[k] for k in ("Vx", "Ux", "Vh", "Uh", "bias")]
    h, c, _, _, Th = pf.pf_lowrank_lstm_stack_fwd(a["x"], a["h0"], a["c0"], *f, 4)
    for t0, h0, c0 in ((0, a["h0"][0], a["c0"][0]), (half, h[0][half - 1], c[0][half - 1])):
        o = pf.pf_lowrank_lstm_stack_fwd(a["x"][t0:t0 + half], [h0], [c0], *f, 4)
        assert _rel(h[0][t0:t0 + half], o[0][0]) <= 1e-5
        assert _rel(Th[0][t0:t0 + half], o[4][0]) <= 1e-5


def test_backward():
    """Three layers, rank 384, batch 32: the sums over dT's slices of 34953 steps and more are beyond 2^31 elements.  The
    gradients are float sums over a million rows: 1e-3 (a missing dT leaves nothing of them)."""
    import paper_2103_03936_amd as pf
    T, half, B, h, r, L = 34976, 17488, 32, 128, 384, 3
    assert (2 * L - 1) * T * r * B > 2 ** 31 > (2 * L - 1) * half * r * B
    a = _inputs(T, B, 8, h, r, L, 1)
    f = [a[k] for k in ("Vx", "Ux", "Vh", "Uh")]
    kept = pf.pf_lowrank_lstm_stack_fwd(a["x"], a["h0"], a["c0"], *f, a["bias"], 1)
    dh = torch.randn((T, B, h), generator=torch.Generator(device="cuda").manual_seed(8), device="cuda")
    dx, dh0, _, grads = pf.pf_lowrank_lstm_stack_bwd(a["x"], a["h0"], a["c0"], *kept, *f, dh)
    part = lambda t0: [[t[t0:t0 + half] for t in k] for k in kept]
    mid = [[k[l][half - 1] for l in range(L)] for k in kept[:2]]
    dx2, dm, dcm, sums = pf.pf_lowrank_lstm_stack_bwd(a["x"][half:], mid[0], mid[1], *part(half), *f, dh[half:])
    dx1, e0, _, sums = pf.pf_lowrank_lstm_stack_bwd(a["x"][:half], a["h0"], a["c0"], *part(0), *f, dh[:half], dm, dcm,
                                                    grads=sums)
    assert _rel(dx, torch.cat([dx1, dx2])) <= 1e-4
    for l in range(L):
        assert _rel(dh0[l], e0[l]) <= 1e-4
        for k in ("dVx", "dUx", "dVh", "dUh", "dbias"):
            assert _rel(grads[l][k], sums[l][k]) <= 1e-3, (l, k)
