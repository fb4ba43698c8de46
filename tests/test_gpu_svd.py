"""GPU truncated-SVD factor initialisation (Algorithm 1) against the oracle's Jacobi SVD.

The factors are unique only up to the sign of each column pair (and rotations inside repeated singular values),
so what is compared is what is unique: the singular values, the rank-r product U V^T, and the balanced-split
invariant U^T U = V^T V = diag(sigma_r).  Tolerance: the outputs are float32, the iteration runs in double.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from parity import assert_close, to_gpu

pytestmark = pytest.mark.gpu

SHAPES = [
    # m, n, r
    (1, 1, 1),
    (6, 4, 2),
    (5, 9, 3),       # more columns than rows: works on the transpose
    (33, 7, 7),      # odd number of columns (one player sits out each round), full rank kept
    (64, 64, 64),
    (200, 130, 40),
    (512, 512, 128),  # VGG-19 fc17/fc18 (Appendix D)
]


def _matrix(m, n, seed):
    return workloads.Stream(workloads.SEED_BASE + 900 + seed, "f32").normal((m, n)).astype(np.float32)


def _check(W, r, tag):
    import paper_2103_03936_amd as pf
    Uo, Vo, so = oracle.svd_split(W.astype(np.float64), r)
    U, V, sigma = pf.pf_svd_split(to_gpu(W), r)
    torch.cuda.synchronize()
    smax = float(so[0]) if so[0] > 0 else 1.0
    got = sigma.double().cpu().numpy()
    assert np.max(np.abs(got - so)) <= 1e-5 * smax, f"{tag}: singular values off by {np.max(np.abs(got - so)) / smax:.2e}"
    assert np.all(np.diff(got) <= 1e-6 * smax), f"{tag}: singular values not in descending order"
    assert_close(U.double() @ V.double().t(), Uo @ Vo.T, "f32", tag + " U V^T")
    Ud, Vd = U.double().cpu().numpy(), V.double().cpu().numpy()
    for name, F in (("U", Ud), ("V", Vd)):
        gram = F.T @ F
        assert np.max(np.abs(gram - np.diag(so[:r]))) <= 2e-5 * smax, f"{tag}: {name}^T {name} is not diag(sigma_r)"


@pytest.mark.parametrize("shape", SHAPES)
def test_svd_split(shape):
    m, n, r = shape
    _check(_matrix(m, n, seed=m + 3 * n), r, f"svd {shape}")


def test_rank_deficient_matrix():
    """Rank 3 matrix, r = 5 kept: two singular values are zero and their factor columns vanish."""
    a, b = _matrix(40, 3, 1).astype(np.float64), _matrix(3, 24, 2).astype(np.float64)
    W = (a @ b).astype(np.float32)
    import paper_2103_03936_amd as pf
    U, V, sigma = pf.pf_svd_split(to_gpu(W), 5)
    s = sigma.double().cpu().numpy()
    assert np.all(s[3:] <= 1e-5 * s[0])
    assert_close(U.double() @ V.double().t(), W.astype(np.float64), "f32", "rank-deficient reconstruction")


def test_convergence_is_reported_and_sweeps_stop():
    """The rounding-level threshold lets a converged sweep end the launches (info[0] well below the 24-sweep cap,
    info[1] == 0), also for an ill-conditioned matrix (singular values over nine decades) and a rank-deficient one."""
    import paper_2103_03936_amd as pf
    q1, _ = np.linalg.qr(_matrix(300, 60, 7).astype(np.float64))
    q2, _ = np.linalg.qr(_matrix(60, 60, 8).astype(np.float64))
    ill = ((q1 * np.logspace(0, -9, 60)) @ q2.T).astype(np.float32)
    deficient = (_matrix(200, 4, 9).astype(np.float64) @ _matrix(4, 90, 10).astype(np.float64)).astype(np.float32)
    # (a graded matrix needs more sweeps of an unpivoted one-sided Jacobi than a well-conditioned one)
    for tag, W, r, cap in (("well conditioned", _matrix(2000, 200, 11), 50, 12), ("ill conditioned", ill, 20, 23),
                           ("rank deficient", deficient, 6, 23)):
        U, V, sigma, info = pf.pf_svd_split(to_gpu(W), r, return_info=True)
        sweeps, last = (int(v) for v in info.cpu())
        assert last == 0, f"{tag}: {last} rotations in the last of {sweeps} sweeps"
        assert 1 <= sweeps <= cap, f"{tag}: {sweeps} sweeps"
        Uo, Vo, so = oracle.svd_split(W.astype(np.float64), r)
        assert np.max(np.abs(sigma.double().cpu().numpy() - so)) <= 1e-5 * so[0], tag
        assert_close(U.double() @ V.double().t(), Uo @ Vo.T, "f32", tag + " U V^T")


def test_conv_filter_bank():
    """ResNet-18 conv4_x filter bank 256 x 256 x 3 x 3 at rank 64 (Section 2.2 unrolling): the factorized layer's
    composed dense filters equal the oracle's rank-64 truncation."""
    import paper_2103_03936_amd as pf
    Wd = workloads.Stream(workloads.SEED_BASE + 950, "f32").normal((256, 256, 3, 3)).astype(np.float32) * 0.05
    Uko, Vpo, so = oracle.svd_split_conv(Wd.astype(np.float64), 64)
    Uk, Vp, sigma = pf.pf_svd_split_conv(to_gpu(Wd), 64)
    assert Uk.shape == (64, 256, 3, 3) and Vp.shape == (256, 64)
    got = torch.einsum("or,rcij->ocij", Vp.double(), Uk.double())
    want = np.einsum("or,rcij->ocij", Vpo, Uko)
    assert_close(got, want, "f32", "composed filters")
    assert np.max(np.abs(sigma.double().cpu().numpy() - so)) <= 1e-5 * so[0]


def test_deterministic():
    import paper_2103_03936_amd as pf
    W = to_gpu(_matrix(96, 48, 5))
    a = pf.pf_svd_split(W, 12)
    b = pf.pf_svd_split(W, 12)
    for u, v in zip(a, b):
        assert torch.equal(u, v)


def test_conv_info():
    """The filter bank's call hands out the convergence report too."""
    import paper_2103_03936_amd as pf
    Wd = to_gpu(_matrix(12, 8 * 9, 21).reshape(12, 8, 3, 3))
    plain = pf.pf_svd_split_conv(Wd, 4)
    *same, info = pf.pf_svd_split_conv(Wd, 4, return_info=True)
    assert len(plain) == 3 and all(torch.equal(a, b) for a, b in zip(plain, same))
    assert 1 <= int(info[0]) <= 24 and int(info[1]) == 0


@pytest.mark.parametrize("m,n,kept", [(60, 24, 20), (30, 12, 5), (200, 130, 70), (576, 64, 20)])
def test_zero_rows(m, n, kept):
    """Fewer rows other than zero than columns (filters of pruned inputs): factors and singular values are finite and right, whatever
    the rounding of columns that the rotations cancel; those columns come out zero, and the sweeps end."""
    import paper_2103_03936_amd as pf
    for seed in range(40):
        W = _matrix(m, n, 101 + seed)
        W[np.random.default_rng(seed).permutation(m)[kept:]] = 0.0
        U, V, sigma, info = pf.pf_svd_split(to_gpu(W), n, return_info=True)
        assert int(info[1]) == 0, seed
        assert all(torch.count_nonzero(t[..., kept:]) == 0 for t in (U, V, sigma)), seed
        ref = np.linalg.svd(W.astype(np.float64), compute_uv=False)
        assert np.max(np.abs(sigma.double().cpu().numpy() - ref)) <= 2.0 ** -23 * ref[0], seed
        got = U.double().cpu().numpy() @ V.double().cpu().numpy().T
        assert np.linalg.norm(got - W) <= 2.0 ** -22 * np.linalg.norm(W.astype(np.float64)), seed


@pytest.mark.parametrize("scale", [1e-6, 1e-9, 1e-12, 1e-20, 1e-26])
@pytest.mark.parametrize("lower", [False, True])
def test_blocks_of_very_different_size(scale, lower):
    """Two blocks that share no row and no column, one of them tiny: every singular value to the rounding of its float, whether or not the
    large one's null space holds columns of rounding noise."""
    import paper_2103_03936_amd as pf
    a, b = _matrix(40, 20, 121).astype(np.float64), scale * _matrix(30, 20, 122).astype(np.float64)
    if lower:
        a[8:] = 0.0
    W = np.zeros((70, 40))
    W[:40, ::2], W[40:, 1::2] = a, b
    W = W.astype(np.float32)
    _, _, sigma, info = pf.pf_svd_split(to_gpu(W), 40, return_info=True)
    assert int(info[1]) == 0
    ref = np.concatenate([np.linalg.svd(W[:40, ::2][:8 if lower else 40].astype(np.float64), compute_uv=False),
                          np.linalg.svd(W[40:, 1::2].astype(np.float64), compute_uv=False)])
    got = sigma.double().cpu().numpy()
    assert np.max(np.abs(got[:len(ref)] / ref - 1)) <= 2.0 ** -22
    # (noise: what the rotations of the tiny block's columns round, and twice the rounding of the large one's)
    assert not lower or np.max(got[len(ref):]) <= 2.0 ** -44 * ref[-20] + 2.0 ** -100 * ref[0]


@pytest.mark.parametrize("shape", [(40, 1), (30, 24), (17, 70), (300, 130)])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
def test_not_finite_is_reported(shape, value):
    """A matrix with one element that is not finite: info says so, and so do the factors."""
    import paper_2103_03936_amd as pf
    W = _matrix(*shape, seed=31)
    W[shape[0] // 2, shape[1] // 3] = value
    U, V, sigma, info = pf.pf_svd_split(to_gpu(W), 1, return_info=True)
    assert int(info[1]) != 0
    assert not (torch.isfinite(U).all() and torch.isfinite(V).all() and torch.isfinite(sigma).all())


@pytest.mark.parametrize("m,n,big", [(256, 64, 400.0), (256, 64, 1000.0), (600, 200, 300.0)])
def test_close_singular_values_are_separated(m, n, big):
    """Singular values a relative 1e-6 apart under a few large ones: the vectors themselves, up to sign.  Columns orthogonal to
    t = max(m, n) 2^-52 are mixed by t / (2 d) at most for values a relative d apart, the factors round by 2^-24, and the
    float64 reference is off by 2^-52 sigma_1 / (sigma d)."""
    import paper_2103_03936_amd as pf
    top = n // 8
    s = np.concatenate([big * np.linspace(2, 1, top), 1 + 1e-6 * np.arange(n - top, 0, -1)])
    q1, _ = np.linalg.qr(_matrix(m, n, 41).astype(np.float64))
    q2, _ = np.linalg.qr(_matrix(n, n, 42).astype(np.float64))
    W = ((q1 * s) @ q2.T).astype(np.float32)
    U, V, _, info = pf.pf_svd_split(to_gpu(W), n, return_info=True)
    assert int(info[1]) == 0
    u, sv, vt = np.linalg.svd(W.astype(np.float64), full_matrices=False)
    d = np.min(-np.diff(sv) / sv[1:])
    bound = 2.0 ** -24 + 2.0 ** -52 * (m / (2 * d) + sv[0] / (sv[-1] * d))
    for got, ref in ((U, u), (V, vt.T)):
        got, ref = got.double().cpu().numpy(), ref * np.sqrt(sv)
        err = np.abs(got * np.sign((got * ref).sum(0)) - ref).max(0) / np.abs(ref).max(0)
        assert err.max() <= bound, (err.max(), bound)


@pytest.mark.parametrize("n", [16, 17, 63, 64, 65, 128, 129, 255, 257, 511, 513, 1023, 1025, 1537, 2033, 2048, 2049])
def test_eigenvector_route(n):
    """Both sides of every size at which the tridiagonal preconditioner changes its split (16 columns: Jacobi's), odd sizes, tall and
    nearly square: float32 factors, so the oracle's product to a few roundings, and no rotations left."""
    import paper_2103_03936_amd as pf
    W, r = _matrix(n + 3 if n % 2 else 2 * n, n, seed=51 + n), max(1, n // 4)
    U, V, sigma, info = pf.pf_svd_split(to_gpu(W), r, return_info=True)
    assert int(info[1]) == 0 and int(info[0]) <= 3
    u, s, vt = np.linalg.svd(W.astype(np.float64), full_matrices=False)
    assert np.max(np.abs(sigma.double().cpu().numpy() - s)) <= 2.0 ** -23 * s[0]
    # U and V round by 2^-24 each, element by element
    want = (u[:, :r] * s[:r]) @ vt[:r]
    got = U.double().cpu().numpy() @ V.double().cpu().numpy().T
    assert np.linalg.norm(got - want) <= 2.0 ** -22 * np.linalg.norm(want)


def _uncoupled(m, n, seed):
    """A quarter of the columns zero (pruned filters), two more large and alone in their rows, the others small."""
    W = 1e-2 * _matrix(m, n, seed).astype(np.float64)
    zero, single = np.arange(1, n, 4), [0, n // 4 * 2]
    W[:, zero] = 0.0
    W[:2] = 0.0
    for i, j in enumerate(single):
        W[:, j] = 0.0
        W[i, j] = 10.0 * (i + 1)
    return W.astype(np.float32), zero, single


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("m,n", [(40, 17), (130, 64), (200, 127), (200, 128), (200, 129), (400, 257), (700, 600)])
def test_uncoupled_columns(m, n, transposed):
    """Columns that are orthogonal to all others, zero columns among them: the factors reproduce the matrix (full rank kept) to the
    roundings of its two parts, the rows of zero columns are zero, and nothing is left to rotate."""
    import paper_2103_03936_amd as pf
    W, zero, single = _uncoupled(m, n, 71 + n)
    assert not set(zero) & set(single)
    A = np.ascontiguousarray(W.T) if transposed else W
    U, V, sigma, info = pf.pf_svd_split(to_gpu(A), n, return_info=True)
    assert int(info[1]) == 0 and int(info[0]) <= 3
    U, V = (V, U) if transposed else (U, V)
    assert torch.count_nonzero(V[torch.as_tensor(zero)]) == 0
    assert torch.count_nonzero(sigma[n - len(zero):]) == 0
    got = U.double().cpu().numpy() @ V.double().cpu().numpy().T
    large = np.isin(np.arange(n), single)
    for part in (large, ~large):
        assert np.linalg.norm((got - W)[:, part]) <= 2.0 ** -22 * np.linalg.norm(W[:, part].astype(np.float64))
    ref = np.linalg.svd(W.astype(np.float64), compute_uv=False)
    assert np.max(np.abs(sigma.double().cpu().numpy() - ref)) <= 2.0 ** -23 * ref[0]


@pytest.mark.parametrize("kind", ["zero columns", "diagonal", "zero"])
def test_uncoupled_columns_take_no_longer(kind):
    """Eigenvalues of uncoupled columns may coincide without a second preconditioner: with one, these calls took 1.8 (diagonal) to 8
    (zero columns) times as long as one on an ordinary matrix of their size."""
    import paper_2103_03936_amd as pf
    plain = to_gpu(_matrix(1024, 512, 81))
    other = plain.clone()
    if kind == "zero columns":
        other[:, ::4] = 0
    else:
        other.zero_()
        if kind == "diagonal":
            other[range(512), range(512)] = 1

    def best(X):
        times = []
        for _ in range(8):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            pf.pf_svd_split(X, 128)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        return min(times[2:])

    assert best(other) <= 1.4 * best(plain)


def _lower_rank(kind, m, n, seed):
    """A product of two thin matrices (of a quarter of the rank), or one of which an eighth of the columns are there twice."""
    W = _matrix(m, n, seed)
    if kind == "product":
        return (W[:, :n // 4].astype(np.float64) @ _matrix(n // 4, n, seed + 1)).astype(np.float32)
    W[:, :n // 8] = W[:, n // 2:n // 2 + n // 8]
    return W


@pytest.mark.parametrize("kind", ["product", "twice"])
@pytest.mark.parametrize("m,n", [(40, 17), (96, 96), (200, 129), (300, 256), (700, 600), (1300, 1030), (1700, 1600)])
def test_lower_rank(kind, m, n):
    """Null spaces of many dimensions, on every size of the tridiagonal route: the factors reproduce the matrix and nothing is left to
    rotate."""
    import paper_2103_03936_amd as pf
    W = _lower_rank(kind, m, n, 91 + n)
    U, V, sigma, info = pf.pf_svd_split(to_gpu(W), n, return_info=True)
    assert int(info[1]) == 0
    got = U.double().cpu().numpy() @ V.double().cpu().numpy().T
    assert np.linalg.norm(got - W) <= 2.0 ** -22 * np.linalg.norm(W.astype(np.float64))
    ref = np.linalg.svd(W.astype(np.float64), compute_uv=False)
    assert np.max(np.abs(sigma.double().cpu().numpy() - ref)) <= 2.0 ** -23 * ref[0]


@pytest.mark.parametrize("kind,m,n,times", [("product", 576, 64, 6.2), ("product", 64, 64, 5.2), ("twice", 1024, 512, 9.5)])
def test_lower_rank_takes_one_preconditioner(kind, m, n, times):
    """Eigenvalues that coincide at zero need no second preconditioner; with one, these calls took 7.3, 6.5 and 13 times as long as one
    on an ordinary matrix of their size, now 4.8, 3.9 and 6."""
    import paper_2103_03936_amd as pf

    def best(W):
        W, taken = to_gpu(W), []
        for _ in range(8):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            pf.pf_svd_split(W, n // 4)
            end.record()
            end.synchronize()
            taken.append(start.elapsed_time(end))
        return min(taken[2:])

    ratio = best(_lower_rank(kind, m, n, 83)) / best(_matrix(m, n, 85))
    assert ratio <= times, ratio


@pytest.mark.parametrize("kind", ["orthonormal", "zero rows", "repeated", "diagonal", "graded"])
def test_clustered_matrices(kind):
    """Eigenvalues that coincide, a matrix that falls apart, and values over seven decades: whichever preconditioner runs, the
    factors reproduce the matrix (full rank kept) and nothing is left to rotate."""
    import paper_2103_03936_amd as pf
    m, n = 200, 96
    q, _ = np.linalg.qr(_matrix(m, n, 61).astype(np.float64))
    p, _ = np.linalg.qr(_matrix(n, n, 62).astype(np.float64))
    s = {"repeated": np.repeat([4.0, 2.0, 1.0], n // 3), "graded": np.logspace(0, -7, n)}.get(kind, np.ones(n))
    W = (q * s) @ p.T
    if kind == "zero rows":
        W = _matrix(m, n, 63).astype(np.float64)
        W[:, 10:40] = 0.0
    if kind == "diagonal":
        W = np.zeros((m, n))
        W[np.arange(n), np.arange(n)] = np.arange(n) % 7 + 1.0
    W = W.astype(np.float32)
    U, V, sigma, info = pf.pf_svd_split(to_gpu(W), n, return_info=True)
    assert int(info[1]) == 0
    got = U.double().cpu().numpy() @ V.double().cpu().numpy().T
    assert np.linalg.norm(got - W) <= 2.0 ** -22 * np.linalg.norm(W.astype(np.float64))
    ref = np.linalg.svd(W.astype(np.float64), compute_uv=False)
    assert np.max(np.abs(sigma.double().cpu().numpy() - ref)) <= 2.0 ** -23 * ref[0]


@pytest.mark.parametrize("m,n", [(2049, 2049), (2100, 2056)])
def test_more_columns_than_the_eigenvectors_take(m, n):
    """Jacobi as the preconditioner in a launch of its own.  Bounds as for lower ranks."""
    import paper_2103_03936_amd as pf
    W = _matrix(m, n, 97)
    U, V, sigma, info = pf.pf_svd_split(to_gpu(W), n, return_info=True)
    assert int(info[1]) == 0
    w = torch.from_numpy(W).double()
    assert float((U.double().cpu() @ V.double().cpu().T - w).norm()) <= 2.0 ** -22 * float(w.norm())
    ref = torch.linalg.eigvalsh(w.T @ w).clamp_min(0).sqrt().flip(0)  # (to 2^-53 of the largest eigenvalue, 2^-26 of its root)
    assert float((sigma.double().cpu() - ref).abs().max()) <= 2.0 ** -23 * float(ref[0])


@pytest.mark.parametrize("m,n", [(20000, 16), (20000, 40), (9000, 100)])
def test_tall_matrices_of_lower_rank(m, n):
    """Workgroups without a pair of columns wait while few sweep for long: preconditioner and B.  Bounds as for lower ranks."""
    import paper_2103_03936_amd as pf
    W = _lower_rank("product", m, n, 99)
    U, V, sigma, info = pf.pf_svd_split(to_gpu(W), n, return_info=True)
    assert int(info[1]) == 0 and int(info[0]) > 2
    w = torch.from_numpy(W).double()
    assert float((U.double().cpu() @ V.double().cpu().T - w).norm()) <= 2.0 ** -22 * float(w.norm())
    ref = np.linalg.svd(W.astype(np.float64), compute_uv=False)
    assert np.max(np.abs(sigma.double().cpu().numpy() - ref)) <= 2.0 ** -23 * ref[0]


@pytest.mark.parametrize("n", [1, 5, 16])
@pytest.mark.parametrize("m", [2048, 2049, 30001])
def test_few_columns_of_many_rows(m, n):
    """Both sides of the rows from which Jacobi's preconditioner and the products have launches of their own.  Bounds as above."""
    import paper_2103_03936_amd as pf
    W = _matrix(m, n, 101)
    U, V, sigma, info = pf.pf_svd_split(to_gpu(W), n, return_info=True)
    assert int(info[1]) == 0 and int(info[0]) <= 2
    w = torch.from_numpy(W).double()
    assert float((U.double().cpu() @ V.double().cpu().T - w).norm()) <= 2.0 ** -22 * float(w.norm())
    ref = np.linalg.svd(W.astype(np.float64), compute_uv=False)
    assert np.max(np.abs(sigma.double().cpu().numpy() - ref)) <= 2.0 ** -23 * ref[0]
