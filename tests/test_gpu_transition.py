"""GPU parity of the direct transition W -> (U, S, V) (Algorithm 1, Eq. 3, Algorithm 2), called
through the C ABI, against the fp64 numpy oracle on the same seeded inputs.  Integer results
(ternary vectors) must match exactly; fp64 results within the tolerances stated at each check."""
import numpy as np
import pytest

from oracle import transition as tr

pytestmark = pytest.mark.gpu

THETA = 0.576


@pytest.fixture(scope="module")
def tsvd():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no fallback")
    import paper_2308_07641_amd as t
    t.load_library()
    return t


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("n", [1, 2, 7, 64, 255, 256, 257, 1000, 4096, 8192])
def test_ternarize_matches_the_oracle_exactly(tsvd, n):
    """Algorithm 1 on Laplace, Gaussian and tied (small-integer) vectors, several thresholds; rows
    for which no ternary vector exists must be flagged and zero, as the oracle raises."""
    rng = np.random.default_rng(1000 + n)
    rows = [rng.laplace(size=n), rng.standard_normal(n), rng.integers(-3, 4, size=n).astype(np.float64),
            np.abs(rng.standard_normal(n)) + 5.0, np.zeros(n), -rng.laplace(size=n) * 1e-30]
    x = np.stack(rows)
    for theta in (0.2, THETA, np.pi / 4, 1.2):
        print(f"case ternarize n={n} theta={theta:.3f}", flush=True)
        t, status = tsvd.tsvd_ternarize(_dev(x), theta)
        t, status = t.cpu().numpy(), status.cpu().numpy()
        for r in range(x.shape[0]):
            try:
                want = tr.ternarize(x[r], theta)
                assert status[r] == 0, (r, theta)
                assert np.array_equal(t[r], want), (r, theta)
            except ValueError:
                assert status[r] == 1 and not t[r].any(), (r, theta)


@pytest.mark.parametrize("M,N,K", [(9, 7, 5), (64, 48, 40), (130, 70, 300), (512, 256, 96)])
def test_fit_scales_and_residual(tsvd, M, N, K):
    """Eq. (3) and R = W - U diag(S) V: S against the oracle's pseudo-inverse solution (relative
    1e-9: conjugate gradients in fp64 to a residual of 1e-13), R and its norm to rounding."""
    rng = np.random.default_rng(M + N + K)
    U = rng.choice([-1, 0, 1], size=(M, K), p=[0.15, 0.7, 0.15]).astype(np.int8)
    V = rng.choice([-1, 0, 1], size=(K, N), p=[0.15, 0.7, 0.15]).astype(np.int8)
    W = rng.laplace(size=(M, N))
    print(f"case fit M={M} N={N} K={K}", flush=True)
    S, iters = tsvd.tsvd_fit_scales(_dev(U), _dev(V), _dev(W))
    S = S.cpu().numpy()
    want = tr.fit_scales(U, V, W)
    Rw = W - (U * want[None, :]) @ V.astype(np.float64)
    Rg = W - (U * S[None, :]) @ V.astype(np.float64)
    assert int(iters.cpu()[0]) > 0                                               # converged
    if K <= min(M, N):                                                           # unique solution
        assert np.max(np.abs(S - want)) <= 1e-9 * np.max(np.abs(want))
    assert abs(np.linalg.norm(Rg) - np.linalg.norm(Rw)) <= 1e-10 * np.linalg.norm(W)   # the same optimum
    R, n2 = tsvd.tsvd_residual(_dev(W), _dev(U), _dev(S), _dev(V))
    assert np.max(np.abs(R.cpu().numpy() - Rg)) <= 1e-12 * np.max(np.abs(W)) * K
    assert abs(float(n2.cpu()[0]) - np.sum(Rg * Rg)) <= 1e-12 * np.sum(W * W)


def test_fit_scales_minimum_norm_for_duplicated_components(tsvd):
    rng = np.random.default_rng(5)
    U = rng.integers(-1, 2, size=(20, 6)).astype(np.int8)
    V = rng.integers(-1, 2, size=(6, 15)).astype(np.int8)
    U[:, 5], V[5, :] = U[:, 2], V[2, :]
    W = rng.standard_normal((20, 15))
    S, _ = tsvd.tsvd_fit_scales(_dev(U), _dev(V), _dev(W))
    assert np.max(np.abs(S.cpu().numpy() - tr.fit_scales(U, V, W))) <= 1e-9


@pytest.mark.parametrize("M,N", [(40, 30), (512, 256), (100, 700)])
def test_leading_singular_pair(tsvd, M, N):
    """Against the library SVD on a matrix with a clear leading component and on a plain Laplace
    matrix, whose leading singular values are close (the squarings must still separate them)."""
    rng = np.random.default_rng(M + N)
    u0 = rng.standard_normal(M); u0 /= np.linalg.norm(u0)
    v0 = rng.standard_normal(N); v0 /= np.linalg.norm(v0)
    noise = rng.laplace(size=(M, N))
    for planted in (True, False):
        R = noise + (2.0 * np.linalg.norm(noise, 2) * np.outer(u0, v0) if planted else 0.0)
        u, sigma, v, iters = tsvd.tsvd_leading_singular_pair(_dev(R))
        u, sigma, v = u.cpu().numpy(), float(sigma.cpu()[0]), v.cpu().numpy()
        ur, sr, vr = np.linalg.svd(R, full_matrices=False)
        print(f"case leading pair M={M} N={N} planted={planted}: {int(iters.cpu()[0])} steps, gap {1 - sr[1] / sr[0]:.4f}", flush=True)
        assert abs(np.linalg.norm(u) - 1) < 1e-12 and abs(np.linalg.norm(v) - 1) < 1e-12
        assert abs(sigma - sr[0]) <= 1e-12 * sr[0]
        sign = np.sign(u @ ur[:, 0])
        # (the vectors are determined to about rounding / gap)
        assert np.max(np.abs(sign * u - ur[:, 0])) < 1e-8 and np.max(np.abs(sign * v - vr[0, :])) < 1e-8


@pytest.mark.parametrize("M,N", [(1, 1), (1, 70), (70, 1), (64, 64), (65, 63), (129, 200), (384, 400), (385, 385), (500, 420),
                                 (257, 300), (320, 321), (330, 321), (513, 513), (576, 600), (640, 641), (641, 700)])
def test_leading_singular_pair_by_squarings_at_tile_edges(tsvd, M, N):
    """Sizes around the tiles of the squaring kernels (16 and 32 rows, padding to 64, the change at 384; the most tiles that are dealt to the XCDs by groups of
    rows, up to 320 with the smaller ones and 640 with the larger, and one more), both orientations;
    a rank-one matrix (done after one squaring) and a pair of equal leading singular values (never of rank one: the pair must
    still be a singular pair)."""
    rng = np.random.default_rng(100 * M + N)
    cases = {"laplace": rng.laplace(size=(M, N)), "rank one": np.outer(rng.standard_normal(M), rng.standard_normal(N)),
             "zero": np.zeros((M, N))}
    if min(M, N) > 4:
        A, _ = np.linalg.qr(rng.standard_normal((M, 4)))
        B, _ = np.linalg.qr(rng.standard_normal((N, 4)))
        cases["equal"] = (A * np.array([3.0, 3.0, 1.0, 0.5])[None, :]) @ B.T
    for name, R in cases.items():
        print(f"case squarings M={M} N={N} {name}", flush=True)
        u, sigma, v, steps = tsvd.tsvd_leading_singular_pair(_dev(R))
        u, sigma, v = u.cpu().numpy(), float(sigma.cpu()[0]), v.cpu().numpy()
        if name == "zero":
            assert sigma == 0.0 and not u.any() and not v.any()
            continue
        top = np.linalg.svd(R, compute_uv=False)[0]
        assert abs(sigma - top) <= 1e-12 * top
        assert abs(np.linalg.norm(u) - 1) < 1e-12 and abs(np.linalg.norm(v) - 1) < 1e-12
        assert np.linalg.norm(R @ v - sigma * u) <= 1e-12 * top and np.linalg.norm(R.T @ u - sigma * v) <= 1e-12 * top
        start = 1.0 + 0.5 * np.sin(1.0 + 0.7 * np.arange(N))
        assert v @ start > 0                                                        # the sign is that of the start vector


@pytest.mark.parametrize("M,N", [(128, 64), (64, 128), (500, 420)])
@pytest.mark.parametrize("cos", [0.0, 1e-12, 1e-6])
def test_leading_singular_pair_whatever_its_angle_to_the_start_vector(tsvd, M, N, cos):
    """The leading direction is orthogonal to the fixed start vector, or nearly: the pair must be as exact as any other."""
    rng = np.random.default_rng(M + N)
    n = min(M, N)
    start = 1.0 + 0.5 * np.sin(1.0 + 0.7 * np.arange(N))
    start /= np.linalg.norm(start)
    v0 = rng.standard_normal(N)
    v0 -= start * (start @ v0)
    v0 = np.sqrt(1.0 - cos * cos) * v0 / np.linalg.norm(v0) + cos * start
    A = np.linalg.qr(rng.standard_normal((M, n)))[0]
    B = np.linalg.qr(np.column_stack([v0, rng.standard_normal((N, n - 1))]))[0]
    R = (A * 0.9 ** np.arange(n)) @ B.T
    print(f"case pair off the start vector M={M} N={N} cos={cos}", flush=True)
    u, sigma, v, _ = tsvd.tsvd_leading_singular_pair(_dev(R))
    u, sigma, v = u.cpu().numpy(), float(sigma.cpu()[0]), v.cpu().numpy()
    assert abs(sigma - 1.0) <= 1e-12
    assert np.linalg.norm(R @ v - sigma * u) <= 1e-12 and np.linalg.norm(R.T @ u - sigma * v) <= 1e-12
    assert abs(abs(v @ v0) - 1.0) <= 1e-12


@pytest.mark.parametrize("M,N", [(2060, 2048), (2048, 2060), (2049, 2060)])
def test_leading_singular_pair_where_the_method_changes(tsvd, M, N):
    """The largest size of the squarings, both orientations, and the first of the Lanczos steps; the leading vectors are
    the last unit vectors, so the column that the squarings pick is the last one."""
    rng = np.random.default_rng(M)
    n = min(M, N)
    A, B = (np.linalg.qr(np.column_stack([np.eye(L)[:, -1], rng.standard_normal((L, n - 1))]))[0] for L in (M, N))
    R = (A * np.concatenate([[1.0], np.linspace(0.97, 0.0, n - 1)])) @ B.T
    print(f"case pair at the change M={M} N={N}", flush=True)
    u, sigma, v, steps = tsvd.tsvd_leading_singular_pair(_dev(R))
    u, sigma, v = u.cpu().numpy(), float(sigma.cpu()[0]), v.cpu().numpy()
    assert (int(steps.cpu()[0]) > 16) == (n > 2048)
    assert abs(sigma - 1.0) <= 1e-12 and abs(abs(u[-1]) - 1.0) <= 1e-12 and abs(abs(v[-1]) - 1.0) <= 1e-12
    assert np.linalg.norm(R @ v - sigma * u) <= 1e-12 and np.linalg.norm(R.T @ u - sigma * v) <= 1e-12


@pytest.mark.parametrize("M,N", [(128, 64), (64, 128), (500, 420)])
@pytest.mark.parametrize("power", [330, -330, 490, -490])
def test_leading_singular_pair_of_very_large_and_small_entries(tsvd, M, N, power):
    """Entries of 1e99 to 1e147 and their inverses: scaling a matrix by a power of two scales sigma by it and leaves the vectors."""
    R = np.random.default_rng(M + N).laplace(size=(M, N))
    print(f"case pair range M={M} N={N} power={power}", flush=True)
    u, sigma, v, _ = tsvd.tsvd_leading_singular_pair(_dev(R))
    us, sigmas, vs, _ = tsvd.tsvd_leading_singular_pair(_dev(np.ldexp(R, power)))
    assert abs(np.ldexp(float(sigmas.cpu()[0]), -power) - float(sigma.cpu()[0])) <= 1e-13 * float(sigma.cpu()[0])
    assert (us - u).abs().max() <= 1e-11 and (vs - v).abs().max() <= 1e-11
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(R), THETA, 0.0, 3)
    Us, Ss, Vs, errss, status_s = tsvd.tsvd_transition(_dev(np.ldexp(R, power)), THETA, 0.0, 3)
    assert status == status_s == 0
    assert (U == Us).all() and (V == Vs).all()
    assert np.max(np.abs(np.ldexp(Ss.cpu().numpy(), -power) - S.cpu().numpy())) <= 1e-12 * float(S.abs().max())


def test_transition_follows_the_oracle_on_separated_spectra(tsvd):
    """Algorithm 2 end to end.  W is built with well separated singular values, so every residual
    has a clear leading pair and both sides must pick the same ternary vectors: U S V, S and the
    error path are compared (columns of U / rows of V up to the common sign of a singular pair)."""
    rng = np.random.default_rng(9)
    M, N, r = 96, 80, 12
    A, _ = np.linalg.qr(rng.standard_normal((M, r)))
    B, _ = np.linalg.qr(rng.standard_normal((N, r)))
    W = (A * (2.0 ** -np.arange(r))[None, :]) @ B.T
    Uo, So, Vo, eo = tr.transition(W, THETA, max_rank=10)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), THETA, 0.0, 10)
    assert status == 0
    U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
    assert U.shape == Uo.shape and V.shape == Vo.shape
    for k in range(10):
        sign = 1 if np.array_equal(U[:, k], Uo[:, k]) else -1
        assert np.array_equal(sign * U[:, k], Uo[:, k]) and np.array_equal(sign * V[k, :], Vo[k, :]), k
    assert np.max(np.abs(S - So)) <= 1e-8 * np.max(np.abs(So))
    assert np.max(np.abs(np.array(errs) - np.array(eo))) <= 1e-9


@pytest.mark.parametrize("q", [2, 3, 4])
def test_transition_with_several_components_per_iteration(tsvd, q):
    """q > 1: the top q singular triples of one residual per iteration (by deflation on the GPU, by a full SVD in the
    oracle).  Separated spectrum: both must pick the same ternary vectors, scales and errors; a rank limit that q does
    not divide ends with a shorter last iteration."""
    rng = np.random.default_rng(9)           # (a seed at which every leading vector has a ternary neighbour within theta)
    M, N, r = 96, 80, 14
    A, _ = np.linalg.qr(rng.standard_normal((M, r)))
    B, _ = np.linalg.qr(rng.standard_normal((N, r)))
    W = (A * (1.7 ** -np.arange(r))[None, :]) @ B.T
    rank = 12
    Uo, So, Vo, eo = tr.transition(W, THETA, q=q, max_rank=rank)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), THETA, 0.0, rank, q=q)
    assert status == 0
    U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
    assert U.shape == Uo.shape == (M, rank) and V.shape == Vo.shape
    for k in range(rank):
        sign = 1 if np.array_equal(U[:, k], Uo[:, k]) else -1
        assert np.array_equal(sign * U[:, k], Uo[:, k]) and np.array_equal(sign * V[k, :], Vo[k, :]), k
    assert np.max(np.abs(S - So)) <= 1e-8 * np.max(np.abs(So))
    assert np.max(np.abs(np.array(errs)[q - 1::q] - np.array(eo))) <= 1e-9          # one error per iteration
    # rank limit 7 with q = 3: iterations of 3, 3 and 1 components; the first six equal the oracle's two rounds
    if q == 3:
        U7, S7, V7, e7, status = tsvd.tsvd_transition(_dev(W), THETA, 0.0, 7, q=3)
        assert status == 0 and U7.shape == (M, 7) and len(e7) == 7
        Uo6 = tr.transition(W, THETA, q=3, max_rank=6)[0]
        U7 = U7.cpu().numpy()
        assert all(np.array_equal(U7[:, k], Uo6[:, k]) or np.array_equal(-U7[:, k], Uo6[:, k]) for k in range(6))


@pytest.mark.parametrize("q", [1, 2])
@pytest.mark.parametrize("M,N", [(96, 80), (80, 96)])
def test_transition_with_a_nearly_degenerate_residual(tsvd, M, N, q):
    """The leading singular values of W are 1e-7 of themselves apart, which takes 27 squarings: the iteration that meets them is taken
    again with more of them, those after it are not, and all follow the oracle."""
    rng = np.random.default_rng(10)          # (as above: with ternary neighbours, and gaps of 2e-2 from the second iteration on)
    r = 12
    A, _ = np.linalg.qr(rng.standard_normal((M, r)))
    B, _ = np.linalg.qr(rng.standard_normal((N, r)))
    sv = 1.7 ** -np.arange(r)
    sv[1] = 1.0 - 1e-7
    W = (A * sv[None, :]) @ B.T
    rank = 8
    Uo, So, Vo, eo = tr.transition(W, THETA, q=q, max_rank=rank)
    print(f"case nearly degenerate {M} {N} {q}", flush=True)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), THETA, 0.0, rank, q=q)
    assert status == 0
    U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
    for k in range(rank):
        sign = 1 if np.array_equal(U[:, k], Uo[:, k]) else -1
        assert np.array_equal(sign * U[:, k], Uo[:, k]) and np.array_equal(sign * V[k, :], Vo[k, :]), k
    assert np.max(np.abs(S - So)) <= 1e-8 * np.max(np.abs(So))
    assert np.max(np.abs(np.array(errs)[q - 1::q] - np.array(eo))) <= 1e-9


@pytest.mark.parametrize("q,rank", [(1, 14), (2, 12), (3, 14)])
def test_transition_with_coinciding_components(tsvd, q, rank):
    """The residual's leading pair has its largest entries where the component before it was taken, so the same component is
    appended again: the Gram matrix of Eq. (3) is singular and the loop leaves its Cholesky factor for conjugate gradients, for this
    and all later iterations.  Residual, errors and factors must still be the oracle's."""
    rng = np.random.default_rng(8)          # (gaps of 1e-2 at least in every iteration)
    M, N, half, theta = 60, 50, 24, 1.0
    c, r = np.zeros(M), np.zeros(N)
    c[1:half], r[1:half] = rng.uniform(0.8, 1.2, half - 1), rng.uniform(0.8, 1.2, half - 1)
    c, r = c / np.linalg.norm(c), r / np.linalg.norm(r)
    W = 0.5 * np.outer(c, r)
    W[0] += r
    W[:, 0] += c
    W[0, 0] = 3.0            # then the pair of [[0, 1], [1, 0.5]] in the bases (e_0, c), (e_0, r) leads: (0.62, 0.79)
    A = np.linalg.qr(rng.standard_normal((M - half, 6)))[0]
    B = np.linalg.qr(rng.standard_normal((N - half, 6)))[0]
    W[half:, half:] = (A * np.array([2.0, 1.1, 0.9, 0.7, 0.4, 0.2])) @ B.T
    Uo, So, Vo, eo = tr.transition(W, theta, q=q, max_rank=rank - rank % q)
    G = (Uo.T @ Uo).astype(float) * (Vo @ Vo.T)
    first = next(k for k in range(1, Uo.shape[1] + 1) if np.linalg.matrix_rank(G[:k, :k]) < k)      # components up to the first repeated one
    print(f"case coinciding components q={q}: repeated at {first} of {Uo.shape[1]}", flush=True)
    assert first < Uo.shape[1]
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), theta, 0.0, rank, q=q)
    assert status == 0 and U.shape == (M, rank)
    U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
    for k in range(Uo.shape[1]):
        sign = 1 if np.array_equal(U[:, k], Uo[:, k]) else -1
        assert np.array_equal(sign * U[:, k], Uo[:, k]) and np.array_equal(sign * V[k, :], Vo[k, :]), k
    assert np.max(np.abs(np.array(errs)[q - 1:len(eo) * q:q] - np.array(eo))) <= 1e-9
    best = W - tr.reconstruction(U, tr.fit_scales(U, V, W), V)
    assert np.max(np.abs(W - tr.reconstruction(U, S, V) - best)) <= 1e-9


def test_transition_wide_matrix_and_rank_limit(tsvd):
    """M < N, exit by the rank limit, status and shapes; the first components equal the oracle's."""
    W = np.random.default_rng(12).laplace(size=(48, 160))
    Uo, So, Vo, eo = tr.transition(W, THETA, max_rank=6)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), THETA, 0.0, 6)
    assert status == 0 and U.shape == (48, 6) and V.shape == (6, 160) and len(errs) == 6
    U, V = U.cpu().numpy(), V.cpu().numpy()
    for k in range(6):
        sign = 1 if np.array_equal(U[:, k], Uo[:, k]) else -1
        assert np.array_equal(sign * U[:, k], Uo[:, k]) and np.array_equal(sign * V[k, :], Vo[k, :]), k
    assert np.max(np.abs(np.array(errs) - np.array(eo))) <= 1e-9


@pytest.mark.parametrize("M,N", [(2049, 2049), (2100, 2500)])
def test_transition_beyond_the_sizes_of_the_squarings(tsvd, M, N):
    """min(M, N) above 2048: leading pairs by Lanczos steps.  W has rank five, so the residual of K components has rank 5 + K and its
    leading pair follows from thin factors.  Exit by the rank limit, by the tolerance and by a vector without a ternary neighbour."""
    rng = np.random.default_rng(M + N)
    A = np.linalg.qr(rng.standard_normal((M, 5)))[0] * 2.0 ** -np.arange(5)
    B = np.linalg.qr(rng.standard_normal((N, 5)))[0].T
    W = A @ B
    Uo, Vo, scales, errors = np.zeros((M, 0)), np.zeros((0, N)), [np.zeros(0)], []
    for _ in range(3):
        ql, rl = np.linalg.qr(np.hstack([A, -Uo * scales[-1]]))
        qr, rr = np.linalg.qr(np.vstack([B, Vo]).T)
        a, _, b = np.linalg.svd(rl @ rr.T)
        Uo = np.column_stack([Uo, tr.ternarize(ql @ a[:, 0], THETA)])
        Vo = np.vstack([Vo, tr.ternarize(qr @ b[0, :], THETA)])
        scales.append(np.linalg.solve((Uo.T @ Uo) * (Vo @ Vo.T), np.einsum("mk,mk->k", Uo, A @ (B @ Vo.T))))
        errors.append(np.linalg.norm(W - (Uo * scales[-1]) @ Vo) / np.linalg.norm(W))
    for K, tol in ((3, 0.0), (2, 0.5 * (errors[0] + errors[1]))):
        print(f"case transition {M} {N} tol={tol}", flush=True)
        U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), THETA, tol, 3)
        assert status == 0 and U.shape == (M, K) and V.shape == (K, N)
        U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
        for k in range(K):
            sign = 1 if np.array_equal(U[:, k], Uo[:, k]) else -1
            assert np.array_equal(sign * U[:, k], Uo[:, k]) and np.array_equal(sign * V[k, :], Vo[k, :]), k
        assert np.max(np.abs(S - scales[K])) <= 1e-8 * np.max(np.abs(S))
        assert np.max(np.abs(np.array(errs) - np.array(errors[:K]))) <= 1e-9
    with pytest.raises(tsvd.TsvdError):
        tsvd.tsvd_transition(_dev(W), 0.05, 0.0, 3)


def test_transition_reports_a_vector_without_ternary_neighbour(tsvd):
    """At a tiny theta no ternary vector is close enough: the oracle raises, the GPU call returns
    the value error with rank 0."""
    W = np.random.default_rng(13).laplace(size=(40, 30))
    with pytest.raises(ValueError):
        tr.transition(W, 0.05, max_rank=3)
    lib = tsvd.load_library()
    import ctypes, torch
    Wd = _dev(W)
    U = torch.zeros((40, 3), dtype=torch.int8, device="cuda:0"); V = torch.zeros((3, 30), dtype=torch.int8, device="cuda:0")
    S = torch.zeros((3,), dtype=torch.float64, device="cuda:0")
    rank = ctypes.c_int64(-1)
    st = lib.tsvd_transition(Wd.data_ptr(), 40, 30, 0.05, 0.0, 3, U.data_ptr(), S.data_ptr(), V.data_ptr(), ctypes.byref(rank), None, None)
    assert st == 2 and rank.value == 0


def test_transition_on_a_laplace_matrix(tsvd):
    """The paper's random-matrix setting (Laplace entries, theta = 0.576), [128, 64] to tolerance
    7 %: neighbouring singular values are close there, so the leading pair is not unique to
    rounding and the greedy paths may part; what both must satisfy is checked: every scale
    vector is the least-squares optimum for the chosen factors, the error never increases, the
    tolerance is met with about the oracle's rank, and the non-zero rate is about 0.29."""
    W = np.random.default_rng(3).laplace(size=(128, 64))
    Uo, So, Vo, eo = tr.transition(W, THETA, tol=0.07)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), THETA, 0.07, 400)
    assert status == 0
    U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
    K = U.shape[1]
    print(f"case transition laplace: GPU rank {K}, oracle rank {Uo.shape[1]}", flush=True)
    assert set(np.unique(U)) <= {-1, 0, 1} and set(np.unique(V)) <= {-1, 0, 1}
    assert all(b <= a + 1e-9 for a, b in zip(errs, errs[1:]))
    assert errs[-1] <= 0.07 < errs[-2]
    R = W - (U * S[None, :]) @ V.astype(np.float64)
    assert abs(np.linalg.norm(R) / np.linalg.norm(W) - errs[-1]) < 1e-9
    Sopt = tr.fit_scales(U, V, W)
    Ropt = W - (U * Sopt[None, :]) @ V.astype(np.float64)
    assert np.linalg.norm(R) <= np.linalg.norm(Ropt) * (1 + 1e-9)
    assert abs(K - Uo.shape[1]) <= 0.05 * Uo.shape[1] + 2
    r = (np.count_nonzero(U) + np.count_nonzero(V)) / (U.size + V.size)
    assert 0.25 < r < 0.33


def test_transition_scratch_is_reused_by_calls_of_any_size_thread_and_stream(tsvd):
    """Scratch that other sizes left behind, threads with streams of their own at the same time, more of them than pieces are kept, and calls after the
    scratch was given back: every result is the one of a call on fresh scratch."""
    import threading
    import torch
    rng = np.random.default_rng(21)
    cases = [(96, 80, 5, 1), (40, 130, 6, 2), (300, 64, 4, 1), (130, 129, 5, 3), (20, 70, 3, 1), (1500, 900, 2, 1)]
    Ws = [_dev(rng.laplace(size=c[:2])) for c in cases]
    def run(i, stream=None):
        M, N, rank, q = cases[i]
        U, S, V, errs, status = tsvd.tsvd_transition(Ws[i], 0.65, 0.0, rank, stream=stream, q=q)
        (stream or torch.cuda.current_stream()).synchronize()
        return U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy(), errs, status
    def same(a, b):
        return all(np.array_equal(x, y) for x, y in zip(a, b))
    want = []
    for i in range(len(cases)):
        tsvd.tsvd_transition_release()
        want.append(run(i))
    print("case transition scratch", flush=True)
    for i in [0, 3, 1, 5, 0, 2, 4, 3, 5, 1]:
        assert same(run(i), want[i]), i
    got = {}
    def work(t):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for i in range(len(cases)):
                got[t, i] = run((i + t) % len(cases), stream)
    threads = [threading.Thread(target=work, args=(t,)) for t in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(got) == 36 and all(same(r, want[(i + t) % len(cases)]) for (t, i), r in got.items())
    tsvd.tsvd_transition_release()
    assert same(run(1), want[1])


def test_transition_is_refused_under_capture(tsvd):
    """The host waits for the device, so a transition cannot be captured: with scratch at hand or without it is refused before anything is enqueued, the capture stays
    whole, and the graph's replays are those of its other work."""
    import torch
    W = _dev(np.random.default_rng(22).laplace(size=(140, 130)))
    want = [t.clone() for t in tsvd.tsvd_transition(W, 0.65, 0.0, 6)[:3]]
    x = torch.zeros(1000, device="cuda:0")
    for fresh in (False, True):
        if fresh:
            tsvd.tsvd_transition_release()
        print(f"case transition under capture, {'no ' if fresh else ''}scratch at hand", flush=True)
        out = (torch.zeros((140, 6), dtype=torch.int8, device="cuda:0"), torch.zeros((6,), dtype=torch.float64, device="cuda:0"), torch.zeros((6, 130), dtype=torch.int8, device="cuda:0"))
        import ctypes
        rank = ctypes.c_int64(-1)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            x.add_(1.0)
            st = tsvd.load_library().tsvd_transition_q(W.data_ptr(), 140, 130, 0.65, 0.0, 6, 1, out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(), ctypes.byref(rank), None,
                                                       torch.cuda.current_stream().cuda_stream)
        assert st == 4 and rank.value == 0
        x.zero_()
        for replay in range(3):
            graph.replay()
            got = tsvd.tsvd_transition(W, 0.65, 0.0, 6)
            assert all(torch.equal(a, b) for a, b in zip(got, want)), replay
            assert torch.equal(x, torch.full_like(x, replay + 1.0)) and all(int(t.abs().sum()) == 0 for t in out)


def test_transition_of_equal_singular_values(tsvd):
    """A Hadamard matrix: all singular values equal, so no number of squarings leaves a matrix of low rank and any vector will do; the
    pair taken is a unit vector and a column (or row), which is ternary, and every component removes one of 32."""
    H = np.ones((1, 1))
    for _ in range(5):
        H = np.block([[H, H], [H, -H]])
    print("case equal singular values", flush=True)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(3.0 * H), THETA, 0.0, 4)
    assert status == 0 and U.shape == (32, 4)
    assert np.max(np.abs(np.array(errs) - np.sqrt(1.0 - np.arange(1, 5) / 32.0))) <= 1e-12


@pytest.mark.parametrize("M,N", [(64, 65), (70, 60), (300, 250), (768, 790), (769, 800)])
def test_transition_with_many_close_singular_values(tsvd, M, N):
    """Twenty leading singular values within a tenth of each other: the squarings end with a dozen directions, at the sizes on both sides of a
    workgroup's and of the largest whose end is factorised; each residual's pair is separated by 5e-3, and all must follow the oracle."""
    rng = np.random.default_rng(12)
    r = 24
    A = np.linalg.qr(rng.standard_normal((M, r)))[0]
    B = np.linalg.qr(rng.standard_normal((N, r)))[0]
    W = (A * np.concatenate([1.0 - 0.005 * np.arange(20), [0.5, 0.4, 0.3, 0.2]])) @ B.T
    rank = 3
    Uo, So, Vo, eo = tr.transition(W, THETA, max_rank=rank)
    print(f"case many close {M} {N}", flush=True)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), THETA, 0.0, rank)
    assert status == 0
    U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
    for k in range(rank):
        sign = 1 if np.array_equal(U[:, k], Uo[:, k]) else -1
        assert np.array_equal(sign * U[:, k], Uo[:, k]) and np.array_equal(sign * V[k, :], Vo[k, :]), k
    assert np.max(np.abs(np.array(errs) - np.array(eo))) <= 1e-9


def _of_spectrum(M, N, s, seed):
    rng = np.random.default_rng(seed)
    return (np.linalg.qr(rng.standard_normal((M, len(s))))[0] * s) @ np.linalg.qr(rng.standard_normal((N, len(s))))[0].T


def _follows_the_oracle(tsvd, W, theta, rank, q):
    """A transition against the oracle; (kept, taken again) of its shifted iterations"""
    Uo, So, Vo, eo = tr.transition(W, theta, q=q, max_rank=rank)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(W), theta, 0.0, rank, q=q)
    shifts = tsvd.tsvd_tuning_transition_shifts()
    assert status == 0
    U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
    for k in range(rank):
        sign = 1 if np.array_equal(U[:, k], Uo[:, k]) else -1
        assert np.array_equal(sign * U[:, k], Uo[:, k]) and np.array_equal(sign * V[k, :], Vo[k, :]), k
    assert np.max(np.abs(S - So)) <= 1e-8 * np.max(np.abs(So))
    assert abs(errs[-1] - eo[-1]) <= 1e-9
    return shifts


SHIFT_SPECTRA = {
    "steps": 1.0 - 0.006 * np.arange(60),                                    # shifts that hold from the second pair on
    "fall": 3.0 ** -np.arange(24),                                           # the second eigenvalue is lost beside the first: no shift
    "shelf": np.concatenate([1.0 - 0.006 * np.arange(4), 0.2 - 0.002 * np.arange(60)]),      # a step down behind a few
}
SHIFT_SIZES = [(150, 129, 2), (128, 128, 1), (129, 300, 3), (200, 384, 4), (385, 400, 5), (400, 385, 6)]


@pytest.mark.parametrize("spectrum", list(SHIFT_SPECTRA))
@pytest.mark.parametrize("M,N,seed", SHIFT_SIZES + [(127, 300, 7), (300, 127, 8)])
def test_pairs_squared_with_shifts_follow_the_oracle(tsvd, M, N, seed, spectrum):
    """Nine components, at the smallest shorter side that is shifted and the largest that is not, and on both sides of the one where tiles of 32 begin, either side the
    shorter: where the pair before leaves a shift, leaves none, and where there is a step between the two."""
    print(f"case shifts {M} {N} {spectrum}", flush=True)
    kept, again = _follows_the_oracle(tsvd, _of_spectrum(M, N, SHIFT_SPECTRA[spectrum], seed), 0.65, 9, 1)
    assert again == 0
    assert kept >= 4 if spectrum == "steps" and min(M, N) >= 128 else kept == 0 or (spectrum == "shelf" and min(M, N) >= 128), kept


@pytest.mark.parametrize("M,N,seed", [(150, 129, 2), (129, 300, 3), (400, 385, 6)])
def test_three_pairs_an_iteration_are_not_shifted(tsvd, M, N, seed):
    print(f"case shifts {M} {N}, three an iteration", flush=True)
    assert _follows_the_oracle(tsvd, _of_spectrum(M, N, SHIFT_SPECTRA["steps"], seed), 0.65, 9, 3) == (0, 0)


@pytest.mark.parametrize("M,N,seed,spectrum,squarings", [size + ("steps", 3) for size in SHIFT_SIZES] + [(150, 129, 2, "squares", 8)])
def test_iterations_whose_shifts_do_not_hold_are_taken_again(tsvd, M, N, seed, spectrum, squarings):
    """Shifts where the rule takes none: too few squarings leave more than sixteen directions, and of a spectrum that falls like 1 / k^2 a pair's leading value lies below what
    the one before led to expect, so that none counts.  The device tells both, and they are done again without."""
    s = SHIFT_SPECTRA["steps"] if spectrum == "steps" else (1.0 + np.arange(60)) ** -2.0
    print(f"case shifts do not hold {M} {N} {spectrum} {squarings}", flush=True)
    try:
        tsvd.tsvd_tuning_set("TSVD_TRANSITION_SHIFTED", squarings)
        kept, again = _follows_the_oracle(tsvd, _of_spectrum(M, N, s, seed), 0.65, 9, 1)
    finally:
        tsvd.tsvd_tuning_reset()
    assert again >= 1, (kept, again)


UNSHIFTED_SPECTRA = {
    "power 1/2": (1.0 + np.arange(120)) ** -0.5,
    "power 1": (1.0 + np.arange(120)) ** -1.0,
    "power 2": (1.0 + np.arange(120)) ** -2.0,
    "halves": 0.5 ** np.arange(60),
    "thirds": 3.0 ** -np.arange(24),
    "groups": 0.9 ** (np.arange(120) // 8),                                  # jumps from one direction to eight more
    "shelf": np.concatenate([1 - 0.01 * np.arange(4), 0.2 * (1 - 0.002 * np.arange(100))]),
}


@pytest.mark.parametrize("spectrum", list(UNSHIFTED_SPECTRA))
@pytest.mark.parametrize("M,N,seed", [(150, 129, 2), (129, 300, 3), (385, 400, 5), (400, 385, 6)])
def test_shifted_squarings_are_not_taken_again_where_a_spectrum_falls(tsvd, M, N, seed, spectrum):
    """Falling and stepped spectra: an iteration whose shifts do not hold costs two and more, a third of a call of a few components, so none may be lost where the
    pairs before tell that there is little to gain."""
    print(f"case fall {M} {N} {spectrum}", flush=True)
    U, S, V, errs, status = tsvd.tsvd_transition(_dev(_of_spectrum(M, N, UNSHIFTED_SPECTRA[spectrum], seed)), 0.65, 0.0, 12)
    kept, again = tsvd.tsvd_tuning_transition_shifts()
    assert status == 0 and U.shape[1] == 12
    assert again == 0, (kept, again)


@pytest.mark.parametrize("spectrum", ["close", "equal"])
def test_clustered_spectra_cost_little_more_than_others(tsvd, spectrum):
    """Singular values within 1e-6 of each other, and groups of 32 equal ones: the leading pair needs up to all of the squarings, an iteration that got
    too few is taken again, and the host has to arrive at their number in a few steps (arriving by threes took 4.7 and 8.6 times as long as a
    Laplace matrix, now 1.5 and 2.0)."""
    import time
    import torch
    M, N = 512, 256
    rng = np.random.default_rng(3)
    s = 1.0 + 1e-6 * np.arange(N)[::-1] / N if spectrum == "close" else 0.9 ** (np.arange(N) // 32)
    W = (np.linalg.qr(rng.standard_normal((M, N)))[0] * s) @ np.linalg.qr(rng.standard_normal((N, N)))[0].T
    def median(W):
        W = _dev(W)
        times = []
        for _ in range(6):
            t = time.perf_counter()
            _, _, _, errs, _ = tsvd.tsvd_transition(W, 0.65, 0.0, 24, q=4)
            torch.cuda.synchronize()
            times.append((time.perf_counter() - t) * 1e3)
        return sorted(times[1:])[2], errs
    print(f"case clustered {spectrum}", flush=True)
    plain, _ = median(rng.laplace(size=(M, N)))
    clustered, errs = median(W)
    print(f"{plain:.2f} ms, clustered {clustered:.2f}", flush=True)
    assert len(errs) == 24 and all(b <= a + 1e-9 for a, b in zip(errs, errs[1:]))
    assert clustered <= 3.0 * plain
