"""GPU parity of the offline quantizer (paper App. A.1 Algorithm 2; App. A.2.2; App. A.2.3; Sec. 3.2)
against its fp64 oracle, step by step through the C ABI, on seeded synthetic weight matrices (Gaussian
rows with a row offset and a planted low-rank part: the paper's own matrices are pretrained weights).
Both sides compute in fp64 and differ in summation order only, so the bar is 1e-9 relative on every
step that has a unique result.  The truncated SVD is iterative: with a planted gap behind sigma_k it
is held to 1e-8; without one the singular vectors are not determined to that accuracy by any method,
and the test compares what is unique -- the residual energy (Eckart-Young optimum), the rank, the
singular values -- and the descent of the loss."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import bwla_oracle as fwd
from oracle import bwla_quantizer_oracle as Q

pytestmark = pytest.mark.gpu


def _qb():
    from paper_2605_00422_amd import quantizer_binding as qb
    return qb


def _dev(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _rand_orth(rng, n):
    q, r = np.linalg.qr(rng.standard_normal((n, n)))
    return q * np.sign(np.diag(r))


def _problem(seed, n, n1, n2, k, planted=0.0):
    rng = np.random.default_rng(seed)
    m = n1 * n2
    W = rng.standard_normal((n, m)) * 0.02 + rng.standard_normal((n, 1)) * 0.004
    if planted:
        W += planted * (rng.standard_normal((n, k)) @ rng.standard_normal((k, m))) / np.sqrt(k)
    R1, R2 = _rand_orth(rng, n1), _rand_orth(rng, n2)
    U, s, Vt = np.linalg.svd(rng.standard_normal((n, m)) * 0.003, full_matrices=False)
    A, Bt = U[:, :k] * s[:k], Vt[:k].T.copy()
    return rng, W, A, Bt, R1, R2


def _ws(n, m, n1, n2, k):
    return torch.zeros(_qb().workspace_size(n, m, n1, n2, k), dtype=torch.uint8, device="cuda")


def _rel(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300))


SHAPES = [(24, 4, 6, 2), (150, 16, 32, 8), (200, 12, 10, 5), (333, 64, 64, 8), (70, 80, 64, 4), (6, 112, 128, 3),
          (10, 86, 64, 3)]


@pytest.mark.parametrize("n,n1,n2,k", SHAPES)
def test_okt_rows_em_and_loss(n, n1, n2, k):
    """X = (W - M) R H, the empirical start, one EM update and L_GMM (Sec. 3.2; App. A.2.2)."""
    qb = _qb()
    _, W, A, Bt, R1, R2 = _problem(1, n, n1, n2, k)
    m = n1 * n2
    ws = _ws(n, m, n1, n2, k)
    X = torch.empty(n, m, dtype=torch.float64, device="cuda")
    ybar = torch.empty(n, dtype=torch.float64, device="cuda")
    qb.okt_rows(_dev(W), _dev(A), _dev(Bt), _dev(R1), _dev(R2), X, ybar, ws)
    M = A @ Bt.T
    Xo = Q.okt_rows(W, M, R1, R2)
    assert _rel(X.cpu().numpy(), Xo) < 1e-11
    assert np.allclose(ybar.cpu().numpy(), fwd.kron_rotate(W - M, R1, R2).mean(axis=1), rtol=1e-9, atol=1e-15)
    # without a low-rank term
    qb.okt_rows(_dev(W), None, None, _dev(R1), _dev(R2), X, None, _ws(n, m, n1, n2, 0))
    assert _rel(X.cpu().numpy(), Q.okt_rows(W, np.zeros_like(W), R1, R2)) < 1e-11
    Xd = _dev(Xo)
    c = torch.empty(n, dtype=torch.float64, device="cuda")
    s2 = torch.empty(n, dtype=torch.float64, device="cuda")
    qb.init_theta(Xd, Q.S2_MIN, c, s2)
    co, s2o = Q.init_theta(Xo)
    assert np.allclose(c.cpu().numpy(), co, rtol=1e-12) and np.allclose(s2.cpu().numpy(), s2o, rtol=1e-11)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    qb.gmm_nll(Xd, c, s2, out, ws)
    assert abs(out.item() - Q.gmm_nll(Xo, co, s2o)) < 1e-11 * abs(Q.gmm_nll(Xo, co, s2o))
    for _ in range(3):
        qb.em_step(Xd, Q.S2_MIN, c, s2)
        co, s2o = Q.em_step(Xo, co, s2o)
        assert np.allclose(c.cpu().numpy(), co, rtol=1e-10) and np.allclose(s2.cpu().numpy(), s2o, rtol=1e-10)


def test_em_floor_and_degenerate_rows():
    """The variance floor (rows of two exact points +-c) and an all-zero row."""
    qb = _qb()
    n, m = 6, 64
    rng = np.random.default_rng(5)
    X = np.where(rng.random((n, m)) < 0.5, -1.0, 1.0) * 0.25
    X[:, : m // 2] = 0.25
    X[:, m // 2:] = -0.25
    X[3] = 0.0
    Xd = _dev(X)
    c = torch.empty(n, dtype=torch.float64, device="cuda")
    s2 = torch.empty(n, dtype=torch.float64, device="cuda")
    qb.init_theta(Xd, 1e-6, c, s2)
    co, s2o = Q.init_theta(X, 1e-6)
    assert np.array_equal(s2.cpu().numpy(), s2o) and np.all(s2o == 1e-6)
    qb.em_step(Xd, 1e-6, c, s2)
    co, s2o = Q.em_step(X, co, s2o, 1e-6)
    assert np.allclose(c.cpu().numpy(), co, rtol=1e-12, atol=1e-300)
    assert np.allclose(s2.cpu().numpy(), s2o, rtol=1e-12)


# (rows in registers, and a row that is read again by every step)
@pytest.mark.parametrize("m", [2048, 16386])
@pytest.mark.parametrize("c0", [1.0, 1e-3, 1e-8, 1e-200])
def test_em_step_keeps_the_digits_of_a_small_c(m, c0):
    """c = mean of x tanh(c x / s^2), terms of one sign, with c far below s: all of them small.  A term is right to some four roundings
    and a sum of m to log2 m more of them (threads' sums and trees), against 80 bits."""
    qb = _qb()
    n = 4
    X = np.random.default_rng(m).standard_normal((n, m))
    c, s2 = _dev(np.full(n, c0)), _dev(np.full(n, 1.1))
    qb.em_step(_dev(X), Q.S2_MIN, c, s2)
    x, c80, v80 = X.astype(np.longdouble), np.longdouble(c0), np.longdouble(1.1)
    t = np.tanh(c80 * x / v80)
    want = (t * x).mean(1)
    assert np.max(np.abs(c.cpu().numpy() - want) / want) < (8 + np.log2(m)) * 2.0 ** -52
    v = ((1 + t) / 2 * (x - want[:, None]) ** 2 + (1 - t) / 2 * (x + want[:, None]) ** 2).mean(1)
    assert np.max(np.abs(s2.cpu().numpy() - v) / v) < (8 + np.log2(m)) * 2.0 ** -52


@pytest.mark.parametrize("nn", [1, 2, 5, 16, 33, 64, 100, 160, 224, 256])
def test_svd_square_against_lapack(nn):
    """One-sided Jacobi: singular values, orthogonality and the reconstruction G = U S V^T."""
    qb = _qb()
    rng = np.random.default_rng(nn)
    G = rng.standard_normal((nn, nn)) * np.exp(rng.standard_normal((1, nn)))
    sig = torch.empty(nn, dtype=torch.float64, device="cuda")
    Ut = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
    Vt = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
    ws = torch.zeros(2 * nn * nn * 8 + 256, dtype=torch.uint8, device="cuda")
    qb.svd_square(_dev(G), sig, Ut, Vt, ws)
    s, us, v = sig.cpu().numpy(), Ut.cpu().numpy(), Vt.cpu().numpy()
    so = np.linalg.svd(G, compute_uv=False)
    assert np.all(np.diff(s) <= 0)
    assert np.allclose(s, so, rtol=1e-11, atol=1e-13 * so[0])
    assert np.max(np.abs(v @ v.T - np.eye(nn))) < 1e-12
    assert np.max(np.abs(us.T @ v - G)) < 1e-12 * so[0]                     # sum_j (s_j u_j) v_j^T
    u = us / np.maximum(s[:, None], 1e-300)
    assert np.max(np.abs(u @ u.T - np.eye(nn))) < 1e-9


@pytest.mark.parametrize("nn", [3, 7, 8, 9, 12, 17, 57, 63])
def test_svd_square_blocks_of_columns(nn):
    """Numbers of columns around the blocks of four (and pairs of blocks) that a wavefront holds up to 64;
    a zero and a repeated column among them."""
    qb = _qb()
    rng = np.random.default_rng(100 + nn)
    G = rng.standard_normal((nn, nn)) * np.exp(rng.standard_normal((1, nn)))
    G[:, 1] = G[:, 0]
    if nn > 3:
        G[:, nn - 1] = 0.0
    sig = torch.empty(nn, dtype=torch.float64, device="cuda")
    Ut = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
    Vt = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
    ws = torch.zeros(2 * nn * nn * 8 + 256, dtype=torch.uint8, device="cuda")
    qb.svd_square(_dev(G), sig, Ut, Vt, ws)
    s, us, v = sig.cpu().numpy(), Ut.cpu().numpy(), Vt.cpu().numpy()
    so = np.linalg.svd(G, compute_uv=False)
    assert np.all(np.diff(s) <= 0)
    assert np.allclose(s, so, rtol=1e-11, atol=1e-13 * so[0])
    # exact null directions are given as zero vectors: compare what is unique
    assert np.max(np.abs(us.T @ v - G)) < 1e-12 * so[0]
    live = s > 1e-12 * so[0]
    assert np.max(np.abs(v[live] @ v[live].T - np.eye(int(live.sum())))) < 1e-12


def _singular_values_80_bits(G):
    """One-sided Jacobi in the host's extended precision, every rotation from its three inner products."""
    W = G.astype(np.longdouble)
    n = W.shape[1]
    for _ in range(60):
        rotated = False
        for p in range(n - 1):
            for q in range(p + 1, n):
                x, y = W[:, p], W[:, q]
                al, be, ga = x @ x, y @ y, x @ y
                if al > 0 and be > 0 and abs(ga) > np.longdouble(1e-18) * np.sqrt(al) * np.sqrt(be):
                    z = (be - al) / (2 * ga)
                    t = (1 if z >= 0 else -1) / (abs(z) + np.sqrt(1 + z * z))
                    c = 1 / np.sqrt(1 + t * t)
                    W[:, p], W[:, q] = c * x - c * t * y, c * t * x + c * y
                    rotated = True
        if not rotated:
            break
    return np.sort(np.sqrt((W * W).sum(0)))[::-1]


@pytest.mark.parametrize("kind", ["normal", "graded", "half rank", "condition", "gram"])
@pytest.mark.parametrize("nn", [16, 33, 48, 72])
def test_svd_square_errors_stay_at_the_roundings(nn, kind):
    """Against extended precision.  A column takes part in nn - 1 rotations a sweep, some ten sweeps; each errs by three
    roundings of its norm, which add up as a random walk: 3 eps sqrt(10 nn), and the largest of nn^2 entries lies
    within four times that."""
    qb = _qb()
    rng = np.random.default_rng(200 + nn)
    q, p = _rand_orth(rng, nn), _rand_orth(rng, nn)
    G = {"normal": lambda: rng.standard_normal((nn, nn)),
         "graded": lambda: rng.standard_normal((nn, nn)) * 10.0 ** -np.linspace(0, 12, nn)[None, :],
         "half rank": lambda: rng.standard_normal((nn, nn // 2)) @ rng.standard_normal((nn // 2, nn)),
         "condition": lambda: (q * 10.0 ** -np.linspace(0, 14, nn)) @ p.T,
         "gram": lambda: (q * 10.0 ** -np.linspace(0, 14, nn)) @ q.T}[kind]()
    sig = torch.empty(nn, dtype=torch.float64, device="cuda")
    Ut = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
    Vt = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
    qb.svd_square(_dev(G), sig, Ut, Vt, torch.zeros(2 * nn * nn * 8 + 256, dtype=torch.uint8, device="cuda"))
    s, us, v = (t.cpu().numpy().astype(np.longdouble) for t in (sig, Ut, Vt))
    want = _singular_values_80_bits(G)
    bound = 4 * 3 * 2.0 ** -52 * np.sqrt(10.0 * nn)
    errs = (np.max(np.abs(s - want)) / want[0], np.max(np.abs(us.T @ v - G)) / want[0], np.max(np.abs(v @ v.T - np.eye(nn))))
    print(kind, nn, ["%.1e" % e for e in errs], "%.1e" % bound)
    assert max(errs) < bound


@pytest.mark.parametrize("exponent", [-60, 60])
def test_svd_square_of_scaled_columns(exponent):
    """Rotations between columns whose norms are 60 decades apart, and inner products far from one: the tangent's
    reciprocals and root at the ends of their range."""
    qb = _qb()
    nn = 12
    rng = np.random.default_rng(3)
    G = rng.standard_normal((nn, nn)) * 10.0 ** np.where(np.arange(nn) % 2, exponent, 0)[None, :]
    sig = torch.empty(nn, dtype=torch.float64, device="cuda")
    Ut = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
    Vt = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
    qb.svd_square(_dev(G), sig, Ut, Vt, torch.zeros(2 * nn * nn * 8 + 256, dtype=torch.uint8, device="cuda"))
    want = _singular_values_80_bits(G)
    s, us, v = (t.cpu().numpy() for t in (sig, Ut, Vt))
    # one-sided rotations keep each singular value to its own size while the scaled columns are well conditioned
    assert np.max(np.abs(s - want) / want) < 1e-12
    assert np.max(np.abs(v @ v.T - np.eye(nn))) < 1e-13 and np.max(np.abs(us.T @ v - G) / np.linalg.norm(G, axis=0)) < 1e-13


@pytest.mark.parametrize("n1,n2", [(128, 80), (128, 82)])
def test_rows_at_the_length_that_lds_keeps(n1, n2):
    """Rows of 10240 columns keep their first pass's values in LDS, longer ones take them again."""
    qb = _qb()
    n, m = 4, n1 * n2
    _, W, _, _, R1, R2 = _problem(7, n, n1, n2, 1)
    X = Q.okt_rows(W, np.zeros_like(W), R1, R2)
    c, s2 = Q.init_theta(X)
    cd, sd = _dev(c), _dev(s2)
    qb.em_step(_dev(X), Q.S2_MIN, cd, sd)
    c, s2 = Q.em_step(X, c, s2)
    assert np.allclose(cd.cpu().numpy(), c, rtol=1e-10) and np.allclose(sd.cpu().numpy(), s2, rtol=1e-10)
    ws = _ws(n, m, n1, n2, 0)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    qb.gmm_nll(_dev(X), cd, sd, out, ws)
    assert abs(out.item() - Q.gmm_nll(X, c, s2)) < 1e-11 * abs(Q.gmm_nll(X, c, s2))
    targets, lam = Q.mm_row_targets(W, R1, R2, c, s2)
    Rn = torch.empty(n1, n1, dtype=torch.float64, device="cuda")
    qb.procrustes(1, _dev(W), _dev(R1), _dev(R2), cd, sd, Rn, ws)
    want = Q.procrustes_r1(W, R2, targets, lam, n1, n2)
    assert np.max(np.abs(Rn.cpu().numpy() - want)) < 1e-8


# (rows in registers: 4 or 16 entries a thread of 256, 512 and 1024 threads, full and one column past; longer ones read again)
@pytest.mark.parametrize("m", [1, 63, 1024, 1025, 4096, 4097, 8192, 8193, 16384, 16385, 20000])
def test_row_steps_at_any_length(m):
    qb = _qb()
    n = 3
    X = Q.center_rows(np.random.default_rng(m).standard_normal((n, m)) + 0.5 * np.sign(np.random.default_rng(m + 1).standard_normal((n, m))))
    c, s2 = torch.empty(n, dtype=torch.float64, device="cuda"), torch.empty(n, dtype=torch.float64, device="cuda")
    qb.init_theta(_dev(X), Q.S2_MIN, c, s2)
    co, s2o = Q.init_theta(X)
    assert np.allclose(c.cpu().numpy(), co, rtol=1e-12, atol=1e-300) and np.allclose(s2.cpu().numpy(), s2o, rtol=1e-11)
    qb.em_step(_dev(X), Q.S2_MIN, c, s2)
    co, s2o = Q.em_step(X, co, s2o)
    assert np.allclose(c.cpu().numpy(), co, rtol=1e-10, atol=1e-300) and np.allclose(s2.cpu().numpy(), s2o, rtol=1e-10)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    qb.gmm_nll(_dev(X), c, s2, out, torch.zeros(256, dtype=torch.uint8, device="cuda"))
    want = Q.gmm_nll(X, co, s2o)
    assert abs(out.item() - want) < 1e-10 * max(abs(want), 1.0)


@pytest.mark.parametrize("n1,n2", [(256, 64), (256, 65)])
def test_targets_of_long_rows(n1, n2):
    """Targets of rows that registers still hold (16384 columns) and of longer ones, by way of the update of R2."""
    qb = _qb()
    n = 5
    _, W, _, _, R1, R2 = _problem(9, n, n1, n2, 1)
    c, s2 = Q.init_theta(Q.okt_rows(W, np.zeros_like(W), R1, R2))
    targets, lam = Q.mm_row_targets(W, R1, R2, c, s2)
    Rn = torch.empty(n2, n2, dtype=torch.float64, device="cuda")
    qb.procrustes(2, _dev(W), _dev(R1), _dev(R2), _dev(c), _dev(s2), Rn, _ws(n, n1 * n2, n1, n2, 0))
    assert np.max(np.abs(Rn.cpu().numpy() - Q.procrustes_r2(W, R1, targets, lam, n1, n2))) < 1e-9


@pytest.mark.parametrize("n,m,k", [(1, 1, 1), (2, 3, 1), (3, 2, 2), (5, 40, 5), (17, 9, 4)])
def test_truncate_rank_of_tiny_matrices(n, m, k):
    """Blocks as wide as the matrix: the truncation is exact after one product."""
    qb = _qb()
    Y = np.random.default_rng(n * 100 + m).standard_normal((n, m))
    A = torch.empty(n, k, dtype=torch.float64, device="cuda")
    Bt = torch.empty(m, k, dtype=torch.float64, device="cuda")
    ws = torch.zeros(qb.workspace_size(n, m, 1, 1, k), dtype=torch.uint8, device="cuda")
    qb.truncate_rank(_dev(Y), k, 60, 1e-14, A, Bt, None, ws)
    assert _rel(A.cpu().numpy() @ Bt.cpu().numpy().T, Q.truncate_rank(Y, k)) < 1e-9


def test_nll_keeps_the_terms_below_the_rounding_of_one():
    """Entries on a component whose other component is 40 nats down add log1p(exp(-40)) = 4.2e-18 each, less than
    the rounding of 1 + exp(-40).  With s^2 next to 1 / (8 pi) the leading terms, log 2 - log 2, vanish exactly at some
    of the neighbouring doubles (rounding of log decides at which), and what is left there is the sum of these."""
    qb = _qb()
    m = 5000
    tail = np.log1p(np.exp(-40.0))
    ws = torch.zeros(256, dtype=torch.uint8, device="cuda")
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    got = []
    v = 1.0 / (8.0 * np.pi)
    for _ in range(8):
        v = np.nextafter(v, 0.0)
    for _ in range(16):
        v = np.nextafter(v, 1.0)
        c = np.sqrt(20.0 * v)                               # 2 c^2 / s^2 = 40
        qb.gmm_nll(torch.full((1, m), c, dtype=torch.float64, device="cuda"), _dev(np.array([c])), _dev(np.array([v])), out, ws)
        got.append(out.item())
    # exp's argument is off by a few roundings of 40, the sums by m roundings at the very most
    assert any(abs(g + tail) < 1e-10 * tail for g in got), got
    assert all(abs(g) < 1e-14 for g in got)


@pytest.mark.parametrize("n,n1,n2,k", SHAPES)
def test_procrustes_updates(n, n1, n2, k):
    """Both Procrustes updates against the oracle's (App. A.2.2); the new factor is orthogonal and
    does not increase the surrogate it minimizes."""
    qb = _qb()
    _, W, A, Bt, R1, R2 = _problem(2, n, n1, n2, k)
    m = n1 * n2
    Wres = W - A @ Bt.T
    c, s2 = Q.init_theta(Q.okt_rows(W, A @ Bt.T, R1, R2))
    c, s2 = Q.em_step(Q.okt_rows(W, A @ Bt.T, R1, R2), c, s2)
    ws = _ws(n, m, n1, n2, 0)
    targets, lam = Q.mm_row_targets(Wres, R1, R2, c, s2)
    for which, nn in ((1, n1), (2, n2)):
        Rn = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
        qb.procrustes(which, _dev(Wres), _dev(R1), _dev(R2), _dev(c), _dev(s2), Rn, ws)
        got = Rn.cpu().numpy()
        want = (Q.procrustes_r1(Wres, R2, targets, lam, n1, n2) if which == 1
                else Q.procrustes_r2(Wres, R1, targets, lam, n1, n2))
        assert np.max(np.abs(got.T @ got - np.eye(nn))) < 1e-12
        assert np.max(np.abs(got - want)) < 1e-9
        before = Q.surrogate(Wres, R1, R2, targets, lam)
        after = Q.surrogate(Wres, got, R2, targets, lam) if which == 1 else Q.surrogate(Wres, R1, got, targets, lam)
        assert after <= before * (1 + 1e-12)


# (up to 96 the polar factor is the work of one workgroup, in tiles of 16: a tile and one, odd, full, one short of full;
# C2 has rank n n1 at most, so n is several times n2 / n1)
@pytest.mark.parametrize("n,n1,n2", [(40, 17, 96), (60, 80, 65), (160, 3, 95), (50, 64, 16)])
def test_procrustes_of_ragged_factors(n, n1, n2):
    qb = _qb()
    _, W, A, Bt, R1, R2 = _problem(6, n, n1, n2, 4)
    Wres = W - A @ Bt.T
    c, s2 = Q.init_theta(Q.okt_rows(W, A @ Bt.T, R1, R2))
    targets, lam = Q.mm_row_targets(Wres, R1, R2, c, s2)
    for which, nn in ((1, n1), (2, n2)):
        Rn = torch.empty(nn, nn, dtype=torch.float64, device="cuda")
        qb.procrustes(which, _dev(Wres), _dev(R1), _dev(R2), _dev(c), _dev(s2), Rn, _ws(n, n1 * n2, n1, n2, 0))
        got = Rn.cpu().numpy()
        want = (Q.procrustes_r1(Wres, R2, targets, lam, n1, n2) if which == 1
                else Q.procrustes_r2(Wres, R1, targets, lam, n1, n2))
        assert np.max(np.abs(got.T @ got - np.eye(nn))) < 1e-12
        assert np.max(np.abs(got - want)) < 1e-9


@pytest.mark.parametrize("n1", [16, 48, 64, 80, 96])
def test_procrustes_is_orthogonal_to_rounding(n1):
    """An entry of R^T R is a sum of n1 products, sqrt(n1) eps off by their roundings; the largest of n1^2, and as much again from the
    products that made R: within 16 times that.  Matrices of condition 1 to 1e5, whose iterations end at different distances."""
    qb = _qb()
    n, n2 = 300, 16
    for seed in range(3):
        rng = np.random.default_rng(seed * 7 + n1)
        W = rng.standard_normal((n, n1 * n2)) * np.exp(rng.standard_normal((1, n1 * n2)) * (0.2 + seed))
        R1, R2 = np.linalg.qr(rng.standard_normal((n1, n1)))[0], np.linalg.qr(rng.standard_normal((n2, n2)))[0]
        c, s2 = np.abs(rng.standard_normal(n)) * 0.3 + 0.5, np.abs(rng.standard_normal(n)) * 0.3 + 0.2
        R = torch.empty(n1, n1, dtype=torch.float64, device="cuda")
        qb.procrustes(1, _dev(W), _dev(R1), _dev(R2), _dev(c), _dev(s2), R, _ws(n, n1 * n2, n1, n2, 0))
        r = R.cpu().numpy().astype(np.longdouble)
        assert np.max(np.abs(r.T @ r - np.eye(n1))) < 16 * 2.0 ** -52 * np.sqrt(n1)


@pytest.mark.parametrize("n1", [32, 80])
def test_procrustes_of_a_singular_matrix(n1):
    """Rows of V_i that are zero in every row of the layer: C1 is singular, its polar factor not unique, the result finite."""
    qb = _qb()
    n, n2 = 40, 16
    _, W, _, _, R1, R2 = _problem(7, n, n1, n2, 4)
    Wres = W.reshape(n, n1, n2).copy()
    Wres[:, :2, :] = 0.0
    Wres = Wres.reshape(n, n1 * n2)
    R1, R2 = np.eye(n1), np.eye(n2)
    c, s2 = Q.init_theta(Q.okt_rows(Wres, np.zeros_like(Wres), R1, R2))
    Rn = torch.empty(n1, n1, dtype=torch.float64, device="cuda")
    qb.procrustes(1, _dev(Wres), _dev(R1), _dev(R2), _dev(c), _dev(s2), Rn, _ws(n, n1 * n2, n1, n2, 0))
    assert np.all(np.isfinite(Rn.cpu().numpy()))


# (rank 72: blocks of more than 136 vectors)
@pytest.mark.parametrize("n,n1,n2,k", [(90, 24, 20, 0), (90, 24, 20, 4), (200, 16, 16, 72)])
def test_start_at_the_identity_is_the_start_from_an_identity(n, n1, n2, k):
    """Factors that start at the identity are not multiplied by in the first round; the general path says the same."""
    qb = _qb()
    t, m = 2, n1 * n2
    _, W, _, _, _, _ = _problem(8, n, n1, n2, max(k, 1), planted=0.03)
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda")
    out = []
    for identity in (1, 0):
        R1, R2 = torch.eye(n1, device="cuda"), torch.eye(n2, device="cuda")
        Wrot, U, V = f32(n, m), f32(m, k) if k else None, f32(n, k) if k else None
        hist = torch.empty(1 + 3 * t, dtype=torch.float64, device="cuda")
        qb.quantize_layer(_dev(W, torch.float32), n1, n2, k, t, R1, R2, Wrot, U, V, None, None, hist, _ws(n, m, n1, n2, k),
                          svd_tol=1e-14, init_identity=identity)
        out.append((Wrot.cpu().numpy(), R1.cpu().numpy(), R2.cpu().numpy(), hist.cpu().numpy()))
    for a, b in zip(*out):
        assert np.max(np.abs(a - b)) < 1e-6 * max(1.0, np.max(np.abs(a)))      # fp32 results of fp64 work


# (the last five: blocks of 80, 128, 132, 160 and 256 vectors -- the Gram matrix's eigenproblem in a row pair of
# lanes per column pair and in a wavefront per pair with the matrix in LDS; above 136 vectors the block is
# orthonormalized by the Newton-Schulz iteration and the eigenproblem is solved once, in scratch)
@pytest.mark.parametrize("n,m,k", [(40, 30, 3), (300, 128, 8), (96, 512, 16), (513, 200, 5), (300, 256, 40),
                                   (400, 300, 64), (300, 280, 66), (400, 320, 80), (500, 300, 128)])
def test_truncate_rank_with_a_gap(n, m, k):
    """Planted rank-k part above a noise floor: the truncation itself is determined, and matches."""
    qb = _qb()
    rng = np.random.default_rng(n + m)
    Y = (rng.standard_normal((n, k)) * np.linspace(3.0, 1.0, k)) @ rng.standard_normal((k, m)) + 0.05 * rng.standard_normal((n, m))
    A = torch.empty(n, k, dtype=torch.float64, device="cuda")
    Bt = torch.empty(m, k, dtype=torch.float64, device="cuda")
    sig = torch.empty(k, dtype=torch.float64, device="cuda")
    ws = torch.zeros(qb.workspace_size(n, m, 1, 1, k), dtype=torch.uint8, device="cuda")
    qb.truncate_rank(_dev(Y), k, 60, 1e-14, A, Bt, sig, ws)
    got = A.cpu().numpy() @ Bt.cpu().numpy().T
    want = Q.truncate_rank(Y, k)
    so = np.linalg.svd(Y, compute_uv=False)
    assert np.allclose(sig.cpu().numpy(), so[:k], rtol=1e-10)
    assert _rel(got, want) < 1e-8
    b = Bt.cpu().numpy()
    assert np.max(np.abs(b.T @ b - np.eye(k))) < 1e-12


# (blocks of 24, 80, 128 and 132 vectors -- both ways of keeping the Cholesky factor, one to three elements of a column a
# lane; a spread of 3000, its square past 1e6, has the filter's first product deflated)
@pytest.mark.parametrize("n,m,k,spread", [(300, 200, 8, 300.0), (300, 256, 40, 300.0), (333, 300, 64, 100.0),
                                          (300, 280, 66, 300.0), (300, 200, 8, 3000.0), (70, 81, 40, 1.0)])
def test_truncate_rank_of_a_wide_spectrum(n, m, k, spread):
    """Singular values far apart: the filtered block's Gram matrix is graded over the fourth power of the spread.
    A singular value is as good as products with Y are, eps sigma_1 (some 100 roundings of them)."""
    qb = _qb()
    rng = np.random.default_rng(n + m)
    u, v = np.linalg.qr(rng.standard_normal((n, k)))[0], np.linalg.qr(rng.standard_normal((m, k)))[0]
    edge = 0.02 * (n ** 0.5 + m ** 0.5)
    Y = 0.02 * rng.standard_normal((n, m)) + (u * (1.5 * edge * np.geomspace(spread, 1, k))) @ v.T
    A = torch.empty(n, k, dtype=torch.float64, device="cuda")
    Bt = torch.empty(m, k, dtype=torch.float64, device="cuda")
    sig = torch.empty(k, dtype=torch.float64, device="cuda")
    ws = torch.zeros(qb.workspace_size(n, m, 1, 1, k), dtype=torch.uint8, device="cuda")
    qb.truncate_rank(_dev(Y), k, 60, 1e-14, A, Bt, sig, ws)
    so = np.linalg.svd(Y, compute_uv=False)
    assert np.allclose(sig.cpu().numpy(), so[:k], rtol=100 * 2.2e-16 * max(spread, 10.0))
    assert _rel(A.cpu().numpy() @ Bt.cpu().numpy().T, Q.truncate_rank(Y, k)) < 1e-8
    b = Bt.cpu().numpy()
    assert np.max(np.abs(b.T @ b - np.eye(k))) < 1e-12


def _spectrum(n, m, s, seed):
    """A matrix of the given singular values, and its truncation."""
    rng = np.random.default_rng(seed)
    p = min(n, m)
    u, v = np.linalg.qr(rng.standard_normal((n, p)))[0], np.linalg.qr(rng.standard_normal((m, p)))[0]
    s = np.sort(np.asarray(s))[::-1]
    return (u * s) @ v.T, lambda k: (u[:, :k] * s[:k]) @ v[:, :k].T


def _truncated(Y, k, iters, tol):
    qb = _qb()
    n, m = Y.shape
    A = torch.empty(n, k, dtype=torch.float64, device="cuda")
    Bt = torch.empty(m, k, dtype=torch.float64, device="cuda")
    ws = torch.zeros(qb.workspace_size(n, m, 1, 1, k), dtype=torch.uint8, device="cuda")
    qb.truncate_rank(_dev(Y), k, iters, tol, A, Bt, None, ws)
    b = Bt.cpu().numpy()
    assert np.max(np.abs(b.T @ b - np.eye(k))) < 1e-12
    return A.cpu().numpy() @ b.T


@pytest.mark.parametrize("factor", [3.0, 5.0, 10.0])
@pytest.mark.parametrize("n,m,k", [(400, 300, 8), (900, 640, 32)])
def test_truncate_rank_stops_no_farther_than_plain_iterations(n, m, k, factor):
    """Leading values in one group above the rest: subspace iteration without a filter, stopped by the same rule (the leading Ritz values
    moved by at most tol), is not nearer to the truncation where it stops -- but for the rounding of products with Y, 1e-13."""
    p = min(n, m)
    rng = np.random.default_rng(1)
    Y, best = _spectrum(n, m, np.concatenate([factor * (1 + 0.01 * rng.uniform(0, 1, k)), rng.uniform(0.05, 1.0, p - k)]), 5)
    want = best(k)
    for iters, tol in ((200, 1e-12), (60, 1e-14)):
        block, before = np.linalg.qr(rng.standard_normal((m, max(2 * k, k + 16))))[0], None
        for _ in range(iters):
            w, g = np.linalg.eigh((Y @ block).T @ (Y @ block))
            w, nxt = w[::-1], np.linalg.qr(Y.T @ (Y @ block))[0]
            if before is not None and np.max(np.abs(w[:k] ** 2 - before[:k] ** 2) / w[:k] ** 2) <= tol:
                break
            before, block = w, nxt
        z = Y @ block
        g = np.linalg.eigh(z.T @ z)[1][:, ::-1][:, :k]
        plain = _rel(z @ g @ (block @ g).T, want)
        assert _rel(_truncated(Y, k, iters, tol), want) <= max(plain, 1e-13)


# (blocks of 24, 64 and 132 vectors)
@pytest.mark.parametrize("n,m,k", [(400, 300, 8), (900, 640, 32), (300, 280, 66)])
@pytest.mark.parametrize("top", [[3e3], [1e4], [1e5, 3e3, 1e2], [1e6]])
def test_truncate_rank_with_one_value_far_above(n, m, k, top):
    """A few strong directions over values of which the smallest wanted one is 2 % above the others: what the truncation loses beyond the
    best is what its values have moved in the last iteration (tol); what is measured, besides, the result's rounding, eps sigma_1 times the
    residual."""
    p = min(n, m)
    rng = np.random.default_rng(1)
    lead = 1.02 + np.linspace(0.3, 0, k)
    lead[:len(top)] = top
    s = np.sort(np.concatenate([lead, rng.uniform(0.05, 1.0, p - k)]))[::-1]
    Y, _ = _spectrum(n, m, s, 5)
    got = _truncated(Y, k, 200, 1e-12)
    best = np.sum(s[k:] ** 2)
    assert abs(np.sum((Y - got) ** 2) / best - 1) < 1e-12 + 4 * 2.0 ** -52 * s[0] / np.sqrt(best)


# (contractions past 2048 with ragged ends, results of 24 to 80 columns in tiles of 64: the kernels that take operands
# straight from memory, with and without a split of the contraction)
@pytest.mark.parametrize("n,m,k", [(2055, 64, 8), (3001, 98, 40), (2500, 2306, 30)])
def test_truncate_rank_of_long_contractions(n, m, k):
    qb = _qb()
    rng = np.random.default_rng(n)
    Y = (rng.standard_normal((n, k)) * np.linspace(3.0, 1.0, k)) @ rng.standard_normal((k, m)) + 0.05 * rng.standard_normal((n, m))
    A = torch.empty(n, k, dtype=torch.float64, device="cuda")
    Bt = torch.empty(m, k, dtype=torch.float64, device="cuda")
    ws = torch.zeros(qb.workspace_size(n, m, 1, 1, k), dtype=torch.uint8, device="cuda")
    qb.truncate_rank(_dev(Y), k, 40, 1e-14, A, Bt, None, ws)
    assert _rel(A.cpu().numpy() @ Bt.cpu().numpy().T, Q.truncate_rank(Y, k)) < 1e-8


@pytest.mark.parametrize("rank", [0, 1, 4])
def test_truncate_rank_of_a_matrix_of_lower_rank(rank):
    """Fewer directions than are asked for: the matrix itself comes back, finite factors and zero singular values."""
    qb = _qb()
    n, m, k = 130, 90, 8
    rng = np.random.default_rng(5)
    Y = rng.standard_normal((n, rank)) @ rng.standard_normal((rank, m))
    A = torch.empty(n, k, dtype=torch.float64, device="cuda")
    Bt = torch.empty(m, k, dtype=torch.float64, device="cuda")
    sig = torch.empty(k, dtype=torch.float64, device="cuda")
    ws = torch.zeros(qb.workspace_size(n, m, 1, 1, k), dtype=torch.uint8, device="cuda")
    qb.truncate_rank(_dev(Y), k, 60, 1e-12, A, Bt, sig, ws)
    got = A.cpu().numpy() @ Bt.cpu().numpy().T
    scale = max(float(np.linalg.norm(Y)), 1.0)
    assert np.linalg.norm(got - Y) < 1e-7 * scale         # (what sweeps on the Gram matrix itself reached: 4e-8)
    assert np.all(np.isfinite(got)) and np.all(sig.cpu().numpy()[rank:] < 1e-7 * scale)


def test_truncate_rank_without_a_gap():
    """A Gaussian matrix: what is unique is the residual energy sum_{j>k} sigma_j^2 (Eckart-Young)."""
    qb = _qb()
    n, m, k = 400, 256, 8
    rng = np.random.default_rng(9)
    Y = rng.standard_normal((n, m))
    A = torch.empty(n, k, dtype=torch.float64, device="cuda")
    Bt = torch.empty(m, k, dtype=torch.float64, device="cuda")
    sig = torch.empty(k, dtype=torch.float64, device="cuda")
    ws = torch.zeros(qb.workspace_size(n, m, 1, 1, k), dtype=torch.uint8, device="cuda")
    qb.truncate_rank(_dev(Y), k, 400, 1e-13, A, Bt, sig, ws)
    got = A.cpu().numpy() @ Bt.cpu().numpy().T
    so = np.linalg.svd(Y, compute_uv=False)
    best = float(np.sum(so[k:] ** 2))
    assert np.linalg.matrix_rank(got, tol=1e-9) == k
    res = float(np.sum((Y - got) ** 2))
    assert best * (1 - 1e-12) <= res <= best * (1 + 1e-6)
    assert np.allclose(sig.cpu().numpy(), so[:k], rtol=1e-5)


@pytest.mark.parametrize("n,n1,n2,k", [(150, 16, 32, 8), (333, 64, 64, 8), (200, 16, 16, 72)])
def test_psp_step(n, n1, n2, k):
    """The proximal step with the default mu: the proximal point has a planted low-rank part, so the
    new M matches the oracle's; and L(W - M) does not increase (App. A.2.3)."""
    qb = _qb()
    _, W, A, Bt, R1, R2 = _problem(3, n, n1, n2, k, planted=0.05)
    m = n1 * n2
    M = A @ Bt.T
    X = Q.okt_rows(W, M, R1, R2)
    c, s2 = Q.em_step(X, *Q.init_theta(X))
    Ad, Btd = _dev(A), _dev(Bt)
    qb.psp_step(_dev(W), Ad, Btd, _dev(R1), _dev(R2), _dev(c), _dev(s2), 0.0, 300, 1e-14, _ws(n, m, n1, n2, k))
    got = Ad.cpu().numpy() @ Btd.cpu().numpy().T
    want = Q.psp_step(W, M, R1, R2, c, s2, k)
    before = Q.gmm_nll(X, c, s2)
    after = Q.gmm_nll(Q.okt_rows(W, got, R1, R2), c, s2)
    assert after <= before + 1e-13
    assert abs(after - Q.gmm_nll(Q.okt_rows(W, want, R1, R2), c, s2)) < 1e-9
    # the proximal point and its optimum: residual energy equal to the oracle's
    Yp = M - Q.grad_m(W, M, R1, R2, c, s2) / Q.default_mu(s2, n, m)
    assert np.sum((Yp - got) ** 2) <= np.sum((Yp - want) ** 2) * (1 + 1e-9)
    # an explicit mu goes through the same path
    Ad, Btd = _dev(A), _dev(Bt)
    mu = 3.0 * Q.default_mu(s2, n, m)
    qb.psp_step(_dev(W), Ad, Btd, _dev(R1), _dev(R2), _dev(c), _dev(s2), mu, 300, 1e-14, _ws(n, m, n1, n2, k))
    got = Ad.cpu().numpy() @ Btd.cpu().numpy().T
    want = Q.psp_step(W, M, R1, R2, c, s2, k, mu)
    Yp = M - Q.grad_m(W, M, R1, R2, c, s2) / mu
    assert np.sum((Yp - got) ** 2) <= np.sum((Yp - want) ** 2) * (1 + 1e-9)


@pytest.mark.parametrize("n,n1,n2,k,t", [(150, 16, 32, 4, 3), (256, 32, 32, 0, 3), (333, 64, 64, 8, 2), (200, 16, 16, 72, 2)])
def test_quantize_layer_history_and_outputs(n, n1, n2, k, t):
    """Algorithm 2 end to end: the loss after every sub-step follows the oracle's history and never
    increases; the factors are orthogonal; W_rot = (W - V U^T)(R1 (x) R2); and the result packs and
    runs through the forward path's own pack call."""
    qb = _qb()
    _, W, _, _, _, _ = _problem(4, n, n1, n2, max(k, 1), planted=0.03)
    W = W.astype(np.float32).astype(np.float64)
    m = n1 * n2
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda")
    R1, R2, Wrot = f32(n1, n1), f32(n2, n2), f32(n, m)
    U, V = (f32(m, k), f32(n, k)) if k else (None, None)
    c = torch.empty(n, dtype=torch.float64, device="cuda")
    s2 = torch.empty(n, dtype=torch.float64, device="cuda")
    hist = torch.empty(1 + 3 * t, dtype=torch.float64, device="cuda")
    qb.quantize_layer(_dev(W, torch.float32), n1, n2, k, t, R1, R2, Wrot, U, V, c, s2, hist, _ws(n, m, n1, n2, k),
                      svd_iters=300, svd_tol=1e-14)
    h = hist.cpu().numpy()
    ref = Q.quantize_layer(W, n1, n2, k, t_outer=t)
    want = [v for (_, name, v) in ref["history"]]
    if k == 0:                                            # the oracle records no PSP entry then
        it = iter(want[1:])
        full = [want[0]]
        for _ in range(t):
            em = next(it)
            full += [em, em, next(it)]
        want = full
    assert np.all(np.diff(h) <= 1e-12), h
    assert np.allclose(h, want, rtol=1e-7, atol=1e-9), (h, want)
    r1, r2 = R1.double().cpu().numpy(), R2.double().cpu().numpy()
    assert np.max(np.abs(r1.T @ r1 - np.eye(n1))) < 1e-5 and np.max(np.abs(r2.T @ r2 - np.eye(n2))) < 1e-5
    Mg = V.double().cpu().numpy() @ U.double().cpu().numpy().T if k else np.zeros_like(W)
    wr = Wrot.double().cpu().numpy()
    assert _rel(wr, fwd.kron_rotate(W - Mg, r1, r2)) < 1e-5
    assert abs(Q.gmm_nll(Q.center_rows(wr), c.cpu().numpy(), s2.cpu().numpy()) - h[-1]) < 1e-6
    if k:
        # balanced factors: column norms of V and U agree (both sigma_j^(1/2))
        nv = np.linalg.norm(V.double().cpu().numpy(), axis=0)
        nu = np.linalg.norm(U.double().cpu().numpy(), axis=0)
        assert np.allclose(nv, nu, rtol=1e-5)
    if m % 32 == 0:
        from paper_2605_00422_amd import binding as B
        layer = B.pack_weights(Wrot, R1, R2, U, V, n1, n2, centered=True)
        sgn, alpha = B.unpack_signs(layer)
        so, ao, _ = fwd.binarize_rows_centered(wr)
        assert np.mean(sgn.cpu().numpy() != so) < 1e-3


def test_quantize_layer_at_the_7b_shape():
    """11008 x 4096 (64 x 64), rank 32 -- the shape the benchmark times.  At this size the oracle checks
    what it can compute in seconds: the loss never increases over the sub-steps, the last entry is
    L_GMM of the returned W_rot under the returned mixtures, the factors are orthogonal, and sampled
    rows of W_rot equal (W - V U^T)_i (R1 (x) R2)."""
    qb = _qb()
    n, n1, n2, k, t = 11008, 64, 64, 32, 2
    m = n1 * n2
    rng = np.random.default_rng(7)
    W = (rng.standard_normal((n, m)) * 0.02 + rng.standard_normal((n, 1)) * 0.004).astype(np.float32)
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda")
    R1, R2, Wrot, U, V = f32(n1, n1), f32(n2, n2), f32(n, m), f32(m, k), f32(n, k)
    c = torch.empty(n, dtype=torch.float64, device="cuda")
    s2 = torch.empty(n, dtype=torch.float64, device="cuda")
    hist = torch.empty(1 + 3 * t, dtype=torch.float64, device="cuda")
    qb.quantize_layer(_dev(W, torch.float32), n1, n2, k, t, R1, R2, Wrot, U, V, c, s2, hist, _ws(n, m, n1, n2, k),
                      svd_iters=20, svd_tol=0.0)
    h = hist.cpu().numpy()
    assert np.all(np.isfinite(h)) and np.all(np.diff(h) <= 1e-12), h
    assert h[-1] < h[0] - 1e-3
    r1, r2 = R1.double().cpu().numpy(), R2.double().cpu().numpy()
    assert np.max(np.abs(r1.T @ r1 - np.eye(n1))) < 1e-5 and np.max(np.abs(r2.T @ r2 - np.eye(n2))) < 1e-5
    wr = Wrot.double().cpu().numpy()
    assert abs(Q.gmm_nll(Q.center_rows(wr), c.cpu().numpy(), s2.cpu().numpy()) - h[-1]) < 1e-6
    rows = np.concatenate([[0, n - 1], rng.choice(n, 62, replace=False)])
    Vh, Uh = V.double().cpu().numpy(), U.double().cpu().numpy()
    want = fwd.kron_rotate(W[rows].astype(np.float64) - Vh[rows] @ Uh.T, r1, r2)
    assert _rel(wr[rows], want) < 1e-5
    assert np.linalg.matrix_rank(Vh, tol=1e-9) == k


def test_quantized_layer_through_the_online_path():
    """Algorithm 2's result handed to the online path (Sec. 3.2: Y = Q(X R) B'^T + (X U) V^T): the factors,
    W_rot and the balanced U, V are packed by the forward path's own call and one decode call runs a few
    tokens through them.  The output equals the oracle's forward on the same factors (criterion of
    the parity tests), and against the dense product X W^T it is closer than the layer binarized as it
    stands (identity rotations, no low-rank branch): the planted low-rank part, which dominates the
    binarization error of the raw matrix, now travels through the PSP branch in fp16."""
    from paper_2605_00422_amd import binding as B
    from parity_util import check_output
    qb = _qb()
    n, n1, n2, k, t, M = 512, 32, 32, 8, 3, 8
    m = n1 * n2
    rng, W, _, _, _, _ = _problem(11, n, n1, n2, k, planted=0.05)
    W = W.astype(np.float32).astype(np.float64)
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda")
    R1, R2, Wrot, U, V = f32(n1, n1), f32(n2, n2), f32(n, m), f32(m, k), f32(n, k)
    qb.quantize_layer(_dev(W, torch.float32), n1, n2, k, t, R1, R2, Wrot, U, V, None, None, None, _ws(n, m, n1, n2, k),
                      svd_iters=100, svd_tol=1e-12)
    X = fwd.to_bf16(rng.standard_normal((M, m)))
    Xg = _dev(X, torch.bfloat16)
    dense = X @ W.T

    def run(layer):
        act = B.Activations(layer, M)
        Y = torch.empty((M, n), dtype=torch.float32, device="cuda")
        B.decode_forward(layer, Xg, act, Y)
        torch.cuda.synchronize()
        return Y.double().cpu().numpy()

    Yq = run(B.pack_weights(Wrot, R1, R2, U, V, n1, n2, centered=True))
    ref = fwd.forward(X, R1.double().cpu().numpy(), R2.double().cpu().numpy(), Wrot.double().cpu().numpy(),
                      U.double().cpu().numpy(), V.double().cpu().numpy(), centered=True)
    check_output(Yq, ref["Y"])
    eye = lambda s: torch.eye(s, dtype=torch.float32, device="cuda")
    Y0 = run(B.pack_weights(_dev(W, torch.float32), eye(n1), eye(n2), None, None, n1, n2, centered=True))
    err = lambda Y: float(np.linalg.norm(Y - dense) / np.linalg.norm(dense))
    print(dict(quantized=err(Yq), as_it_stands=err(Y0)), flush=True)
    assert err(Yq) < 0.85 * err(Y0)
