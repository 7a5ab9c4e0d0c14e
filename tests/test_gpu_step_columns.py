"""kmp_path_step by a Cholesky factor per column (step.hip) against the
oracle's dense step: orders on the edges of its 64-row tiles, one and several
columns, odd leading dimensions, in place, and matrices whose 2 lambda I +
K/(n kappa) is not positive definite, which go by the factorisation of K."""
import numpy as np
import pytest

from oracle import gram as OG
from oracle import losses as OL
from tests.gpu_common import announce, device

pytestmark = pytest.mark.gpu

STEP_RTOL = 1e-9     # that of the single-step test: relative to the larger max |alpha|


def _mm_step(K, y, alpha, beta, lam, loss, delta, tau, kap):
    """oracle.mm.mm_step with a pivoted solve, for M of either sign."""
    n = y.shape[0]
    z = OL.point_psi(loss, y, K @ alpha + beta, delta, tau) / n
    w, d0 = z + 2.0 * lam * alpha, z.sum()
    M = 2.0 * lam * np.eye(n) + K / (n * kap)
    x, v = np.linalg.solve(M, np.stack([w, np.full(n, 1.0 / (n * kap))], axis=1)).T
    g, t = 1.0 / (2.0 * lam * v.sum()), v @ (K @ w)
    return alpha - x - g * (t - d0) * v, beta - g * (d0 - t)


def _step(loss, n, C, K, in_place=False, lam_lo=-4.0):
    import torch
    from paper_2606_06742_amd import kmpath as km
    dev = device()
    rng = np.random.default_rng(n + C)
    y = np.where(rng.standard_normal(n) > 0, 1.0, -1.0) if loss != "check" else rng.standard_normal(n)
    lambdas = 10.0 ** np.linspace(lam_lo, 0.0, C)
    delta = None if loss == "logistic" else 0.125
    taus = np.linspace(0.1, 0.9, C) if loss == "check" else None
    A = rng.uniform(-1, 1, (C, n)) / (2 * n * lambdas[:, None])
    B = rng.uniform(-0.5, 0.5, C)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
    a_in, b_in = t(A), t(B)
    a_out, b_out = (a_in, b_in) if in_place else (torch.empty_like(a_in), torch.empty_like(b_in))
    kkt = torch.empty_like(b_in)
    announce(f"kmp_path_step loss={loss} n={n} C={C} in_place={in_place}")
    km.kmp_path_step(loss, delta, t(K), t(y), lambdas, a_in, b_in, a_out, b_out, kkt, taus=taus)
    torch.cuda.synchronize()
    ag, bg, kg = a_out.cpu().numpy(), b_out.cpu().numpy(), kkt.cpu().numpy()
    kap = OL.kappa(loss, delta)
    for c in range(C):
        tau = taus[c] if taus is not None else None
        ao, bo = _mm_step(K, y, A[c], B[c], lambdas[c], loss, delta, tau, kap)
        scale = max(np.abs(ao).max(), np.abs(A[c]).max())
        assert np.abs(ag[c] - ao).max() <= STEP_RTOL * scale, c
        assert abs(bg[c] - bo) <= STEP_RTOL * max(1.0, abs(bo), np.abs(A[c]).max()), c
        z = OL.point_psi(loss, y, K @ A[c] + B[c], delta, tau) / n
        ko = n * max(np.linalg.norm(z + 2 * lambdas[c] * A[c]), abs(z.sum()))
        assert abs(kg[c] - ko) <= 1e-9 * ko, c


@pytest.mark.parametrize("loss,n,C", [
    ("hinge", 2, 1), ("check", 63, 3), ("logistic", 64, 5), ("hinge", 65, 1), ("check", 128, 17),
    ("logistic", 191, 2), ("hinge", 449, 33),
])
def test_step_edges(loss, n, C):
    X = np.random.default_rng(n).standard_normal((n, 3))
    _step(loss, n, C, OG.rbf_gram(X, X, 1.5), in_place=n % 2 == 1)


def test_step_without_positive_pivots():
    """Eigenvalues of K far below zero: the dense step still exists, and the call
    gives it as before."""
    n = 100
    U, _ = np.linalg.qr(np.random.default_rng(1).standard_normal((n, n)))
    e = np.linspace(-40.0, 60.0, n)
    _step("hinge", n, 2, (U * e) @ U.T, lam_lo=-1.0)


def test_step_from_a_state_that_is_not_finite():
    """A column whose state is not finite keeps it, and the others step."""
    import torch
    from paper_2606_06742_amd import kmpath as km
    dev = device()
    n = 70
    rng = np.random.default_rng(5)
    X = rng.standard_normal((n, 3))
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
    a_in, y = t(rng.uniform(-1, 1, (3, n)) / n), t(np.where(X[:, 0] > 0, 1.0, -1.0))
    announce("kmp_path_step: an intercept that is not a number")
    out = []
    for beta in (0.1, np.nan):
        b_in = t([0.2, beta, 0.3])
        a, b, k = torch.empty_like(a_in), torch.empty_like(b_in), torch.empty_like(b_in)
        km.kmp_path_step("logistic", None, t(OG.rbf_gram(X, X, 1.5)), y, np.array([0.1, 0.01, 1.0]),
                         a_in, b_in, a, b, k)
        out.append((a.cpu().numpy(), b.cpu().numpy()))
    (a0, b0), (a1, b1) = out
    assert np.array_equal(a0[[0, 2]], a1[[0, 2]]) and np.array_equal(b0[[0, 2]], b1[[0, 2]])
    assert np.array_equal(a1[1], a_in[1].cpu().numpy()) and np.isnan(b1[1])


def test_step_from_two_threads():
    """Steps of different orders, so of different LDS sizes, at the same time: each
    thread's results are those of its calls alone."""
    import threading

    import torch
    from paper_2606_06742_amd import kmpath as km
    dev = device()
    announce("kmp_path_step: two threads, orders 64 and 1024")

    def make(n, C):
        rng = np.random.default_rng(n)
        X = rng.standard_normal((n, 3))
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
        return dict(K=t(OG.rbf_gram(X, X, 1.5)), y=t(np.where(X[:, 0] > 0, 1.0, -1.0)),
                    lam=np.linspace(0.01, 1.0, C), a=t(rng.uniform(-1, 1, (C, n)) / n),
                    b=t(rng.uniform(-1, 1, C)))

    def step(p):
        a, b = torch.empty_like(p["a"]), torch.empty_like(p["b"])
        km.kmp_path_step("hinge", 0.125, p["K"], p["y"], p["lam"], p["a"], p["b"], a, b)
        return a.cpu().numpy(), b.cpu().numpy()

    problems = [make(64, 4), make(1024, 2)]
    alone = [step(p) for p in problems]
    got = [[], []]
    def work(i):
        try:
            for _ in range(12):
                got[i].append(step(problems[i]))
        except Exception as e:                   # seen below
            got[i].append(e)
    threads = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    for i in (0, 1):
        assert len(got[i]) == 12
        for r in got[i]:
            assert not isinstance(r, Exception), r
            assert np.array_equal(r[0], alone[i][0]) and np.array_equal(r[1], alone[i][1])
