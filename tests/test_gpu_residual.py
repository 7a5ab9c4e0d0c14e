"""What the forms that carry f = K alpha by a recurrence (small.hip, dense.hip) report at
small penalties, where the recurrence's rounding is largest: the residual
n_v max(||z + 2 lambda alpha||_2, |1'z|) formed outside the library, in extended
precision on the library's own kernel matrix, against the bar that a converged
column claims and against the batched iteration (KMP_FLAG_GLOBAL_SOLVE) on the
same problem."""
import numpy as np
import pytest

from oracle import losses as OL
from tests.gpu_common import announce, device

pytestmark = pytest.mark.gpu

TOL = 1e-9
EPS = np.finfo(float).eps


def _problem(loss, n, d, data):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, d))
    if loss == "check":
        return X, X[:, 0] + (1.0 if data == "random" else 0.05) * rng.standard_normal(n)
    if data == "random":
        return X, np.where(rng.random(n) < 0.5, 1.0, -1.0)
    return X, np.where(X[:, 0] + 0.3 * rng.standard_normal(n) > 0, 1.0, -1.0)


def _fits(loss, n, d, sigma, data, delta, lam, max_iter, restart=True):
    """Full-data fits at the penalties lam by the library's own choice of form
    and in batched form: results, residuals and what rounding adds to these."""
    import torch
    from paper_2606_06742_amd import kmpath as km
    dev = device()
    X, y = _problem(loss, n, d, data)
    rows = torch.arange(n, dtype=torch.int32, device=dev)
    K = torch.empty((1, n, n), dtype=torch.float64, device=dev)
    km.kmp_rbf_gram(torch.as_tensor(X, device=dev), rows, rows, np.array([sigma]), K)
    K = K[0].cpu().numpy().astype(np.longdouble)
    tau = 0.5 if loss == "check" else None
    slope = 0.25 if loss == "logistic" else 1.0 / (2.0 * delta)
    out = []
    for flag in (0, km.KMP_FLAG_GLOBAL_SOLVE):
        r = km.PathRunner(X, y, loss, np.array([sigma]), np.array(lam), np.zeros(n, np.int32), 1,
                          refit=True, taus=np.array([0.5]) if loss == "check" else None,
                          max_iter=max_iter, delta0=delta, n_stages=1)
        r.spec.flags |= flag
        if not restart:
            r.spec.flags &= ~km.KMP_FLAG_RESTART
        code = r.run()
        g = r.results()
        kkt, noise = [], []
        for l, lm in enumerate(lam):
            a, b = g["alpha"][0, 0, 0, l].astype(np.longdouble), g["beta"][0, 0, 0, l]
            z = OL.point_psi(loss, y, (K @ a + b).astype(float), delta, tau)
            kkt.append(max(np.linalg.norm(z + 2 * n * lm * a.astype(float)), abs(z.sum())))
            # an f_i that is off by 2 eps ||alpha||_1
            noise.append(2 * EPS * float(np.abs(a).sum()) * np.sqrt(n) * slope)
        out.append((code, g, np.array(kkt), np.array(noise)))
    return out


@pytest.mark.parametrize("loss,n,d,sigma,data,delta,lam", [
    ("hinge", 60, 2, 5.0, "shift", 1.0, 1e-8),
    ("hinge", 180, 2, 5.0, "shift", 0.125, 1e-8),
    ("hinge", 180, 5, 3.0, "shift", 0.125, 1e-6),
    ("hinge", 250, 5, 20.0, "shift", 1.0, 1e-8),
    ("check", 180, 5, 3.0, "shift", 0.125, 1e-6),
    ("logistic", 180, 2, 5.0, "shift", 1.0, 1e-9),
    ("hinge", 420, 2, 5.0, "shift", 1.0, 1e-9),
    ("hinge", 420, 5, 3.0, "shift", 0.125, 1e-6),
    ("check", 420, 5, 20.0, "shift", 0.125, 1e-8),
    ("logistic", 420, 2, 5.0, "shift", 1.0, 1e-9),
])
def test_a_converged_column_is_converged(loss, n, d, sigma, data, delta, lam):
    """A column reported as converged has the residual that this claims, up to the
    rounding of one product K alpha; one reported otherwise is so in batched form."""
    announce(f"residual of converged columns loss={loss} n={n} sigma={sigma} lambda={lam}")
    (_, g, kkt, noise), (_, gb, kb, _) = _fits(loss, n, d, sigma, data, delta, [lam], 20000)
    print(g["status"].ravel(), g["iters"].ravel(), kkt, noise, gb["status"].ravel(), kb)
    if g["status"].ravel()[0] == 0:
        # f formed through the factor (where one was made) has the factor's backward
        # error, which the batched form's result shows
        bar = TOL + noise[0] + (2 * kb[0] if g["timings"]["factor_ms"] > 0 else 0.0)
        assert kkt[0] <= bar, (kkt, noise, kb)
    else:
        assert gb["status"].ravel()[0] != 0 and kkt[0] <= 10 * kb[0]


@pytest.mark.parametrize("loss,n,d,sigma,data,delta,lam,max_iter", [
    ("hinge", 180, 5, 20.0, "random", 0.125, 1e-12, 3000),
    ("hinge", 250, 2, 5.0, "random", 0.125, 1e-13, 3000),
    ("check", 60, 5, 20.0, "shift", 1.0, 1e-12, 3000),
    ("logistic", 120, 5, 20.0, "random", 1.0, 1e-13, 3000),
    ("hinge", 420, 2, 5.0, "shift", 0.125, 1e-12, 3000),
    ("check", 420, 5, 20.0, "random", 0.125, 1e-13, 3000),
])
def test_max_iter_with_another_f(loss, n, d, sigma, data, delta, lam, max_iter):
    """A column whose carried f is not K alpha any more is not stopped by max_iter
    on its account: the result is that of the batched iteration."""
    announce(f"residual at max_iter loss={loss} n={n} sigma={sigma} lambda={lam}")
    (c, g, kkt, _), (cb, gb, kb, _) = _fits(loss, n, d, sigma, data, delta, [lam, 0.1], max_iter)
    print(g["status"].ravel(), g["iters"].ravel(), kkt, gb["status"].ravel(), kb)
    assert c == cb and np.array_equal(g["status"], gb["status"])
    assert np.all(kkt <= np.maximum(10 * kb, 10 * TOL)), (kkt, kb)
    assert g["timings"]["factor_ms"] > 0            # the batched form was taken


def test_more_iterations_than_one_launch():
    """A column of more than 8192 iterations goes on in further launches."""
    announce("small order, several launches of a column")
    (c, g, kkt, noise), (cb, gb, kb, _) = _fits("logistic", 100, 5, 0.5, "random", 1.0, [1e-7, 1e-2],
                                               60000, restart=False)
    print(g["status"].ravel(), g["iters"].ravel(), kkt, noise, gb["iters"].ravel(), kb)
    assert c == cb == 0 and g["iters"].max() > 8192 and g["timings"]["factor_ms"] == 0
    assert np.all(kkt <= TOL + noise), (kkt, noise)


@pytest.mark.parametrize("n", [180, 420])
def test_stopped_by_max_iter_means_that_many_iterations(n):
    """Columns that stop as converged by their carried f and go on near max_iter:
    no column is reported as stopped by max_iter after fewer iterations."""
    announce(f"iterations of columns stopped by max_iter n={n}")
    lam = [1e-6, 1e-5, 1e-4]
    _, g, _, _ = _fits("hinge", n, 5, 3.0, "shift", 0.125, lam, 20000)[0]
    assert np.all(g["status"] == 0)
    most = int(g["iters"].max())
    for limit in (most - 1, most - 20, most // 2, most):
        for code, g, kkt, _ in _fits("hinge", n, 5, 3.0, "shift", 0.125, lam, limit):
            st, it = g["status"].ravel(), g["iters"].ravel()
            print(limit, st, it, kkt)
            assert np.all(it[st == 1] == limit) and np.all(it <= limit) and np.all(st <= 1)


@pytest.mark.parametrize("sigma,data,max_iter", [(4.0, "random", 1500), (2.0, "random", 1500)])
def test_small_order_left_to_the_batched_form(sigma, data, max_iter):
    """Columns of small orders whose carried f does not settle on K alpha, or that
    stop at max_iter by another f: the fit is made in batched form."""
    announce(f"small order left to the batched form sigma={sigma}")
    (c, g, kkt, noise), (cb, gb, kb, _) = _fits("hinge", 200, 5, sigma, data, 0.125, [9e-7], max_iter)
    print(c, g["iters"].ravel(), kkt, noise, cb, gb["iters"].ravel(), kb)
    assert g["timings"]["factor_ms"] > 0
    assert c == cb and np.array_equal(g["status"], gb["status"])
    assert kkt[0] <= TOL + noise[0] + 10 * kb[0], (kkt, kb)


def test_dense_columns_done_again_in_batched_form():
    """Dense columns that stop at max_iter by another f than K alpha's: the batch is
    done again, with the bits of a workspace without room for dense columns."""
    from paper_2606_06742_amd import kmpath as km
    device()
    n, limit = 300, 2500
    X, y = _problem("hinge", n, 5, "shift")
    announce("dense columns done again in batched form")
    out = []
    for optional in (True, False):
        r = km.PathRunner(X, y, "hinge", np.array([20.0]), np.array([2e-8]), np.zeros(n, np.int32), 1,
                          refit=True, max_iter=limit, delta0=1.0 / 64, n_stages=1, tol=2e-6, eager=True,
                          kernel_timing=("update", "gemm_f"))
        if not optional:
            spec = km.kmp_default_spec("hinge", flags=r.spec.flags | km.KMP_FLAG_GLOBAL_SOLVE)
            r.ws_bytes = km.kmp_workspace_bytes(spec, n, 5, 1, r.fold, 1, 1, 1, 1)
        code = r.run()
        seen = dict(zip(km.KERNEL_CLASSES, r.timings.kernel_seen))
        print(code, seen["update"], seen["gemm_f"])
        out.append((code, r.results(), seen["update"] - seen["gemm_f"]))
    (c, g, dense), (cb, gb, none) = out
    assert dense > 0 and none == 0
    assert c == cb == km.KMP_WMAXITER and g["iters"].ravel()[0] == limit
    for k in ("alpha", "beta", "objective", "iters", "status"):
        assert np.array_equal(g[k], gb[k]), k
