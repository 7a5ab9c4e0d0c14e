"""Small orders (small.hip: a column's whole path in one workgroup) and the
dense form of a stage's last columns (dense.hip) against the batched iteration
(KMP_FLAG_GLOBAL_SOLVE, which takes neither) on the same problem: the objective
and coefficient bars of the oracle comparisons. Sizes lie on the edges of the
variants: orders 64 to 256, the first order above, odd sizes, and more columns
than compute units."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import ALPHA_RTOL, CV_RTOL, OBJ_RTOL, announce, device

pytestmark = pytest.mark.gpu


def _both(inp, loss, ws=None, **kw):
    from paper_2606_06742_amd import kmpath as km
    device()
    out = []
    for flag in (0, km.KMP_FLAG_GLOBAL_SOLVE):
        r = km.PathRunner(inp["X"], inp["y"], loss, inp["sigmas"], inp["lambdas"], inp["fold_id"],
                          inp["V"], taus=inp["taus"] if loss == "check" else None, **kw)
        r.spec.flags |= flag
        if ws is not None:
            r.ws_bytes = ws(r, km)
        out.append((r.run(), r.results()))
    return out


def _agree(a, b):
    (ca, ga), (cb, gb) = a, b
    assert ca == cb and np.array_equal(ga["status"], gb["status"])
    assert np.all(np.abs(ga["objective"] - gb["objective"]) <= OBJ_RTOL * np.abs(gb["objective"]))
    scale = np.abs(gb["alpha"]).max(axis=-1, keepdims=True)
    assert np.all(np.abs(ga["alpha"] - gb["alpha"]) <= ALPHA_RTOL * scale)
    assert np.all(np.abs(ga["cv_sum"] - gb["cv_sum"]) <= CV_RTOL * np.maximum(1.0, gb["cv_sum"]))
    assert np.array_equal(ga["selected"], gb["selected"])


@pytest.mark.parametrize("loss,n,V,mode", [
    ("hinge", 85, 4, {}),                    # order 64, one row short of it
    ("check", 97, 3, {}),                    # order 128 (65 rows)
    ("logistic", 191, 3, {}),
    ("hinge", 233, 6, {}),                   # order 256
    ("hinge", 256, 1, {"refit": True}),      # order 256, no padding
    ("check", 257, 1, {"refit": True}),      # the first order above one compute unit
    ("logistic", 601, 3, {}),
    ("hinge", 701, 3, {}),
    ("hinge", 190, 5, {"shared": True}),
    ("check", 333, 4, {"shared": True}),
])
def test_dense_matches_batched(loss, n, V, mode):
    inp = W.small_problem(loss, n, 5, seed=n, V=max(V, 2), L=7, lam_lo=-4.0, lam_hi=0.0)
    announce(f"dense columns loss={loss} n={n} V={V} {mode}")
    a, b = _both(inp, loss, **mode)
    assert a[0] == 0
    _agree(a, b)


def test_small_leave_one_out():
    """n = 190: 1140 columns of order 192, several per compute unit."""
    inp = W.small_problem("hinge", 190, 4, seed=7, V=2, L=6, lam_lo=-3.0, lam_hi=0.0)
    inp["fold_id"], inp["V"] = np.arange(190, dtype=np.int32), 190
    announce("small order, leave-one-out n=190 L=6")
    _agree(*_both(inp, "hinge", shared=True))


@pytest.mark.parametrize("n,L", [(67, 8), (130, 7), (150, 3)])
def test_small_one_resolvent_for_several_columns(n, L):
    """Logistic leave-one-out: the columns of a penalty share the resolvent, in
    runs that end inside a penalty's columns and inside the last workgroup's."""
    inp = W.small_problem("logistic", n, 4, seed=n, V=2, L=L, lam_lo=-3.0, lam_hi=0.0)
    inp["fold_id"], inp["V"] = np.arange(n, dtype=np.int32), n
    announce(f"small order, logistic leave-one-out n={n} L={L}")
    _agree(*_both(inp, "logistic", shared=True))


def test_dense_needs_no_workspace():
    """A workspace without the optional part runs batched iterations only, one
    with part of it takes fewer columns: the same results to rounding."""
    inp = W.small_problem("hinge", 450, 4, seed=8, V=3, L=5, lam_lo=-3.0, lam_hi=0.0)
    sizes = []

    def fixed(extra):
        def size(r, km):
            spec = km.kmp_default_spec("hinge", flags=r.spec.flags | km.KMP_FLAG_GLOBAL_SOLVE)
            b = km.kmp_workspace_bytes(spec, 450, 4, 5, r.fold, 3, 1, 1, 1)
            sizes.append((b, r.ws_bytes))
            return b + extra
        return size

    announce("dense columns: workspace without the optional part")
    for extra in (0, 72 << 20):
        _agree(*_both(inp, "hinge", ws=fixed(extra)))
    assert sizes[0][0] < sizes[0][1]


@pytest.mark.parametrize("n,max_iter", [(100, 40), (100, 8), (500, 200), (500, 60)])
def test_dense_stops_at_max_iter(n, max_iter):
    """Columns that reach max_iter in dense form report it after exactly that
    many iterations, as in batched form, from the same iterates."""
    from paper_2606_06742_amd import kmpath as km
    inp = W.small_problem("hinge", n, 4, seed=9, V=3, L=4, lam_lo=-5.0, lam_hi=-3.0)
    announce(f"dense columns: max_iter={max_iter} n={n}")
    (ca, a), (cb, b) = _both(inp, "hinge", max_iter=max_iter)
    assert ca == cb == km.KMP_WMAXITER
    assert np.array_equal(a["status"], b["status"]) and np.array_equal(a["iters"], b["iters"])
    scale = np.abs(b["alpha"]).max(axis=-1, keepdims=True)
    assert np.all(np.abs(a["alpha"] - b["alpha"]) <= ALPHA_RTOL * scale)


@pytest.mark.parametrize("L", [5, 20])
def test_workspace_for_fewer_bandwidths(L):
    """Three bandwidths in a workspace sized for one: a larger batch with fewer
    dense columns or none, the same results."""
    inp = W.small_problem("hinge", 450, 4, seed=8, V=3, L=L, lam_lo=-3.0, lam_hi=0.0)
    inp["sigmas"] = np.asarray(inp["sigmas"])[0] * np.array([1.0, 0.5, 2.0])
    announce(f"workspace sized for one bandwidth of three, L={L}")
    one, _ = _both(inp, "hinge", sigma_batch=1)
    _agree(one, _both(inp, "hinge")[1])


@pytest.mark.parametrize("loss,n,V,L,mode,taken", [
    ("hinge", 701, 3, 7, {}, True),
    ("check", 333, 4, 7, {"shared": True}, True),
    ("logistic", 760, 3, 40, {}, False),     # tens of iterations: over before it would pay
])
def test_dense_form_is_taken_where_it_pays(loss, n, V, L, mode, taken):
    """Every batched iteration has one loss product and one update, a dense one an
    update only."""
    from paper_2606_06742_amd import kmpath as km
    device()
    inp = W.small_problem(loss, n, 12, seed=n, V=V, L=L, lam_lo=-4.0, lam_hi=0.0)
    announce(f"dense form taken: loss={loss} n={n} {mode}")
    r = km.PathRunner(inp["X"], inp["y"], loss, inp["sigmas"], inp["lambdas"], inp["fold_id"], V,
                      taus=inp["taus"] if loss == "check" else None, eager=True,
                      kernel_timing=("update", "gemm_f"), **mode)
    assert r.run() == 0
    seen = dict(zip(km.KERNEL_CLASSES, r.timings.kernel_seen))
    print(seen["update"], seen["gemm_f"], r.iters.max().item())
    assert (seen["update"] > seen["gemm_f"]) == taken and seen["gemm_f"] > 0


@pytest.mark.parametrize("loss,n,V,L,kw,taken", [
    ("hinge", 200, 5, 10, {}, True),
    ("check", 190, 3, 40, {}, True),
    ("hinge", 250, 1, 2000, {"tol": 1e-2, "n_stages": 1}, False),   # the sweeps alone take longer
    ("check", 250, 1, 2000, {"max_iter": 20}, False),
])
def test_small_orders_where_they_pay(loss, n, V, L, kw, taken):
    """A fit in batched form has a factorisation, one of small orders none."""
    from paper_2606_06742_amd import kmpath as km
    device()
    inp = W.small_problem(loss, n, 4, seed=n, V=max(V, 2), L=L, lam_lo=-4.0, lam_hi=0.0)
    announce(f"small orders taken: loss={loss} n={n} L={L} {kw}")
    r = km.PathRunner(inp["X"], inp["y"], loss, inp["sigmas"], inp["lambdas"], inp["fold_id"], V,
                      taus=inp["taus"][:1] if loss == "check" else None, refit=V == 1, **kw)
    assert r.run() >= 0
    assert (r.timings.factor_ms == 0) == taken
