"""kmp_rbf_gram at the edges of its tiles and load forms against direct
differences in numpy: sizes around the 64-point tile, feature counts around
the 16-feature slice, odd feature counts and leading dimensions (single loads
instead of pairs), one list for rows and columns (symmetric form), padding
entries and far points whose kernel value underflows.

Bound: the expansion |x|^2 + |y|^2 - 2 x.y of n terms carries at most
(d + 3) eps (|x|^2 + |y|^2) of error in the squared distance, hence that
times 1/(2 sigma^2) in the relative error of exp, plus a few eps of exp and of
the reference."""
import numpy as np
import pytest

from tests.gpu_common import announce, device

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.mark.parametrize("m,p,d,ldx,S,same", [
    (1, 1, 1, 1, 1, False), (63, 65, 2, 2, 1, False), (64, 64, 16, 16, 2, False),
    (65, 130, 17, 17, 1, False), (129, 40, 33, 40, 3, False), (70, 90, 32, 33, 8, False),
    (64, 64, 15, 16, 1, True), (65, 65, 16, 16, 2, True), (200, 200, 100, 100, 3, True),
    (131, 131, 7, 9, 1, True), (1, 1, 3, 3, 1, True)])
def test_gram_edges(m, p, d, ldx, S, same):
    import torch
    from paper_2606_06742_amd import kmpath as km
    dev = device()
    announce(f"kmp_rbf_gram edges m={m} p={p} d={d} ldx={ldx} S={S} same={same}")
    rng = np.random.default_rng(m * 1000 + p + d)
    n = max(m, p) + 5
    X = rng.standard_normal((n, d))
    X[-1] *= 1e4                                     # its kernel values underflow
    buf = torch.full((n, ldx), np.nan, dtype=torch.float64, device=dev)
    buf[:, :d] = torch.as_tensor(X)
    rows = rng.permutation(n)[:m].astype(np.int32)
    cols = rows if same else rng.permutation(n)[:p].astype(np.int32)
    if m > 4:
        rows = rows.copy()
        rows[[2, m - 1]] = -1, n - 1
        cols = rows if same else cols
    tr = torch.as_tensor(rows, device=dev)
    tc = tr if same else torch.as_tensor(cols, device=dev)
    sig = np.array([1.0, 0.5, 2.0, 4.0, 0.7, 1.3, 3.0, 0.2])[:S] * np.sqrt(d)
    out = torch.full((S, m, p + 3), np.nan, dtype=torch.float64, device=dev)
    km.kmp_rbf_gram(buf[:, :d], tr, tc, sig, out[:, :, :p])
    got = out.cpu().numpy()
    assert np.all(np.isnan(got[:, :, p:]))           # nothing past the columns
    pad = (rows[:, None] < 0) | (cols[None, :] < 0)
    A, B = X[rows], X[cols]
    d2 = ((A[:, None] - B[None]) ** 2).sum(-1)
    size = (A ** 2).sum(-1)[:, None] + (B ** 2).sum(-1)[None]
    for s in range(S):
        f = 1.0 / (2.0 * sig[s] ** 2)
        want = np.where(pad, 0.0, np.exp(-d2 * f))
        want[(rows[:, None] == cols[None, :]) & ~pad] = 1.0
        tol = want * (2.0 * (d + 3) * EPS * size * f + 8.0 * EPS)
        assert np.all(np.abs(got[s, :, :p] - want) <= np.maximum(tol, 1e-300)), s
        if same:
            assert np.array_equal(got[s, :, :p], got[s, :, :p].T)
