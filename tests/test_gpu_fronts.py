"""Front kernels at the edges of their tiles: every supernodal panel of a
factorization against a dense Cholesky factorization, and a solve with it, on
plates whose large fronts end panels of 64 columns and blocks of 16 columns and
rows at full, partial and empty remainders, and on columns whose one-workgroup
fronts do the same at 8 and 16 columns, 16 and 48 rows."""
import sys

import numpy as np
import pytest
import scipy.linalg as sla
import scipy.sparse as sp

from paper_2606_04725_amd import nmpc as N

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _note(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


def _matrix(pat, n, seed):
    """A symmetric diagonally dominant matrix on the pattern, its slot values."""
    rng = np.random.default_rng(seed)
    r, c = pat["k_rows"].astype(np.int64), pat["k_cols"].astype(np.int64)
    v = rng.uniform(-1.0, 1.0, r.size)
    off = r != c
    weight = np.bincount(r[off], np.abs(v[off]), n) + np.bincount(c[off], np.abs(v[off]), n)
    v[~off] = 1.0 + weight[r[~off]]
    K = np.zeros((n, n))
    K[r, c] = v
    K[c, r] = v
    return v, K


def _check(p, seed, name):
    p.analyze()
    z = p.export_symbolic()
    start, rp, rows, perm = z["snode_ptr"], z["snode_rows_ptr"], z["snode_rows"], z["perm"]
    w, m = np.diff(start), np.diff(rp)
    large = m > 200   # such a front's packed triangle exceeds shared memory
    _note(f"{name}: {large.sum()} of {m.size} fronts large, up to {m.max()} rows and {w.max()} columns")
    kv, K = _matrix(p.patterns(), p.n, seed)
    ok, lv = p.factor(kv, eta=0.25)
    assert ok
    A = K[np.ix_(perm, perm)] + 0.25 * np.eye(p.n)
    L = sla.cholesky(A, lower=True)
    # |L - L_ref| <= c n u cond(A) |L| for either factorization; the matrix is
    # diagonally dominant by 1.25 with rows of norm <= 2 |diagonal|
    scale = np.max(np.abs(L))
    cond = 2.0 * np.max(np.diag(A)) / 1.25
    tol = 2 * p.n * U * cond * scale
    off = 0
    for s in range(len(w)):
        P = lv[off:off + m[s] * w[s]].reshape(w[s], m[s]).T
        off += m[s] * w[s]
        R = rows[rp[s]:rp[s + 1]]
        want = L[np.ix_(R, np.arange(start[s], start[s + 1]))]
        low = np.tril(np.ones((m[s], w[s]), bool))
        d = np.max(np.abs(P[low] - want[low]))
        assert d <= tol, (s, int(w[s]), int(m[s]), d, tol)
    b = np.random.default_rng(seed).normal(size=p.n)
    x = p.linear_solve(b)
    M = K + 0.25 * np.eye(p.n)
    back = np.max(np.abs(M @ x - b)) / (np.max(np.sum(np.abs(M), 1)) * np.max(np.abs(x)) + np.max(np.abs(b)))
    assert back <= m.max() * U, back
    return m, w


@pytest.mark.parametrize("G,H", [(16, 6), (20, 5), (12, 20), (16, 14)])
def test_large_front_factor_and_solve(G, H):
    m, w = _check(N.Problem(N.plate_structure(G, H, 0.01)), 7 * G + H, f"plate {G} x {G} x {H}")
    assert np.any(m > 200)


def test_front_wider_than_an_outer_panel():
    """Fronts of more than 512 columns with rows below: the trailing update after
    the first 512 columns crosses from the panel into the update block."""
    p = N.Problem(N.plate_structure(28, 37, 0.01))
    p.analyze()
    z = p.export_symbolic()
    w, m = np.diff(z["snode_ptr"]), np.diff(z["snode_rows_ptr"])
    assert np.any((w > 512) & (m > w))
    _note(f"plate 28 x 28 x 37: widest front {w.max()} columns, {m.max()} rows at most")
    pat = p.patterns()
    rng = np.random.default_rng(5)
    r, c = pat["k_rows"].astype(np.int64), pat["k_cols"].astype(np.int64)
    v = rng.uniform(-1.0, 1.0, r.size)
    off = r != c
    weight = np.bincount(r[off], np.abs(v[off]), p.n) + np.bincount(c[off], np.abs(v[off]), p.n)
    v[~off] = 1.0 + weight[r[~off]]
    ok, _ = p.factor(v, eta=0.25)
    assert ok
    b = rng.normal(size=p.n)
    x = p.linear_solve(b)
    M = sp.coo_matrix((np.concatenate([v, v[off]]), (np.concatenate([r, c[off]]), np.concatenate([c, r[off]]))),
                      shape=(p.n, p.n)).tocsr() + 0.25 * sp.identity(p.n)
    # backward error of a Cholesky solve: at most the largest front's order times the unit roundoff
    back = np.max(np.abs(M @ x - b)) / (np.max(np.abs(M).sum(1)) * np.max(np.abs(x)) + np.max(np.abs(b)))
    assert back <= m.max() * U, back


@pytest.mark.parametrize("trays,H", [(4, 1), (6, 3), (10, 20), (23, 41), (60, 24)])
def test_small_front_factor_and_solve(trays, H):
    m, w = _check(N.Problem(N.distillation_structure(trays, H, 0.05, 2.5)), 100 * trays + H, f"column {trays} x {H}")
    assert not np.any(m > 200)


def test_indefinite_front_is_reported():
    p = N.Problem(N.distillation_structure(10, 20, 0.05, 2.5))
    p.analyze()
    pat = p.patterns()
    kv, _ = _matrix(pat, p.n, 3)
    diag = np.flatnonzero(pat["k_rows"] == pat["k_cols"])
    for at in (diag[0], diag[p.n // 2], diag[-1]):   # one pivot at a time, in different fronts
        for bad in (-1e6, np.nan, np.inf):
            v = kv.copy()
            v[at] = bad
            ok, _ = p.factor(v, want_l=False)
            assert not ok
    ok, _ = p.factor(kv, want_l=False)
    assert ok
