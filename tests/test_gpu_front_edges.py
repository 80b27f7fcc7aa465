"""Front kernels where their rules change, against dense references: large
fronts with fewer columns than a block of 16, pivots over the whole range of
positive doubles and past it, both workgroup sizes on every one-workgroup front."""
import ctypes as C

import numpy as np
import pytest
import scipy.linalg as sla

from paper_2606_04725_amd import capi
from paper_2606_04725_amd import nmpc as N
from test_gpu_fronts import U, _check, _matrix, _note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,H", [(24, 4), (16, 14)])
def test_narrow_large_front(G, H):
    """A panel of fewer than 16 columns at the top of a large front."""
    m, w = _check(N.Problem(N.plate_structure(G, H, 0.01)), 3 * G + H, f"plate {G} x {G} x {H}")
    assert np.any((m > 200) & (w < 16))


def _structure(kind):
    return N.distillation_structure(10, 20, 0.05, 2.5) if kind == "small fronts" else N.plate_structure(16, 6, 0.01)


@pytest.mark.parametrize("kind", ["small fronts", "large fronts"])
def test_every_positive_pivot_is_accepted(kind):
    """A diagonal matrix, its pivots one value from the smallest subnormal to the
    largest double: accepted, and the factor is the root.  The reciprocal root is
    good to 2 roundings and the diagonal is its product with the pivot."""
    p = N.Problem(_structure(kind))
    p.analyze()
    z = p.export_symbolic()
    w, m = np.diff(z["snode_ptr"]), np.diff(z["snode_rows_ptr"])
    assert np.any(m > 200) == (kind == "large fronts")
    pat = p.patterns()
    diag = pat["k_rows"] == pat["k_cols"]
    at = np.concatenate([o + np.arange(a) * (b + 1) for o, a, b in zip(np.cumsum(w * m) - w * m, w, m)])
    for v in (5e-324, 1.5e-323, 1e-320, 1e-310, 5.5e-309, 5.6e-309, 2.3e-308, 1e-300, 3.0, 4e307, 1.7976931348623157e308):
        _note(f"{kind}: pivots {v}")
        ok, lv = p.factor(np.where(diag, v, 0.0))
        assert ok, v
        d = lv[at]
        assert np.max(np.abs(d - np.sqrt(v))) <= 4 * U * np.sqrt(v), (v, d[0], np.sqrt(v))
    for v in (0.0, -5e-324, -1.0, np.inf, np.nan):
        ok, _ = p.factor(np.where(diag, v, 0.0), want_l=False)
        assert not ok, v


@pytest.mark.parametrize("kind", ["small fronts", "large fronts"])
def test_factor_continues_past_a_bad_pivot(kind):
    """A pivot that is not positive and finite counts as 1: the factor returned is
    that of the matrix whose entry there makes it so (positive definite here: the
    entries off the diagonal are small), and solves with it."""
    p = N.Problem(_structure(kind))
    p.analyze()
    z, pat = p.export_symbolic(), p.patterns()
    start, rp, rows, perm = z["snode_ptr"], z["snode_rows_ptr"], z["snode_rows"], z["perm"]
    w, m = np.diff(start), np.diff(rp)
    big = m > 200
    assert np.any(big) == (kind == "large fronts")
    v, K = _matrix(pat, p.n, 17)
    r, c = pat["k_rows"].astype(np.int64), pat["k_cols"].astype(np.int64)
    off = r != c
    v[off] *= 0.1
    K = np.zeros((p.n, p.n))
    K[r, c] = v
    K[c, r] = v
    A = K[np.ix_(perm, perm)]
    slot = np.empty(p.n, np.int64)
    slot[r[~off]] = np.flatnonzero(~off)
    # columns of one front of the kind: the first, one inside and the last of a
    # block of 16, the first of the next one, the front's last
    s = int(np.argmax(np.where(big, w, 0) if kind == "large fronts" else w))
    low = np.arange(m.max())[:, None] >= np.arange(w.max())[None, :]
    for col in sorted({0, 5, min(15, int(w[s]) - 1), min(16, int(w[s]) - 1), int(w[s]) - 1}):
        b = int(start[s]) + col
        A1 = A.copy()
        A1[b, b] = 1.0
        if b > 0:
            A1[b, b] += np.sum(sla.solve_triangular(sla.cholesky(A[:b, :b], lower=True), A[:b, b], lower=True) ** 2)
        L = sla.cholesky(A1, lower=True)
        ev = np.linalg.eigvalsh(A1)
        tol = 2 * p.n * U * (ev[-1] / ev[0]) * np.max(np.abs(L))
        for bad in (-1e6, 0.0, np.inf, np.nan):
            _note(f"{kind}: front {s} ({m[s]} rows, {w[s]} columns), column {col}, entry {bad}")
            kv = v.copy()
            kv[slot[perm[b]]] = bad
            ok, lv = p.factor(kv)
            assert not ok
            o = 0
            for q in range(len(w)):
                P = lv[o:o + m[q] * w[q]].reshape(w[q], m[q]).T
                o += m[q] * w[q]
                want = L[np.ix_(rows[rp[q]:rp[q + 1]], np.arange(start[q], start[q + 1]))]
                at = low[:m[q], :w[q]]
                assert np.max(np.abs(P[at] - want[at])) <= tol, (q, int(m[q]), int(w[q]))
            rhs = np.random.default_rng(col).normal(size=p.n)
            x = np.empty(p.n)
            x[:] = p.linear_solve(rhs)[perm]
            back = np.max(np.abs(A1 @ x - rhs[perm])) / (np.max(np.abs(A1).sum(1)) * np.max(np.abs(x)) + np.max(np.abs(rhs)))
            assert back <= m.max() * U, back


def _force(p, variant):
    f = capi.lib().nmpc_internal_front_variant
    f.restype, f.argtypes = C.c_int32, [C.c_void_p, C.c_int32]
    assert f(p._h, variant) == 0


@pytest.mark.parametrize("kind,a,b", [("column", 4, 1), ("column", 100, 15), ("plate", 12, 14), ("plate", 24, 4)])
def test_every_workgroup_size_on_every_front(kind, a, b):
    """The autotuner may give 256 or 512 threads to any one-workgroup launch: both
    against the dense factor, and the same bits.  The plates have fronts at the
    edges of a wave's rows (64, 65, 112 to 114, 159 to 161) and of the class (200)."""
    st = N.distillation_structure(a, b, 0.05, 2.5) if kind == "column" else N.plate_structure(a, b, 0.01)
    p = N.Problem(st)
    p.analyze()
    z, pat = p.export_symbolic(), p.patterns()
    start, rp, rows, perm = z["snode_ptr"], z["snode_rows_ptr"], z["snode_rows"], z["perm"]
    w, m = np.diff(start), np.diff(rp)
    kv, K = _matrix(pat, p.n, 7 * a + b)
    A = K[np.ix_(perm, perm)] + 0.25 * np.eye(p.n)
    L = sla.cholesky(A, lower=True)
    # as in the checks of the default variants: dominant by 1.25, rows of norm <= 2 |diagonal|
    tol = 2 * p.n * U * (2.0 * np.max(np.diag(A)) / 1.25) * np.max(np.abs(L))
    low = np.arange(m.max())[:, None] >= np.arange(w.max())[None, :]
    seen = []
    for variant in (0, 1):
        _force(p, variant)
        _note(f"{kind} {a} x {b}: fronts of {m.min()} to {m[m <= 200].max()} rows, variant {variant}")
        ok, lv = p.factor(kv, eta=0.25)
        assert ok
        o = 0
        for q in range(len(w)):
            P = lv[o:o + m[q] * w[q]].reshape(w[q], m[q]).T
            o += m[q] * w[q]
            want = L[np.ix_(rows[rp[q]:rp[q + 1]], np.arange(start[q], start[q + 1]))]
            at = low[:m[q], :w[q]]
            d = np.max(np.abs(P[at] - want[at]))
            assert d <= tol, (q, int(w[q]), int(m[q]), d, tol)
            P[~at] = 0.0   # above the diagonal nothing is defined
        seen.append((lv, p.linear_solve(np.ones(p.n))))
    assert np.array_equal(seen[0][0], seen[1][0]) and np.array_equal(seen[0][1], seen[1][1])
