"""Front kernels where their rules change, against dense references: large
fronts with fewer columns than a block of 16, pivots over the whole range of
positive doubles."""
import numpy as np
import pytest

from paper_2606_04725_amd import nmpc as N
from test_gpu_fronts import U, _check, _note

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
