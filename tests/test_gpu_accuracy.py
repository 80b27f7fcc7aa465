"""Rounding of a factorization and solve, against the solution in 64 bits by
conjugate gradients on the matrix (perf/cases.py)."""
import numpy as np
import pytest

from perf import cases
from test_gpu_batch import _note

pytestmark = pytest.mark.gpu

SIZES = [(8, 4), (8, 9), (8, 17), (8, 30), (12, 5), (12, 11), (12, 23), (16, 4), (16, 7), (16, 13), (20, 4), (20, 9)]
# mean over these matrices where pivots go eight columns at a time and everything
# else is summed from zero; the mean is the same from run to run in these digits
EIGHT_COLUMN_PANELS = 1.1316e-15


def test_mean_error_is_that_of_eight_column_panels():
    e = []
    for g, h in SIZES:
        for seed in range(8):
            c = dict(path="factor", model="plate", size=g, horizon=h)
            ok, x = cases.run(cases.prepare(c, seed))
            w = cases.exact(c, seed)[1]
            assert ok
            e.append(np.linalg.norm(np.asarray(x) - w) / np.linalg.norm(w))
        _note(f"plate {g} x {g} x {h}: mean error {np.mean(e[-8:]):.3e}")
    _note(f"mean {np.mean(e):.4e}")
    assert np.mean(e) <= EIGHT_COLUMN_PANELS
