"""The numbered reports that a solve waits for, over the wrap of their 16-bit
number."""
import numpy as np
import pytest

from paper_2606_04725_amd import nmpc as N
from test_gpu_batch import _next, _note, _problem
from workloads import distillation_workload

pytestmark = pytest.mark.gpu


def test_report_numbers_wrap():
    """One report per solve: a solution re-solved on its own barrier problem is
    found converged by the evaluation that opens the solve."""
    w = distillation_workload("small", 31, N=2, H=1, n_resolves=2)
    p = _problem(w)
    o = N.default_options(fixed_mu=1, mu0_warm=1e-6, tol=1e-8)
    assert p.solve(warm=False).status == 0
    assert p.solve(warm=True, options=o).status == 0
    y = p.solution()["y"]
    _note("66000 solves of one report each")
    for k in range(66000):
        r = p.solve(warm=True, options=o)
        assert r.status == 0 and r.iters == 0 and r.passes == 1, k
        if k % 11000 == 0:
            _note(f"solve {k}")
    assert np.array_equal(p.solution()["y"], y)
    _next(p, w, 0)   # and passes after it
    r = p.solve(warm=True)
    q = _problem(w)
    q.solve(warm=False)
    q.solve(warm=True, options=o)
    _next(q, w, 0)
    s = q.solve(warm=True)
    assert r.status == 0 and (r.iters, r.passes) == (s.iters, s.passes)
    assert np.array_equal(p.solution()["y"], q.solution()["y"])
