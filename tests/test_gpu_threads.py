"""Handles used by one host thread each, several threads at a time: creation,
analysis, graph captures (every change of options), solves, iterates, sensitivities
and destruction, with the results of the same work done by one thread."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_2606_04725_amd import nmpc as N
from test_gpu_multi import KEYS, _column, _note, _plate

pytestmark = pytest.mark.gpu


def _work(k):
    make = [lambda: _column(10, 20, 1), lambda: _plate(16, 6, 2), lambda: _column(23, 21, 3), lambda: _plate(8, 5, 4),
            lambda: _column(40, 12, 5), lambda: _plate(12, 9, 6)][k]
    out = []
    for rep in range(2):
        p = make()
        if rep:
            p.autotune(reps=1)
        r = p.solve(warm=False)
        out.append((r.status, r.iters, r.passes))
        for tol in (1e-7, 1e-9, 1e-8):   # other options: the pass is captured again
            r = p.solve(warm=True, options=N.default_options(fixed_mu=1, mu0_warm=1e-7, tol=tol))
            s = p.solution()
            out.append((r.status, r.iters, [s[key] for key in KEYS]))
            out.append(p.first_stage())
        it = p.get_iterate()
        rc, J = p.jacobian_u1_x0()
        out.append((rc, J))
        p.set_iterate(**it)
        r = p.solve(warm=True)
        out.append((r.status, r.iters, p.solution()["y"]))
        q = make()
        B = N.Batch([p, q])
        rc, res = B.solve(warm=False)
        out.append((rc, [x.iters for x in res], p.solution()["y"], q.solution()["y"]))
        B.close()
        kv, rhs = p.assemble(1e-4)
        ok, _ = p.factor(kv, want_l=False)
        out.append((ok, kv, rhs, p.linear_solve(rhs)))
        p.close()
        q.close()
    return out


def _same(a, b):
    if isinstance(a, (list, tuple)):
        return len(a) == len(b) and all(_same(x, y) for x, y in zip(a, b))
    return np.array_equal(a, b) if isinstance(a, np.ndarray) else a == b


def test_threads_with_a_handle_each_equal_one_thread():
    one = [_work(k) for k in range(6)]
    for trial in range(3):
        _note(f"six threads, trial {trial}")
        with ThreadPoolExecutor(6) as ex:
            many = list(ex.map(_work, range(6)))
        for k in range(6):
            assert _same(one[k], many[k]), k
