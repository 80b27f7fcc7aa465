"""Large fronts of several instances in one batch, and the Newton step whose
forward solve runs inside the factorization against the separate solve."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_2606_04725_amd import nmpc as N
from test_gpu_batch import _note
from workloads import distillation_workload, plate_workload

pytestmark = pytest.mark.gpu

U = 2.0 ** -53
KEYS = ("y", "lam", "omega_d", "zL", "zU")


def _plate(G, H, seed):
    w = plate_workload("large", seed, G=G, H=H)
    p = N.Problem(N.plate_structure(G, H, w.dt, t_hi=w.T_hi, c_lo=w.u_lo, c_hi=w.u_hi))
    p.analyze()
    p.set_parameters(w.T0, setpoint=w.target, u_prev=np.full(16, 0.5))
    return p


def _column(n, h, seed):
    w = distillation_workload("small", seed, N=n, H=h)
    p = N.Problem(N.distillation_structure(n, h, w.dt, w.alpha, F=w.F, rho=w.rho))
    p.analyze()
    p.set_parameters(w.x0, setpoint=[w.xD_sp, w.xB_sp], traj=w.zF(0), u_prev=w.u_prev0)
    return p


def _members():
    return [_plate(16, 6, 1), _column(10, 20, 2), _plate(12, 20, 3), _plate(24, 4, 4), _plate(16, 6, 5)]


def test_batch_with_large_fronts_equals_one_by_one():
    """Plates of different sizes (fronts above 200 rows on different levels, one
    with fewer than 16 columns) and a column without any, together and alone."""
    a, b = _members(), _members()
    large = []
    for p in a:
        z = p.export_symbolic()
        large.append(int(np.sum(np.diff(z["snode_rows_ptr"]) > 200)))
    _note(f"large fronts per instance {large}")
    assert sum(n > 0 for n in large) == 4 and len(set(large)) > 2
    B = N.Batch(a)
    for warm in (False, True):
        rc, res = B.solve(warm=warm)
        assert rc == 0
        for k, (p, q) in enumerate(zip(a, b)):
            r = q.solve(warm=warm)
            assert r.status == 0
            assert (res[k].iters, res[k].factorizations, res[k].ls_trials) == (r.iters, r.factorizations, r.ls_trials), k
            s, t = p.solution(), q.solution()
            assert all(np.array_equal(s[key], t[key]) for key in KEYS), k
    B.close()


@pytest.mark.parametrize("make", [lambda: _column(10, 20, 6), lambda: _column(40, 12, 7), lambda: _plate(16, 6, 8),
                                  lambda: _plate(24, 4, 9), lambda: _plate(12, 14, 10)],
                         ids=["column 10x20", "column 40x12", "plate 16x6", "plate 24x4", "plate 12x14"])
def test_fused_step_equals_the_separate_solve(make):
    """One iteration from a held iterate: the step it takes in y solves the
    condensed system of that iterate, as the factorization and the separate solve
    do.  Its residual is a Cholesky solve's backward error plus the rounding of the
    iterates whose difference the step is."""
    p = make()
    mu = 1e-2
    o = N.default_options(fixed_mu=1, mu0_cold=mu, mu0_warm=mu, tol=1e-3, soc_max=0)
    assert p.solve(warm=False, options=o).status == 0
    it = p.get_iterate()
    rng = np.random.default_rng(3)
    # weights beta / s of the condensed system's rows near 100: positive definite, well conditioned
    it["s"] = rng.uniform(0.5, 2.0, p.ml)
    it["beta"] = rng.uniform(50.0, 200.0, p.ml)
    p.set_iterate(**it)
    kv, rhs = p.assemble(mu)
    ok, _ = p.factor(kv, want_l=False)
    assert ok
    dy = p.linear_solve(rhs)
    pat = p.patterns()
    r, c = pat["k_rows"].astype(np.int64), pat["k_cols"].astype(np.int64)
    off = r != c
    K = sp.coo_matrix((np.concatenate([kv, kv[off]]), (np.concatenate([r, c[off]]), np.concatenate([c, r[off]]))),
                      shape=(p.n, p.n)).tocsr()
    norm = np.max(np.abs(K).sum(1))
    m = int(np.max(np.diff(p.export_symbolic()["snode_rows_ptr"])))
    back = np.max(np.abs(K @ dy - rhs)) / (norm * np.max(np.abs(dy)) + np.max(np.abs(rhs)))
    assert back <= m * U, back
    p.set_iterate(**it)
    res = p.solve(warm=True, options=N.default_options(fixed_mu=1, mu0_warm=mu, tol=1e-14, soc_max=0, max_iter=1))
    assert res.iters == 1 and res.factorizations == 1 and res.eta == 0.0
    step = p.get_iterate()["y"] - it["y"]
    alpha = float(dy @ step) / float(dy @ dy)
    _note(f"step length {alpha:.3f}, |dy| {np.max(np.abs(dy)):.2e}, |K| {norm:.2e}")
    assert alpha > 0.0
    d = step / alpha
    tol = m * U * (norm * np.max(np.abs(dy)) + np.max(np.abs(rhs))) + 4 * U * norm * np.max(np.abs(it["y"])) / alpha
    e = np.max(np.abs(K @ d - rhs))
    _note(f"residual {e:.2e}, bound {tol:.2e}, right-hand side {np.max(np.abs(rhs)):.2e}")
    assert tol <= 1e-3 * np.max(np.abs(rhs))   # the bound tells a wrong right-hand side entry
    assert e <= tol
