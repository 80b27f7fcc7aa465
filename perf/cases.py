"""Performance cases: the work a program that controls a plant with this framework has it do.

Every case is a dict with a ``path`` (what is called) and its sizes:

resolve      ``periods`` control periods of Algorithm 1 on one problem: the measured state, setpoint, disturbance
             forecast and last control go in from host memory (``set_parameters``), one warm solve, the applied
             control and the predicted state come out (``first_stage``).
batch        the same for ``count`` columns of uneven sizes solved together (``Batch``).
loop         Algorithm 1 with plant = model on the device (``closed_loop_dev``), tables resident on the GPU.
gradient     the solve as a layer of a differentiable program: ``NMPCSolve`` forward and backward on GPU tensors.
jacobian     control periods whose caller also wants the feedback gain d u1 / d x0 (``jacobian_u1_x0``).
factor       the linear algebra alone: ``factor`` of a condensed matrix and ``linear_solve`` with it.

Models (``model``): the workload column (``column``: trays x horizon), the distillation case study (``reflux``: 32
trays), the heated plate (``plate``: grid x grid x horizon), the heated-plate case study written with index-data patterns
(``plate_case``: 21 x 21, kernels generated by the front end).  Sizes are those of the workloads (columns of 10 x 20 and
40 x 100, 20..60 trays x 40..120 stages in a batch, plates of 8 x 8 x 5 up to several tens squared x 50) and sizes between.

Every solve is of one barrier problem to a tight tolerance (``fixed_mu``, E_mu <= TOL), the setting in which a program
that differentiates the solution or compares solutions needs it: the iterate is then determined far beyond the default
stopping ball.  Inputs come from the seed alone: a measured state is a nominal profile plus measurement noise.
"""
import math
from concurrent.futures import ThreadPoolExecutor
from functools import lru_cache

import numpy as np
import torch

from paper_2606_04725_amd import nmpc as N
from paper_2606_04725_amd import simd
from paper_2606_04725_amd import simd_models as SM
from paper_2606_04725_amd.autograd import NMPCSolve

TOL = 1e-12         # E_mu of every timed solve
MU = 1e-9           # its barrier value (the method's smallest)
NEWTON = 3          # Newton iterations a warm solve takes at least (work only)


def listed():
    return [
        # the smallest real-time controller: a 10-tray column, latency and launches
        dict(name="column 10x20", path="resolve", model="column", size=10, horizon=20, periods=4, kkt="lifted"),
        # the headline workload
        dict(name="column 40x100", path="resolve", model="column", size=40, horizon=100, periods=4, kkt="lifted"),
        # equalities kept exact, conjugate gradients around the factor; odd sizes
        dict(name="column 23x41 hykkt", path="resolve", model="column", size=23, horizon=41, periods=2, kkt="hykkt"),
        # the distillation case study: algebraic variables, horizon of 180 s
        dict(name="reflux 32x90", path="resolve", model="reflux", size=32, horizon=90, periods=3, kkt="lifted"),
        # the heated-plate case study through generated kernels
        dict(name="plate case 21x12", path="resolve", model="plate_case", size=21, horizon=12, periods=2, kkt="lifted"),
        # the large workload plate
        dict(name="plate 32x50", path="resolve", model="plate", size=32, horizon=50, periods=2, kkt="lifted"),
        # many uneven columns served by one GPU
        dict(name="batch 24", path="batch", model="column", size=60, horizon=120, count=24, periods=2),
        # simulation study of a closed loop without host round trips
        dict(name="loop 40x100", path="loop", model="column", size=40, horizon=100, periods=10),
        # a controller inside a training loop, small plate
        dict(name="gradient plate 16x25", path="gradient", model="plate", size=16, horizon=25, periods=2),
        # and the headline column
        dict(name="gradient column 40x100", path="gradient", model="column", size=40, horizon=100, periods=2),
        # the largest: solves and feedback gains of a fine plate
        dict(name="jacobian plate 40x50", path="jacobian", model="plate", size=40, horizon=50, periods=2),
        # the sparse direct solver by itself
        dict(name="factor plate 28x37", path="factor", model="plate", size=28, horizon=37),
    ]


def _log(rng, lo, hi):
    """An integer between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _plate_size(rng, most):
    """Grid (a multiple of 4: four heater segments per edge) and horizon of at most ``most`` unknown temperatures."""
    while True:
        g, h = 4 * _log(rng, 2, 12), _log(rng, 4, 60)
        if g * g * h <= most:
            return dict(size=g, horizon=h)


def draw(rng):
    path = rng.choice(["resolve", "resolve", "resolve", "batch", "loop", "gradient", "jacobian", "factor"])
    column = dict(model="column", size=_log(rng, 6, 60), horizon=_log(rng, 12, 120))
    if path == "resolve":
        kind = rng.choice(["column", "column", "hykkt", "reflux", "plate_case", "plate", "plate"])
        if kind in ("column", "hykkt"):
            return dict(path=path, **column, periods=rng.randint(2, 4), kkt="hykkt" if kind == "hykkt" else "lifted")
        if kind == "plate":
            return dict(path=path, model="plate", **_plate_size(rng, 64_000), periods=2, kkt="lifted")
        if kind == "reflux":
            return dict(path=path, model="reflux", size=32, horizon=_log(rng, 20, 110), periods=2, kkt="lifted")
        return dict(path=path, model="plate_case", size=21, horizon=_log(rng, 4, 24), periods=2, kkt="lifted")
    if path == "batch":
        return dict(path=path, model="column", size=rng.randint(30, 60), horizon=rng.randint(60, 120),
                    count=_log(rng, 3, 24), periods=2)
    if path == "loop":
        return dict(path=path, **column, periods=rng.randint(3, 12))
    if path == "factor":
        return dict(path=path, model="plate", **_plate_size(rng, 64_000))
    if path == "gradient" and rng.random() < 0.5:
        return dict(path=path, **column, periods=2)
    return dict(path=path, model="plate", **_plate_size(rng, 30_000 if path == "gradient" else 40_000), periods=2)


# ---- problems ------------------------------------------------------------------------------------------------------
def _options(kkt="lifted"):
    return N.default_options(fixed_mu=1, mu0_warm=MU, tol=TOL, max_iter=60, kkt=1 if kkt == "hykkt" else 0)


def _profile(nx):
    """Composition profile of a column, condenser to reboiler."""
    return 0.5 + 0.45 * np.tanh(4.0 * (0.5 - np.arange(nx) / (nx - 1)))


@lru_cache(maxsize=None)
def _plate_case_kernels():
    return simd.compile(SM.plate_case_pattern_model(n=21, alpha=230.0, Tb=50.0, loss=50.0, rho=1e-8, Q_lo=50.0,
                                                    q_scale=1e4, dt=0.08))


def _structure(model, size, horizon, alpha=2.5):
    if model == "column":
        return N.distillation_structure(size, horizon, 0.05, alpha)
    if model == "reflux":
        return N.reflux_structure(horizon, N=size)
    if model == "plate":
        return N.plate_structure(size, horizon, 0.01)
    return N.stage_model_structure(_plate_case_kernels(), H=horizon, dt=0.08)


def _inputs(model, size, horizon, periods, rng):
    """The parameters of ``periods`` successive solves: dicts of set_parameters' arguments."""
    out = []
    if model == "column":
        base = _profile(size + 2) + rng.normal(0.0, 0.01, size + 2)
        sp = np.array([rng.uniform(0.90, 0.98), rng.uniform(0.02, 0.10)])
        t0 = rng.uniform(0.0, 6.0)
        for k in range(periods):
            x0 = np.clip(base + rng.normal(0.0, 0.003, size + 2), 0.0, 1.0)
            feed = 0.5 + 0.05 * np.sin(t0 + 0.05 * (k + np.arange(1, horizon + 1)))
            out.append(dict(x0=x0, setpoint=sp, traj=feed, u_prev=np.array([2.0, 2.5]) + rng.normal(0.0, 0.02, 2)))
    elif model == "reflux":
        base = np.linspace(0.85, 0.12, size)
        for k in range(periods):
            out.append(dict(x0=base + rng.normal(0.0, 0.005, size), setpoint=np.array([0.8958, 2.51459]), traj=None,
                            u_prev=np.array([2.0 + rng.normal(0.0, 0.02)])))
    elif model == "plate":
        c = np.arange(1, size + 1) / (size + 1)
        X, Y = np.meshgrid(c, c)
        a, cx, cy, s = rng.uniform(0.3, 0.8), rng.uniform(0.3, 0.7), rng.uniform(0.3, 0.7), rng.uniform(0.1, 0.25)
        target = (a * np.exp(-((X - cx) ** 2 + (Y - cy) ** 2) / (2.0 * s * s))).reshape(-1)
        for k in range(periods):   # the plate warming towards its target
            x0 = (0.2 + 0.1 * k) * target + rng.normal(0.0, 0.005, size * size)
            out.append(dict(x0=x0, setpoint=target, traj=None, u_prev=np.full(16, 0.5)))
    else:
        nx = (size - 2) ** 2
        for k in range(periods):
            out.append(dict(x0=50.0 + k + rng.normal(0.0, 0.2, nx), setpoint=None, traj=np.full(horizon, 58.0),
                            u_prev=np.array([0.005])))
    return out


def _solved(structure, params):
    """An analyzed problem holding the solution for ``params``."""
    p = N.Problem(structure)
    p.analyze()
    p.set_parameters(**params)
    p.solve(warm=False)
    return p


# ---- a condensed matrix of the plate --------------------------------------------------------------------------------
def _plate_rows(grid, horizon):
    """The state rows of the plate: for every row its columns (own node, four neighbours or heater segments, the node a
    stage before; -1 for none), nodes row-major, heater segments after the stage's nodes, edges bottom, right, top, left."""
    q, nx = grid // 4, grid * grid
    b, a = np.divmod(np.arange(nx), grid)
    own = np.arange(nx)
    nb = np.stack([np.where(b > 0, own - grid, nx + a // q), np.where(a < grid - 1, own + 1, nx + 4 + b // q),
                   np.where(b < grid - 1, own + grid, nx + 8 + a // q), np.where(a > 0, own - 1, nx + 12 + b // q)], 1)
    ns = nx + 16
    stage = ns * np.arange(horizon)[:, None, None]
    cols = np.concatenate([np.broadcast_to(own[:, None], (horizon, nx, 1)) + stage, nb[None] + stage,
                           np.where(stage > 0, own[:, None] + stage - ns, -1)], 2)
    return cols.reshape(horizon * nx, 6)


def _plate_matrix(grid, horizon, rng):
    """(rows, cols, values) of the lower triangle of D + J^T Q J: the linear plate's rows J with weights Q and barrier
    terms D as an early iterate has them (the lifted weights grow later), duplicates summed."""
    n = horizon * (grid * grid + 16)
    cols = _plate_rows(grid, horizon)
    a = 0.01 * (grid + 1) ** 2
    coef = np.array([1.0 + 4.0 * a, -a, -a, -a, -a, -1.0]) / (1.0 + 4.0 * a)
    q = 10.0 ** rng.uniform(0.0, 2.0, cols.shape[0])
    keys, vals = [np.arange(n, dtype=np.int64) * (n + 1)], [rng.uniform(1.0, 3.0, n)]
    for i in range(6):
        for j in range(6):
            ci, cj = cols[:, i].astype(np.int64), cols[:, j].astype(np.int64)
            use = (ci >= 0) & (cj >= 0) & (ci >= cj)
            keys.append(ci[use] * n + cj[use])
            vals.append((q * coef[i] * coef[j])[use])
    key, at = np.unique(np.concatenate(keys), return_inverse=True)
    val = np.bincount(at, weights=np.concatenate(vals), minlength=key.size)
    return key // n, key % n, val


def _factor_inputs(case, seed):
    rng = np.random.default_rng(seed)
    r, c, v = _plate_matrix(case["size"], case["horizon"], rng)
    n = case["horizon"] * (case["size"] ** 2 + 16)
    return n, r, c, v, rng.normal(0.0, 1.0, n)


# ---- the interface ---------------------------------------------------------------------------------------------------
def prepare(case, seed):
    rng = np.random.default_rng(seed)
    path, model, size, horizon = case["path"], case["model"], case["size"], case["horizon"]
    periods = case.get("periods", 1)
    if path == "factor":
        p = N.Problem(_structure(model, size, horizon))
        p.analyze()
        n, r, c, v, b = _factor_inputs(case, seed)
        pat = p.patterns()
        want = pat["k_rows"].astype(np.int64) * n + pat["k_cols"]
        have = r * n + c
        at = np.minimum(np.searchsorted(have, want), have.size - 1)
        return dict(path=path, p=p, kv=np.where(have[at] == want, v[at], 0.0), b=b)
    if path == "batch":   # one worker per host thread: the analyses are independent
        uneven = np.random.default_rng([size, horizon, case["count"]])
        shapes = [(int(uneven.integers(size // 3, size + 1)), int(uneven.integers(horizon // 3, horizon + 1)),
                   float(rng.uniform(2.0, 3.0))) for _ in range(case["count"])]
        inputs = [_inputs(model, s, h, periods + 1, rng) for s, h, _ in shapes]
        problems = [N.Problem(_structure(model, s, h, a)) for s, h, a in shapes]
        with ThreadPoolExecutor(8) as ex:
            list(ex.map(lambda p: p.analyze(), problems))
        for p, i in zip(problems, inputs):
            p.set_parameters(**i[-1])
        batch = N.Batch(problems)
        batch.solve(warm=False)
        return dict(path=path, problems=problems, batch=batch, inputs=inputs, periods=periods, options=_options())
    alpha = float(rng.uniform(2.0, 3.0))
    inputs = _inputs(model, size, horizon, periods + 1, rng)
    p = _solved(_structure(model, size, horizon, alpha), inputs[-1])
    s = dict(path=path, p=p, inputs=inputs[:-1], options=_options(case.get("kkt", "lifted")), periods=periods)
    if path == "loop":
        p.solve(warm=True, options=s["options"])
        dev = torch.device("cuda")
        s["traj"] = torch.tensor(np.stack([i["traj"] for i in inputs[:-1]]), device=dev)
        s["noise"] = torch.tensor(rng.normal(0.0, 0.01, (periods, p.nx)), device=dev)
        s["u"] = torch.empty(periods, p.nu, dtype=torch.float64, device=dev)
        s["x"] = torch.empty(periods, p.nx, dtype=torch.float64, device=dev)
    if path == "gradient":
        dev = torch.device("cuda")
        put = lambda a: None if a is None else torch.tensor(a, device=dev)  # noqa: E731
        s["inputs"] = [{k: put(v) for k, v in i.items()} for i in inputs[:-1]]
        s["weight"] = torch.tensor(rng.normal(0.0, 1.0, p.nu), device=dev)
    return s


def run(state):
    path = state["path"]
    if path == "factor":
        p = state["p"]
        ok, _ = p.factor(state["kv"], want_l=False)
        return int(ok), p.linear_solve(state["b"])
    out = []
    if path == "resolve":
        p = state["p"]
        for i in state["inputs"]:
            p.set_parameters(**i)
            p.solve(warm=True, options=state["options"])
            out.append(p.first_stage())
        out.append(p.solution()["y"])   # the last predicted trajectory, for the operator's display
    elif path == "jacobian":
        p = state["p"]
        for i in state["inputs"]:
            p.set_parameters(**i)
            p.solve(warm=True, options=state["options"])
            out.append((*p.first_stage(), p.jacobian_u1_x0()[1]))
    elif path == "batch":
        for k in range(state["periods"]):
            for p, i in zip(state["problems"], state["inputs"]):
                p.set_parameters(**i[k])
            state["batch"].solve(warm=True, options=state["options"])
            out.append(np.concatenate([np.concatenate(p.first_stage()) for p in state["problems"]]))
    elif path == "loop":
        p = state["p"]
        stream = torch.cuda.current_stream().cuda_stream
        p.closed_loop_dev(state["periods"], traj=state["traj"].data_ptr(), noise=state["noise"].data_ptr(),
                          u_out=state["u"].data_ptr(), x_out=state["x"].data_ptr(), options=state["options"],
                          stream=stream)
        out.append((state["u"], state["x"]))
    else:
        p = state["p"]
        for i in state["inputs"]:
            leaf = {k: None if v is None else v.detach().requires_grad_(k != "traj") for k, v in i.items()}
            u1, f = NMPCSolve.apply(p, leaf["x0"], leaf["setpoint"], leaf["traj"], leaf["u_prev"], True,
                                    state["options"])
            ((state["weight"] * u1).sum() + f).backward()
            out.append([u1.detach(), f.detach()] + [t.grad for t in leaf.values() if t is not None and t.requires_grad])
    return out


@lru_cache(maxsize=None)
def _counts(model, size, horizon):
    """Unknowns, lower entries of the condensed matrix and of its factor, and the factorization's operations, under the
    framework's fill-reducing ordering."""
    p = N.Problem(_structure(model, size, horizon))
    p.analyze()
    z = p.symbolic_sizes()
    got = (p.n, p.nnz_k, z["nnz_l"], z["flops"])
    p.close()
    return got


def work(case):
    """Per Newton iteration the matrix is read, the factor written and read twice (forward and back), its operations
    done; a gradient or a gain adds a factorization at the solution and three solves (one and two refinements)."""
    n, nk, nl, fl = _counts(case["model"], case["size"], case["horizon"])
    if case["path"] == "factor":
        return dict(bytes=8.0 * (nk + 3 * nl + 2 * n), flops=fl + 4.0 * nl)
    factors = solves = NEWTON
    seeds = 0
    if case["path"] in ("gradient", "jacobian"):
        factors += 1
        seeds = 1 if case["path"] == "gradient" else 16
    times = case["periods"] * (case["count"] * 0.35 if case["path"] == "batch" else 1.0)
    return dict(bytes=times * 8.0 * (factors * (nk + nl) + 2 * solves * nl + (6 * nl if seeds else 0) + 10 * n),
                flops=times * (factors * fl + 4.0 * nl * (solves + 3 * seeds)))


def exact(case, seed):
    """The linear systems by conjugate gradients in 64 bits on the matrix itself; None for the solves."""
    if case["path"] != "factor":
        return None
    n, r, c, v, b = _factor_inputs(case, seed)
    off = r != c
    i = torch.tensor(np.concatenate([np.stack([r, c]), np.stack([c[off], r[off]])], 1))
    a = torch.sparse_coo_tensor(i, torch.tensor(np.concatenate([v, v[off]])), (n, n)).coalesce().to_sparse_csr()
    d = torch.tensor(np.bincount(r[~off], weights=v[~off], minlength=n))
    b = torch.tensor(b)
    x, res = torch.zeros_like(b), b.clone()
    z = res / d
    p, rz = z.clone(), torch.dot(res, z)
    stop = 1e-15 * float(b.norm())
    for _ in range(3000):
        ap = a @ p
        alpha = rz / torch.dot(p, ap)
        x += alpha * p
        res -= alpha * ap
        if float(res.norm()) <= stop:
            break
        z = res / d
        new = torch.dot(res, z)
        p = z + (new / rz) * p
        rz = new
    return None, x.numpy()
