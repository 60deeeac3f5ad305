"""The work that programs give this framework, as cases that can be timed.

A case is a dict of plain values.  `listed()` gives the named ones, `draw(rng)` one more of
the same ranges.  `prepare` builds what a program holds before the call (the mesh's
hierarchy on the GPU, seeded loads and states), `run` is one pass through the public entry
points, `work` the bytes and operations that the pass cannot do without, and `exact` the
same outputs computed with NumPy in FP64 where that is quick.

Kinds of work (`do`):
  solve   Hierarchy.solve from x = 0: the boundary-value problems of the paper's Sec. 2 and 5
  vcycle  Hierarchy.vcycle from a given iterate: the V-cycle as another program's preconditioner
  steps   the V-cycle's steps on the finest level one at a time (a program with its own cycle)
  batch   Batch.solve: many uneven problems with 1 or 8 right-hand sides each
  time    TimeStepper.run: backward-Euler steps of the nonstationary problem (Sec. 5.1)
  ns      PressureCorrection.run: time steps of the explicit pressure correction (Sec. 5.3)
  asm     Assembly.values: numeric assembly on the GPU for new coefficients
"""
import functools
import math

import numpy as np
import torch

import workloads as W
from paper_2405_05047_amd import gen, mg

# the coarse level is the finest one with at most this many unknowns: the dense coarse solve
# of the benchmark configurations (1,089 to 2,187 unknowns)
COARSE_DOFS = 2500


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest call: the 33 x 33 Poisson model problem over its whole 5-level hierarchy
        # down to one free node, MG iteration to 1e-10; a teaching example, a unit test, or one
        # of many small independent subproblems: launches and latency
        dict(name="poisson2d_33_solve", do="solve", mesh="poisson2d", coarse=2, rounds=4, prec="fp64", whole=True),
        # the 2D transport-diffusion workload: 1.0M unknowns on an adaptive annulus mesh with
        # hanging nodes, FGMRES(10) + V(2,2)
        dict(name="td2d_annulus_1m_solve", do="solve", mesh="td2d", uniform=2, band=6, delta=W.C2_DELTA, prec="fp64"),
        # the headline workload: 129^3 nodes of linear elasticity, 6.4M unknowns, FP64
        dict(name="elast3d_129_solve", do="solve", mesh="elast3d", coarse=2, rounds=6, prec="fp64"),
        # adaptive 3D elasticity (683,741 nodes refined towards a face, a fifth of them hanging)
        # with the 16-bit operator values in an FP32 cycle
        dict(name="elast3d_face6_fp16_solve", do="solve", mesh="face", level=6, prec="fp16"),
        # the linearised flow step, 65^3 nodes with 4 components and a convection field that
        # varies from cell to cell, FP64
        dict(name="oseen3d_65_solve", do="solve", mesh="oseen3d", coarse=2, rounds=5, prec="fp64"),
        # the same flow step at a quarter of a million unknowns in the FP32 cycle
        dict(name="oseen3d_41_fp32_solve", do="solve", mesh="oseen3d", coarse=5, rounds=3, prec="fp32"),
        # a V-cycle on the caller's iterate, mid-size adaptive 2D mesh, FP32 cycle: the
        # preconditioner of another Krylov method
        dict(name="td2d_70k_vcycle_fp32", do="vcycle", mesh="td2d", uniform=2, band=4, delta=W.C2_DELTA, prec="fp32"),
        # the steps of the cycle one by one on 65^3 elasticity (0.8M unknowns)
        dict(name="elast3d_65_steps", do="steps", mesh="elast3d", coarse=2, rounds=5, prec="fp64"),
        # parameter study: 16 uneven transport-diffusion problems, 8 right-hand sides each
        dict(name="batch16x8_solve", do="batch", problems=16, nrhs=8, levels=8, prec="fp64", first=1000),
        # the nonstationary problem on the paper's 1,050,625-unknown mesh, 10 time steps
        dict(name="time_1m_10_steps", do="time", n=10, steps=10),
        # the driven cavity on the graded 32 x 32 x 64 mesh, 2 time steps (1.6M velocity and 71k
        # pressure unknowns)
        dict(name="ns_cavity_32_2_steps", do="ns", cells=32, steps=2),
        # numeric assembly of the face-refined elasticity operator for new material constants
        dict(name="asm_elast3d_face6", do="asm", mesh="face", level=6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_mesh(rng, small):
    """One mesh recipe with its operator; `small` leaves out the largest third."""
    mesh = rng.choice(["poisson2d", "td2d", "td2d", "elast3d", "face", "edge", "vertex", "oseen3d"])
    if mesh == "poisson2d":
        return dict(mesh=mesh, coarse=rng.randint(1, 7), rounds=rng.randint(4, 6 if small else 7))
    if mesh == "td2d":
        return dict(mesh=mesh, uniform=rng.randint(1, 3), band=rng.randint(2, 4 if small else 5),
                    delta=round(rng.uniform(0.02, 0.1), 4))
    if mesh == "elast3d":
        return dict(mesh=mesh, coarse=rng.choice([2, 3, 4, 5, 6]), rounds=rng.randint(2, 3 if small else 4))
    if mesh == "oseen3d":
        return dict(mesh=mesh, coarse=rng.choice([2, 3, 4, 5]), rounds=rng.randint(2, 3))
    top = {"face": 5, "edge": 7, "vertex": 8}[mesh]
    return dict(mesh=mesh, level=rng.randint(3, top - 1 if small else top))


def draw(rng):
    do = rng.choice(["solve"] * 5 + ["vcycle", "vcycle", "steps", "batch", "time", "ns", "asm"])
    if do == "batch":
        return dict(do=do, problems=_log_int(rng, 2, 16), nrhs=rng.choice([1, 8]), levels=rng.randint(5, 7),
                    prec=rng.choice(["fp64", "fp32", "fp16"]), first=rng.randint(1000, 1900))
    if do == "time":
        return dict(do=do, n=rng.randint(6, 10), steps=rng.randint(3, 12))
    if do == "ns":
        return dict(do=do, cells=rng.choice([8, 12, 16, 20, 24, 28]), steps=rng.randint(1, 3))
    if do == "asm":
        while True:
            m = _draw_mesh(rng, False)
            if m["mesh"] != "oseen3d":
                return dict(do=do, **m)
    case = dict(do=do, **_draw_mesh(rng, do != "solve"))
    case["prec"] = rng.choice(["fp64", "fp64", "fp32", "fp16", "bf16", "fp64dict"])
    if do == "solve":
        case["cheb"] = case["mesh"] in ("elast3d", "face", "edge", "vertex") and rng.random() < 0.4
    return case


# ---------------------------------------------------------------- host side of a case
def _workload(case):
    m = case["mesh"]
    if m == "poisson2d":
        c = case["coarse"]
        return W.c1_poisson(case["rounds"]).with_(coarse=(c, c), h0=1.0 / c)
    if m == "td2d":
        return W.c2_td(case["band"], case["delta"], case["uniform"])
    if m == "elast3d":
        c = case["coarse"]
        return W.c3_elasticity(case["rounds"]).with_(coarse=(c, c, c), h0=1.0 / c)
    if m == "oseen3d":
        c = case["coarse"]
        return W.c4_oseen(case["rounds"]).with_(coarse=(c, c, c), h0=1.0 / c)
    return W.c3_adaptive(m, case["level"])


@functools.lru_cache(maxsize=2)
def _problem(wl, time_ops, whole):
    """The host hierarchy, from its coarse level up (every seed of a case shares the mesh)."""
    p = gen.build(wl, time_ops=time_ops)
    if not whole:
        fits = [l for l, lv in enumerate(p.levels) if lv.n * lv.block <= COARSE_DOFS]
        p.levels = p.levels[min(max(fits, default=0), len(p.levels) - 2):]
        p.levels[0].p_rowptr = p.levels[0].p_col = p.levels[0].p_val = None
        p.levels[0].p_cols = 0
    return p


@functools.lru_cache(maxsize=1)
def _batch(problems, nrhs, levels, first):
    wls = W.batch_problems(problems, first, levels)
    return wls, [gen.build(wl, nrhs) for wl in wls]


@functools.lru_cache(maxsize=1)
def _cavity(cells):
    n_levels = 1
    while cells % (1 << n_levels) == 0 and n_levels < 5 and _cavity_nodes(cells >> (n_levels - 1)) > COARSE_DOFS:
        n_levels += 1
    return gen.build_ns((cells, cells, 2 * cells), n_levels=n_levels)


def _cavity_nodes(c):
    return (c + 1) * (c + 1) * (2 * c + 1)


_PRESSURE = W.Workload(name="pressure", dim=3, coarse=(1, 1, 1), h0=1.0, rounds=(), pde=W.PDE_POISSON, block=1,
                       omega=0.8, nu1=2, nu2=2, outer=W.OUTER_FGMRES, gmres_m=10, rtol=1e-8, maxit=400,
                       smoother=W.SMOOTH_CHEBYSHEV)


def _field(rng, X, modes=4):
    """A smooth seeded function on the points X (rows): a few Fourier modes."""
    f = np.full(len(X), rng.uniform(-1.0, 1.0))
    for _ in range(modes):
        k = rng.integers(0, 4, X.shape[1]).astype(np.float64)
        f += rng.uniform(-1.0, 1.0) * np.sin(2.0 * np.pi * (X @ k) + rng.uniform(0.0, 2.0 * np.pi))
    return f


def _points(lv, dim):
    X = lv.lattice[:, :dim].astype(np.float64)
    return X / X.max()


def _load(case, p, rng):
    """A seeded smooth body load on the finest mesh: nodal volumes times smooth functions,
    zero on the constrained unknowns."""
    top, dim = p.finest, p.wl.dim
    corners = top.cells.shape[1]
    vol = np.bincount(top.cells.ravel(), np.repeat(top.cell_size ** dim / corners, corners), top.n)
    X = _points(top, dim)
    b = np.stack([vol * _field(rng, X) for _ in range(top.block)], axis=1)
    b[top.mask != 0] = 0.0
    return b.reshape(-1)


def _vector(case, lv, dim, rng, rough):
    """A seeded iterate: smooth plus a rough part, zero on the constrained unknowns."""
    X = _points(lv, dim)
    v = np.stack([_field(rng, X) for _ in range(lv.block)], axis=1)
    v += rough * rng.standard_normal(v.shape)
    v[lv.mask != 0] = 0.0
    return v.reshape(-1)


def _config(case, wl):
    over = {"smoother": W.SMOOTH_CHEBYSHEV} if case.get("cheb") else {}
    return mg.config_from(wl, precision=case["prec"], **over)


def _hierarchy_inputs(case, seed):
    """Host inputs of a solve, vcycle or steps case: the problem and its seeded vectors."""
    p = _problem(_workload(case), False, bool(case.get("whole")))
    rng = np.random.default_rng(seed)
    v = {"b": _load(case, p, rng)}
    if case["do"] != "solve":
        v["x"] = _vector(case, p.finest, p.wl.dim, rng, 0.1)
    if case["do"] == "steps":
        v["y"] = _vector(case, p.levels[-2], p.wl.dim, rng, 0.1)
    return p, v


def _coefficients(case, wl, seed):
    rng = np.random.default_rng(seed)
    c = mg.asm_coef(wl)
    if wl.pde == W.PDE_ELASTICITY:
        c.lam, c.mu = rng.uniform(0.5, 2.0), rng.uniform(0.3, 1.0)
    else:
        c.eps = 10.0 ** rng.uniform(-4.0, -1.0)
        t = rng.uniform(0.0, 2.0 * math.pi)
        c.bvec[0], c.bvec[1] = math.cos(t), math.sin(t)
    c.mass_coef = rng.uniform(0.5, 50.0)
    return c


def prepare(case, seed):
    do = case["do"]
    s = {"do": do, "case": case}
    if do in ("solve", "vcycle", "steps"):
        p, v = _hierarchy_inputs(case, seed)
        s["h"] = mg.Hierarchy(p.levels, _config(case, p.wl))
        real = torch.float64 if do != "steps" or s["h"].cycle_fp64 else torch.float32
        s.update({k: torch.from_numpy(a).cuda().to(real) for k, a in v.items()})
    elif do == "batch":
        wls, probs = _batch(case["problems"], case["nrhs"], case["levels"], case["first"])
        s["h"] = mg.Batch([p.levels for p in probs], mg.config_from(wls[0], precision=case["prec"]), nrhs=case["nrhs"])
        rng = np.random.default_rng(seed)
        b = []
        for p in probs:
            q = np.asarray(p.b, np.float64).reshape(p.finest.n, case["nrhs"])
            b.append((q * _field(rng, _points(p.finest, 2))[:, None]).reshape(-1))
        s["b"] = torch.from_numpy(np.concatenate(b)).cuda()
    elif do == "time":
        n, steps = case["n"], case["steps"]
        wl = W.td_time(n)
        p = _problem(wl, True, False)
        s["h"] = mg.Hierarchy(p.levels, mg.config_from(wl))
        s["ts"] = mg.TimeStepper(s["h"], p.time, wl.dt)
        t0 = float(np.random.default_rng(seed).uniform(0.0, 1.5))
        X, Y = p.time.coords[:, 0], p.time.coords[:, 1]
        ts = [t0 + k * wl.dt for k in range(1, steps + 1)]
        s["F"] = torch.from_numpy(np.stack([W.td_source(t, X, Y) for t in ts])).cuda()
        s["G"] = torch.from_numpy(np.stack([W.td_exact(t, X, Y)[p.time.g_idx] for t in ts])).cuda()
        th = W.td_exact(t0, X, Y)
        s["theta"] = torch.from_numpy(th).cuda()
        s["x"] = torch.from_numpy(np.where(p.finest.mask.ravel() != 0, 0.0, th)).cuda()
    elif do == "ns":
        prob = _cavity(case["cells"])
        s["h"] = mg.Hierarchy(prob.levels, mg.config_from(_PRESSURE))
        s["pc"] = mg.PressureCorrection(prob, s["h"], 1e-3, 1e-4)
        # the cavity some time after its start: a small smooth flow inside, the moving wall
        rng = np.random.default_rng(seed)
        X = prob.coords_v / prob.coords_v.max(axis=0)
        u = 0.1 * np.prod(X * (1.0 - X), axis=1)[:, None] * np.stack([_field(rng, X) for _ in range(3)], axis=1)
        s["u"] = torch.from_numpy(np.where(prob.dir_mask != 0, prob.dir_val, u)).cuda()
        s["p"] = torch.zeros(prob.n_p, dtype=torch.float64, device="cuda")
    elif do == "asm":
        p = _problem(_workload(case), False, False)
        top = p.finest
        s["a"] = mg.Assembly(top, p.wl.dim)
        s["coef"] = _coefficients(case, p.wl, seed)
        s["val"] = torch.empty(top.nnzb * top.block ** 2, dtype=torch.float64, device="cuda")
    return s


def run(s):
    do = s["do"]
    if do == "solve":
        x = torch.zeros_like(s["b"])
        s["h"].solve(s["b"], x)
        return x
    if do == "vcycle":
        x = s["x"].clone()
        s["h"].vcycle(s["b"], x, x_is_zero=False)
        return x
    if do == "steps":
        h, b, x, L = s["h"], s["b"], s["x"], s["h"].n_levels - 1
        first, r, sw, cor = torch.empty_like(x), torch.empty_like(x), torch.empty_like(x), x.clone()
        d = torch.empty_like(s["y"])
        h.sweep0(L, b, first)
        h.sweep(L, b, first, sw)
        h.defect(L, b, x, r, masked=True)
        h.restrict(L, r, d)
        h.prolong(L, s["y"], cor)
        return {"first": first, "sweep": sw, "defect": r, "restricted": d, "corrected": cor}
    if do == "batch":
        x = torch.zeros_like(s["b"])
        s["h"].solve(s["b"], x)
        return x
    if do == "time":
        th, x = s["theta"].clone(), s["x"].clone()
        s["ts"].run(th, s["F"], s["G"], x)
        return {"theta": th, "x": x}
    if do == "ns":
        u, p, q = s["u"].clone(), s["p"].clone(), s["p"].clone()
        s["pc"].run(s["case"]["steps"], u, p, q)
        return {"u": u, "p": p}
    s["a"].values(s["coef"], s["val"])
    return s["val"]


# ---------------------------------------------------------------- work and exact values
_VALUE = {"fp64": 8, "fp64dict": 8, "fp32": 4, "fp16": 2, "bf16": 2}


def _operator_bytes(lv, value):
    """The stored operator as given (values, column indices) and the level's transfer."""
    p = 0 if lv.p_col is None else 12 * len(lv.p_col)
    return lv.nnzb * (lv.block ** 2 * value + 4) + p


def _cycle_flops(levels):
    """Multiply-adds of one V(2,2): four sweeps' products and one defect per level."""
    return sum(2.0 * 5 * lv.nnzb * lv.block ** 2 for lv in levels)


def work(case):
    do = case["do"]
    if do in ("solve", "vcycle", "steps"):
        p = _problem(_workload(case), False, bool(case.get("whole")))
        top, value = p.finest, _VALUE[case["prec"]]
        N = top.n * top.block
        if do == "steps":
            own = _operator_bytes(top, value)
            return {"bytes": own + 9.0 * N * 8, "flops": 2.0 * 2 * top.nnzb * top.block ** 2}
        every = sum(_operator_bytes(lv, value) for lv in p.levels)
        if do == "vcycle":
            return {"bytes": every + 3.0 * N * 8, "flops": _cycle_flops(p.levels)}
        # a dozen cycles reach 1e-8 on these problems
        return {"bytes": every + 2.0 * N * 8, "flops": 12 * (_cycle_flops(p.levels) + 2.0 * top.nnzb * top.block ** 2)}
    if do == "batch":
        _, probs = _batch(case["problems"], case["nrhs"], case["levels"], case["first"])
        value, nrhs = _VALUE[case["prec"]], case["nrhs"]
        every = sum(_operator_bytes(lv, value) for p in probs for lv in p.levels)
        N = sum(p.finest.n for p in probs) * nrhs
        return {"bytes": every + 2.0 * N * 8, "flops": 12.0 * nrhs * sum(_cycle_flops(p.levels) for p in probs)}
    if do == "time":
        p = _problem(W.td_time(case["n"]), True, False)
        every = sum(_operator_bytes(lv, 8) for lv in p.levels)
        N, steps = p.finest.n, case["steps"]
        return {"bytes": every + steps * 8.0 * N + 4.0 * N * 8, "flops": steps * 3 * _cycle_flops(p.levels)}
    if do == "ns":
        prob = _cavity(case["cells"])
        own = len(prob.V_col) * (4 * 8 + 4) + (len(prob.G_col) + len(prob.D_col)) * (3 * 8 + 4)
        every = sum(_operator_bytes(lv, 8) for lv in prob.levels)
        steps = case["steps"]
        return {"bytes": own + every + 2.0 * (3 * prob.n_v + 2 * prob.n_p) * 8,
                "flops": steps * (2.0 * 15 * len(prob.V_col) + 40 * _cycle_flops(prob.levels))}
    p = _problem(_workload(case), False, False)
    top = p.finest
    return {"bytes": top.nnzb * (top.block ** 2 * 8 + 4.0) + top.cells.size * 4.0, "flops": 8.0 * top.nnzb * top.block ** 2}


def _apply(lv, x):
    """A x for the level's blocks, FP64."""
    y = np.einsum("kij,kj->ki", lv.val, x.reshape(lv.n, lv.block)[lv.col])
    return np.add.reduceat(y, lv.rowptr[:-1], axis=0).reshape(-1)


def _diagonal_inverse(lv):
    rows = np.repeat(np.arange(lv.n), np.diff(lv.rowptr))
    return np.linalg.inv(lv.val[rows == lv.col])


def _sweep(lv, S, omega, b, x):
    r = (b - _apply(lv, x)).reshape(lv.n, lv.block, 1)
    return x + omega * (S @ r).reshape(-1)


def _transfer(lv, lc, y, transpose):
    """P y, or P^T y, with the masks of both levels applied."""
    rows = np.repeat(np.arange(lv.n), np.diff(lv.p_rowptr))
    fine, coarse = lv.mask == 0, lc.mask == 0
    src, dst = (rows, lv.p_col) if transpose else (lv.p_col, rows)
    m_in, m_out = (fine, coarse) if transpose else (coarse, fine)
    v = y.reshape(-1, lv.block) * m_in
    out = np.stack([np.bincount(dst, lv.p_val * v[src, c], len(m_out)) for c in range(lv.block)], axis=1)
    return (out * m_out).reshape(-1)


def _dense(lv):
    A = np.zeros((lv.n, lv.block, lv.n, lv.block))
    rows = np.repeat(np.arange(lv.n), np.diff(lv.rowptr))
    A[rows, :, lv.col, :] = lv.val
    return A.reshape(lv.n * lv.block, -1)


def _cycle(levels, l, wl, b, x):
    if l == 0:
        return np.linalg.solve(_dense(levels[0]), b)
    lv, lc = levels[l], levels[l - 1]
    S = _diagonal_inverse(lv)
    for _ in range(wl.nu1):
        x = _sweep(lv, S, wl.omega, b, x)
    d = _transfer(lv, lc, b - _apply(lv, x), True)
    x = x + _transfer(lv, lc, _cycle(levels, l - 1, wl, d, np.zeros_like(d)), False)
    for _ in range(wl.nu2):
        x = _sweep(lv, S, wl.omega, b, x)
    return x


def exact(case, seed):
    if case["do"] not in ("solve", "vcycle", "steps"):
        return None
    p, v = _hierarchy_inputs(case, seed)
    top = p.finest
    N = top.n * top.block
    if case["do"] == "solve":
        return np.linalg.solve(_dense(top), v["b"]) if N <= 5000 else None
    if top.nnzb * top.block ** 2 > 8e7:
        return None
    if case["do"] == "vcycle":
        return _cycle(p.levels, len(p.levels) - 1, p.wl, v["b"], v["x"])
    lc, S, b = p.levels[-2], _diagonal_inverse(top), v["b"]
    first = _sweep(top, S, p.wl.omega, b, np.zeros(N))
    r = b - _apply(top, v["x"])
    r[top.mask.ravel() != 0] = 0.0
    return {"first": first, "sweep": _sweep(top, S, p.wl.omega, b, first), "defect": r,
            "restricted": _transfer(top, lc, r, True), "corrected": v["x"] + _transfer(top, lc, v["y"], False)}
