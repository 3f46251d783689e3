"""The work that programs have this framework do, as cases that can be timed.

A case is one call of a public entry point on a plan that the program keeps:
the operator K~ itself (``matvec``: products for sampling, log-likelihood
estimates, residuals), conjugate gradients on it (``steps``: a fixed number of
iterations, the unit that long solves are made of; ``solve`` and ``refined``:
whole solves to a tolerance), many right-hand sides at once (``multi``) and
predictions at new points (``mean``).  Dimensions, smoothness, length scales,
sizes and tolerances are those of the generators in
``paper_2407_03608_amd/inputs.py`` and of the tests: d = 1..3, from the smallest
problems, where launches count, to the largest that the benchmark runs, in
both precisions of the grids.
"""
import math

import torch

from paper_2407_03608_amd import gp

_PREC = {"fp64": gp.GP_FP64, "fp32": gp.GP_FP32_BULK}


def _case(kind, d, n, nu, tol, precision, l_min, l_max, eta, **more):
    return dict({"kind": kind, "d": d, "n": n, "nu": nu, "tol": tol, "precision": precision,
                 "l_min": l_min, "l_max": l_max, "eta": eta, "points": "uniform"}, **more)


def listed():
    return [
        # one product of a small time-series model: bound by launches
        dict(_case("matvec", 1, 2000, 1.5, 1e-8, "fp64", 0.02, 0.08, 0.1), name="matvec_1d_2k_fp64"),
        # the whole fit of that model
        dict(_case("solve", 1, 2000, 1.5, 1e-8, "fp64", 0.02, 0.08, 0.1, cg_tol=1e-8), name="solve_1d_2k_fp64"),
        # a long rough time series: the largest 1-D grid (2^20 points)
        dict(_case("matvec", 1, 163_900, 0.5, 1e-4, "fp32", 0.03, 0.06, 0.1), name="matvec_1d_164k_fp32"),
        # few points of a rough field: the grids cost far more than the points (paired: the
        # fp32 operator of a mixed-precision solve, on the Fourier box of the fp64 one)
        dict(_case("matvec", 2, 20_447, 0.5, 1e-4, "fp32", 0.03, 0.06, 0.1, paired=True), name="matvec_2d_20k_fp32"),
        # an ordinary smooth spatial model
        dict(_case("matvec", 2, 100_000, 2.5, 1e-8, "fp64", 0.03, 0.06, 0.3), name="matvec_2d_100k_fp64"),
        # the headline: iterations of the million-point rough field, in both precisions
        dict(_case("steps", 2, 1_000_000, 0.5, 1e-8, "fp64", 0.02, 0.04, 0.05, iters=5), name="steps_2d_1m_fp64"),
        dict(_case("steps", 2, 1_000_000, 0.5, 1e-4, "fp32", 0.02, 0.04, 0.05, iters=5, paired=True), name="steps_2d_1m_fp32"),
        # a solve with fp32 grids inside fp64 refinement, as the server makes it
        dict(_case("refined", 2, 30_057, 2.5, 1e-8, "fp64", 0.04, 0.08, 0.2, cg_tol=1e-6), name="refined_2d_30k"),
        # iterations of block CG for 16 right-hand sides (posterior covariance)
        dict(_case("multi", 2, 100_000, 2.5, 1e-8, "fp64", 0.03, 0.06, 0.3, iters=4, rhs=16), name="block_2d_100k_fp64"),
        # the posterior mean on a raster of new points
        dict(_case("mean", 2, 100_000, 2.5, 1e-8, "fp64", 0.03, 0.06, 0.3, targets=50_001), name="mean_2d_100k_fp64"),
        # a volume in full precision
        dict(_case("matvec", 3, 200_000, 2.5, 1e-6, "fp64", 0.1, 0.2, 0.1), name="matvec_3d_200k_fp64"),
        # ten million clustered points of a volume
        dict(_case("matvec", 3, 10_000_000, 2.5, 1e-4, "fp32", 0.03, 0.047, 0.1, points="mixture"), name="matvec_3d_10m_fp32"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case: kind, dimension, precision and smoothness as above, the
    number of points over its whole range on a logarithmic scale."""
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["matvec", "matvec", "matvec", "steps", "solve", "refined", "multi", "mean"])
        d = {"solve": 1, "refined": 2}.get(kind) or rng.choice([1, 2, 2, 3])
        precision = "fp64" if kind in ("solve", "refined") else rng.choice(["fp64", "fp32"])
        top = {1: 5e5, 2: 1e6, 3: 1e7 if precision == "fp32" else 5e5}[d]
        lo = 300.0
        if kind == "solve":
            top = 4e3
        elif kind == "refined":
            lo, top = 5e3, 4e4
        elif kind in ("multi", "mean"):
            lo, top = 1e3, 2e5
        n = int(_log_uniform(rng, lo, top))
        l0 = _log_uniform(rng, *{1: (0.02, 0.2), 2: (0.02, 0.2), 3: (0.03, 0.2)}[d])
        if kind == "solve":
            l0 = max(l0, 0.03)
        nu = 2.5 if kind == "refined" or d == 3 else rng.choice([0.5, 1.5, 2.5])
        if kind == "solve":
            nu = rng.choice([1.5, 2.5])
        if kind == "refined":
            l0 = max(l0, 0.04)
        l1 = l0 if rng.random() < 0.15 else l0 * rng.uniform(1.2, 2.5)
        tol = 1e-4 if precision == "fp32" else (1e-6 if d == 3 else 1e-8)
        eta = rng.uniform(0.2, 0.4) if kind == "refined" else rng.uniform(0.05, 0.3)
        c = _case(kind, d, n, nu, tol, precision, round(l0, 4), round(l1, 4), round(eta, 3))
        if d == 3 and rng.random() < 0.5:
            c["points"] = "mixture"
        if d == 2 and precision == "fp32" and rng.random() < 0.5:
            c["paired"] = True
        if kind in ("solve", "refined"):
            c["cg_tol"] = 1e-8 if kind == "solve" else 1e-6
        if kind in ("steps", "multi"):
            c["iters"] = rng.randint(2, 5)
        if kind == "multi":
            c["rhs"] = rng.randint(2, 16)
        if kind == "mean":
            c["targets"] = int(_log_uniform(rng, 1, 1e5))
        r = _rules(c)
        grid = (2 * r["M"] + 1) ** d * (r["n_sigma"] + 1) * c.get("rhs", 1)
        if d == 3 and r["M"] > 230:
            continue  # such a grid does not fit beside others
        if grid <= 1.5e9 and work(c)["flops"] <= most:
            return c


# ------------------------------------------------------------------- inputs --

def _field(x, phase):
    """A smooth periodic function of the points, in [-1, 1]."""
    return torch.sin(2 * math.pi * x + phase).mean(dim=1)


def _inputs(case, seed):
    """Points, scales, observations and what else the call takes (CPU, fp64)."""
    g = torch.Generator().manual_seed(1_000_003 * seed + 17)
    rand = lambda *s: torch.rand(*s, generator=g, dtype=torch.float64)  # noqa: E731
    randn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64)  # noqa: E731
    d, n = case["d"], case["n"]
    phase = 2 * math.pi * rand(2, d)

    def points(m):
        if case["points"] == "uniform":
            return rand(m, d)
        centres = 0.2 + 0.6 * rand(8, d)
        which = torch.randint(0, 8, (m,), generator=g)
        return (centres[which] + 0.1 * randn(m, d)).clamp_(0.0, 1.0)

    def scales(x):
        sigma = 1.0 + 0.4 * _field(x, phase[0])
        l = case["l_min"] + (case["l_max"] - case["l_min"]) * 0.5 * (1.0 + _field(x, phase[1]))
        return sigma, l

    x = points(n)
    sigma, l = scales(x)
    y = torch.sin(8.0 * x).mean(dim=1) + case["eta"] * randn(n)
    out = {"x": x, "sigma": sigma, "l": l, "y": y}
    if case["kind"] in ("matvec", "mean"):
        out["alpha"] = randn(n)
    if case["kind"] == "multi":
        out["Y"] = randn(case["rhs"], n)
    if case["kind"] == "mean":
        t = case["targets"]
        # new points inside the box of the data, with scales of the data's range
        i, j = (torch.randint(0, n, (t,), generator=g) for _ in range(2))
        xt = 0.5 * (x[i] + x[j])
        st, _ = scales(xt)
        out.update(xt=xt, st=st, lt=l[j])
    return out




def _box(case):
    """Fourier box of a plan that is used beside a fp64 one (paired), else the plan's own."""
    if not case.get("paired"):
        return {}
    r = gp.plan_rules(case["d"], case["nu"], 1e-8, case["l_min"], case["l_max"], 1.0)
    return {"dw": r["dw"], "M": r["M"]}


def prepare(case, seed):
    dev = {k: v.to("cuda") for k, v in _inputs(case, seed).items()}
    args = (dev["x"], dev["sigma"], dev["l"], case["nu"], case["eta"])
    state = {"case": case, "in": dev}
    state["plan"] = gp.Plan(*args, case["tol"], precision=_PREC[case["precision"]], **_box(case))
    if case["kind"] == "refined":
        info = state["plan"].info()
        state["inner"] = gp.Plan(*args, 1e-4, precision=gp.GP_FP32_BULK, dw=info["dw"], M=info["M"])
    return state


def run(state):
    case, plan, t = state["case"], state["plan"], state["in"]
    kind = case["kind"]
    if kind == "matvec":
        return plan.matvec(t["alpha"], add_noise=True)
    if kind == "steps":
        return plan.cg_solve(t["y"], tol=1e-14, max_iter=case["iters"])[0]
    if kind == "solve":
        return plan.cg_solve(t["y"], tol=case["cg_tol"], max_iter=20000)[0]
    if kind == "refined":
        return gp.cg_solve_refined(state["inner"], plan, t["y"], tol=case["cg_tol"], inner_tol=3e-3)[0]
    if kind == "multi":
        return plan.cg_solve_multi(t["Y"], tol=1e-14, max_iter=case["iters"], block=True)[0]
    return plan.posterior_mean(t["alpha"], t["xt"], t["st"], t["lt"])


# --------------------------------------------------------------- yardsticks --

def _rules(case):
    return gp.plan_rules(case["d"], case["nu"], case["tol"], case["l_min"], case["l_max"], 1.0,
                         _PREC[case["precision"]], **_box(case))


def _products(case):
    """Products with K~ in one pass (solves: a usual number of iterations)."""
    return {"matvec": 1, "mean": 1, "steps": case.get("iters", 0), "solve": 400, "refined": 150,
            "multi": case.get("iters", 0) * case.get("rhs", 0)}[case["kind"]]


def work(case):
    """Bytes: the points, scales, input and output vectors once, and in d >= 2
    the half-transformed grids, which no chip holds, written and read once on
    either side of step 3.  Operations: window sums over the points (w^d cells
    per point and grid, there and back), the transforms of the kept modes and
    step 3, for grids without oversampling."""
    r = _rules(case)
    d, n, s = case["d"], case["n"], 8 if case["precision"] == "fp64" else 4
    if case["kind"] == "refined":
        s = 4
    nk, mc = r["n_sigma"] + 1, 2 * r["M"] + 1
    box = max(1.0, 2 * r["dw"] * mc)  # cells that the points fill, per dimension
    modes = float(mc) ** d
    per = 16.0 * n + (4.0 * nk * box * mc ** (d - 1) * s if d > 1 else 0.0)
    w = math.ceil(math.log10(1 / case["tol"])) + 1
    flops = 4.0 * n * nk * w ** d + 5.0 * nk * modes * math.log2(modes) + 2.0 * nk * nk * modes
    m = _products(case)
    t = case.get("targets", 0)
    return {"bytes": m * per + 8.0 * (n + t) * (d + 3), "flops": m * flops}


def tolerance(case):
    """What other orders of the same sums show (the LDS-atomic spreading, the
    per-bin interpolation and the direct sum over t differ from the default by
    up to 8e-16 with fp64 grids, 2e-7 with fp32 ones), about four times and with
    room for other factorisations of the transforms.  Solves stop at a residual,
    not at a number of iterations, and differ by that residual times the
    system's condition (1e-8 and 7e-8 seen)."""
    if case["kind"] == "refined":
        return {"rel": 2e-6, "max": 1e-4}
    if case["kind"] == "solve":
        return {"rel": 4e-7, "max": 4e-6}
    if case["precision"] == "fp32":
        return {"rel": 1e-6, "max": 2e-5}
    return {"rel": 2e-14, "max": 1e-12}


# -------------------------------------------------------------- exact values --

def _phi(nu, r):
    if nu == 0.5:
        return torch.exp(-r)
    if nu == 1.5:
        s = math.sqrt(3.0) * r
        return (1 + s) * torch.exp(-s)
    s = math.sqrt(5.0) * r
    return (1 + s + s * s / 3) * torch.exp(-s)


def _kernel_rows(nu, xa, sa, la, xb, sb, lb):
    d = xa.shape[1]
    r2 = torch.zeros(xa.shape[0], xb.shape[0], dtype=torch.float64, device=xa.device)
    for k in range(d):
        r2 += (xa[:, k, None] - xb[None, :, k]) ** 2
    l2 = la[:, None] ** 2 + lb[None, :] ** 2
    pre = (2 * la[:, None] * lb[None, :] / l2) ** (0.5 * d)
    return sa[:, None] * sb[None, :] * pre * _phi(nu, torch.sqrt(2 * r2 / l2))


def _cut_off(case):
    """Whether the plan's Fourier box is smaller than its tolerance asks for."""
    return _rules({**case, "paired": False})["m_capped"] or _rules(case)["pred_tail"] > 2 * case["tol"]


def exact(case, seed):
    """The same from the kernel itself in fp64, where its matrix is small
    enough and the plan's Fourier box is not cut off (a rough field's is: there
    the operator is not the kernel to the tolerance)."""
    n, kind = case["n"], case["kind"]
    pairs = float(n) * (case.get("targets", 0) if kind == "mean" else n) * case.get("iters", 1)
    if pairs > 4e10 or _cut_off(case) or (kind in ("solve", "refined") and n > 32_000):
        return None
    dev = {k: v.to("cuda" if torch.cuda.is_available() else "cpu") for k, v in _inputs(case, seed).items()}
    x, sigma, l, nu, eta = dev["x"], dev["sigma"], dev["l"], case["nu"], case["eta"]

    def product(v, xa=None, sa=None, la=None):
        """K(xa, x) v (n x m), in slabs of rows."""
        noise = xa is None
        xa, sa, la = (x, sigma, l) if noise else (xa, sa, la)
        out = torch.empty(xa.shape[0], v.shape[1], dtype=torch.float64, device=v.device)
        step = max(1, int(5e7 // n))
        for i in range(0, xa.shape[0], step):
            out[i:i + step] = _kernel_rows(nu, xa[i:i + step], sa[i:i + step], la[i:i + step], x, sigma, l) @ v
        return out + eta * eta * v if noise else out

    if kind == "matvec":
        return product(dev["alpha"][:, None])[:, 0]
    if kind == "mean":
        return product(dev["alpha"][:, None], dev["xt"], dev["st"], dev["lt"])[:, 0]
    if kind in ("solve", "refined"):
        A = _kernel_rows(nu, x, sigma, l, x, sigma, l)
        A.diagonal().add_(eta * eta)
        return torch.cholesky_solve(dev["y"][:, None], torch.linalg.cholesky(A))[:, 0]
    b = dev["y"][:, None] if kind == "steps" else dev["Y"].T.contiguous()
    # (block) conjugate gradients with an orthonormal search block
    X, R = torch.zeros_like(b), b.clone()
    P = torch.linalg.qr(R)[0]
    for _ in range(case["iters"]):
        Q = product(P)
        S = P.T @ Q
        a = torch.linalg.solve(S, P.T @ R)
        X += P @ a
        R -= Q @ a
        P = torch.linalg.qr(R - P @ torch.linalg.solve(S, Q.T @ R))[0]
    return X[:, 0] if kind == "steps" else X.T.contiguous()
