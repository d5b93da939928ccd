"""The work whose speed this framework is measured by: whole solves through the
public entry points, from the paper's 25 x 17 chamber to the 8193^2 unit square.

Inputs follow the paper and the benchmark: U[0, 1) Dirichlet values on the
perimeter, a zero start inside, no source or a sum of 32 Gaussian bumps.  A pass
takes new boundary data into a resident grid, solves, and reads the field back
(a request creates and destroys its grid as well).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2208_02427_amd as lap

DEV = "cuda:0"

# Multigrid sides are c * 2^k + 1 (both sides of a grid share k, so that a grid
# coarsens k times); line and point relaxation take any side.


def listed():
    return [
        # The paper's chamber solved by its own sequential line method (its ADI
        # optimum w = 1.3, its stopping rule): the comparison that the paper makes.
        dict(name="chamber_adi_paper", kind="paper", m=25, n=17, method="adi_lex", omega=1.3, beta=1.0),
        # The chamber by multigrid to max|r| < 1e-6: the smallest multigrid call,
        # all latency.
        dict(name="chamber_mg", kind="mg", m=25, n=17, precision="fp64", inner=1, smoother="rb", omega=1.0, source=False,
             beta=1.0, stop="res_inf", tol=1e-6),
        # One served request on an idle device: a ragged grid with a source that
        # arrives, is solved alone in mixed precision and leaves.
        dict(name="request_321x225", kind="request", m=321, n=225, precision="mixed", inner=1, smoother="rb", omega=1.0,
             source=True, beta=1.0, stop="rel_l2", tol=1e-8),
        # An anisotropic grid (dx = 2 dy), where the line smoother is the robust choice.
        dict(name="zebra_641x385", kind="mg", m=641, n=385, precision="fp64", inner=1, smoother="zebra", omega=1.0,
             source=True, beta=2.0, stop="rel_l2", tol=1e-10),
        # An ordinary grid of a parameter study, mixed precision with a source.
        dict(name="mixed_1025", kind="mg", m=1025, n=1025, precision="mixed", inner=1, smoother="rb", omega=1.0,
             source=True, beta=1.0, stop="rel_l2", tol=1e-10),
        # The benchmark's single large grids: plain FP64 V(2,2) to 1e-10.
        dict(name="fp64_4097", kind="mg", m=4097, n=4097, precision="fp64", inner=1, smoother="rb", omega=1.0,
             source=False, beta=1.0, stop="rel_l2", tol=1e-10),
        dict(name="fp64_8193", kind="mg", m=8193, n=8193, precision="fp64", inner=1, smoother="rb", omega=1.0,
             source=False, beta=1.0, stop="rel_l2", tol=1e-10),
        # The benchmark's mixed-precision solve with 32 bumps, four FP32 cycles per correction.
        dict(name="mixed_8193", kind="mg", m=8193, n=8193, precision="mixed", inner=4, smoother="rb", omega=1.0,
             source=True, beta=1.0, stop="rel_l2", tol=1e-10),
        # Red-black SOR on a ragged grid: check blocks of 50 sweeps.
        dict(name="sor_3000x2201", kind="sor", m=3000, n=2201, omega=1.997, source=True, beta=1.0, iters=200, check=50),
        # Line ADI (batched Thomas solves) on one grid: check blocks of 10 iterations.
        dict(name="adi_2049x1500", kind="adi", m=2049, n=1500, omega=1.0, source=False, beta=0.8, iters=20, check=10),
        # Ragged batches in merged launches: mixed multigrid and line ADI.
        dict(name="batch_mixed_48", kind="batch", count=48, lo=33, hi=1025, method="mg", precision="mixed", omega=1.0,
             iters=60, check=1, tol=1e-10),
        dict(name="batch_adi_48", kind="batch", count=48, lo=33, hi=1025, method="adi", precision="fp64", omega=1.0,
             iters=20, check=10, tol=1e-10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mg_sides(rng, lo, hi):
    """Two sides c * 2^k + 1 with c in 4..12 and a common k, the longer one at most `hi`."""
    top = math.exp(rng.uniform(math.log(lo), math.log(hi))) - 1
    k = max(0, int(math.log2(top / 4.0)))
    if rng.random() < 0.5:
        k = max(0, k - 1)
    c = min(12, max(4, int(top / 2 ** k)))
    d = rng.randint(4, c)
    m, n = c * 2 ** k + 1, d * 2 ** k + 1
    return (m, n) if rng.random() < 0.5 else (n, m)


def draw(rng):
    kind = rng.choice(("mg", "mg", "mg", "request", "sor", "adi", "paper", "batch"))
    if kind == "paper":
        method, low, high = rng.choice((("jacobi", 1.0, 1.0), ("sor_lex", 1.5, 1.8), ("slor_lex", 1.23, 1.25), ("adi_lex", 1.2, 1.3)))
        return dict(kind=kind, m=rng.randint(9, 25), n=rng.randint(9, 17), method=method, omega=rng.uniform(low, high),
                    beta=1.0)
    if kind in ("mg", "request"):
        m, n = _mg_sides(rng, 17, 8193 if kind == "mg" else 2049)
        mixed = rng.random() < 0.5
        zebra = kind == "mg" and max(m, n) <= 1025 and rng.random() < 0.2
        return dict(kind=kind, m=m, n=n, precision="mixed" if mixed else "fp64",
                    inner=rng.choice((1, 2, 3, 4)) if mixed and not zebra else 1, smoother="zebra" if zebra else "rb",
                    omega=1.0 if zebra else rng.choice((1.0, 1.0, 1.15)), source=rng.random() < 0.5,
                    beta=rng.uniform(0.6, 1.6) if max(m, n) <= 2049 else 1.0, stop="rel_l2",
                    tol=rng.choice((1e-8, 1e-10)))
    if kind == "sor":
        return dict(kind=kind, m=_log_int(rng, 33, 4097), n=_log_int(rng, 33, 4097), omega=rng.uniform(1.2, 1.99),
                    source=rng.random() < 0.5, beta=rng.uniform(0.6, 1.6), iters=100, check=rng.choice((10, 25, 50)))
    if kind == "adi":
        return dict(kind=kind, m=_log_int(rng, 33, 4097), n=_log_int(rng, 33, 4097), omega=1.0,
                    source=rng.random() < 0.5, beta=rng.uniform(0.6, 1.6), iters=10, check=rng.choice((1, 5, 10)))
    mg = rng.random() < 0.5
    return dict(kind=kind, count=rng.randint(3, 48), lo=17, hi=_log_int(rng, 129, 1025), method="mg" if mg else "adi",
                precision=rng.choice(("fp64", "mixed")) if mg else "fp64", omega=1.0, iters=100 if mg else 10,
                check=1 if mg else 5, tol=rng.choice((1e-8, 1e-10)))


# ------------------------------------------------------------------ inputs
def _spacing(m, n, beta):
    """Unit longer side; dx = beta * dy."""
    h = 1.0 / (max(m, n) - 1)
    return h * beta, h


def _boundary(m, n, rng, scale=1.0):
    psi = torch.zeros((n, m), dtype=torch.float64, device=DEV)
    for view, size in ((psi[0, :], m), (psi[n - 1, :], m), (psi[1:n - 1, 0], n - 2), (psi[1:n - 1, m - 1], n - 2)):
        view.copy_(torch.from_numpy(scale * rng.random(size)))
    return psi


def _chamber(psi_ab):
    """The paper's chamber: psi_ab on the top wall and on the side walls above
    the gap, 0 on the bottom wall and below it."""
    psi = np.zeros((17, 25))
    psi[2:, 0] = psi[2:, -1] = psi_ab
    psi[-1, :] = psi_ab
    return torch.from_numpy(psi).to(DEV)


def _bumps(m, n, dx, dy, rng):
    lx, ly = dx * (m - 1), dy * (n - 1)
    amp, cx, cy = rng.standard_normal(32), rng.random(32) * lx, rng.random(32) * ly
    sig = rng.uniform(0.01, 0.1, 32) * max(lx, ly)
    x = dx * torch.arange(m, dtype=torch.float64, device=DEV)
    y = dy * torch.arange(n, dtype=torch.float64, device=DEV)
    f = torch.zeros((n, m), dtype=torch.float64, device=DEV)
    for a, px, py, s in zip(amp, cx, cy, sig):
        f += (float(a) * torch.exp(-(y - float(py)) ** 2 / (2 * s * s)))[:, None] * torch.exp(-(x - float(px)) ** 2 / (2 * s * s))
    return f


def _problem(case, seed):
    """(psi0, f, dx, dy) of a single-grid case."""
    m, n = case["m"], case["n"]
    rng = np.random.default_rng([seed, m, n])
    if (m, n) == (25, 17):
        return _chamber(100.0 * rng.uniform(0.5, 1.5)), None, 0.25, 0.25
    if case["kind"] == "paper":
        return _boundary(m, n, rng, 100.0), None, 0.25, 0.25
    dx, dy = _spacing(m, n, case["beta"])
    psi0 = _boundary(m, n, rng)
    return psi0, _bumps(m, n, dx, dy, rng) if case["source"] else None, dx, dy


def _batch_shapes(case):
    """(m, n, beta) of each grid of a batch: the longer side log-uniform, aspect up to 3:1, beta in [0.5, 2]."""
    rng = np.random.default_rng([4, case["count"], case["hi"]])
    out = []
    while len(out) < case["count"]:
        top = math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]))) - 1
        k = max(0, int(math.log2(top / 4.0)) - int(rng.integers(2)))
        c = min(12, max(4, int(top / 2 ** k)))
        d = int(rng.integers(max(4, (c + 2) // 3), c + 1))
        m, n = c * 2 ** k + 1, d * 2 ** k + 1
        out.append((m, n, rng.uniform(0.5, 2.0)) if rng.random() < 0.5 else (n, m, rng.uniform(0.5, 2.0)))
    return out


def _batch_problems(case, seed):
    """The grids of a batch case: the sizes belong to the case, the boundary data to the seed."""
    rng = np.random.default_rng([seed, case["count"], case["hi"]])
    return [(_boundary(m, n, rng), None, beta / (n - 1), 1.0 / (n - 1)) for m, n, beta in _batch_shapes(case)]


def _alloc(case):
    if case["kind"] == "sor":
        return lap.LAP_ALLOC_ADI   # the smallest set: SOR itself needs no hierarchy
    if case["kind"] == "adi" or case.get("method") == "adi":
        return lap.LAP_ALLOC_ADI
    return lap.LAP_ALLOC_MIXED if case.get("precision") == "mixed" else lap.LAP_ALLOC_FP64


def _options(case):
    kind = case["kind"]
    if kind in ("mg", "request"):
        return dict(method="mg", precision=case["precision"], inner=case["inner"], smoother=case["smoother"],
                    nu1=1 if case["smoother"] == "zebra" else 2, nu2=1 if case["smoother"] == "zebra" else 2,
                    omega=case["omega"], tol=case["tol"], stop=case["stop"], max_iter=200)
    if kind in ("sor", "adi"):
        return dict(method=kind, omega=case["omega"], tol=1e-10, max_iter=case["iters"], check_every=case["check"])
    if kind == "paper":
        return dict(method=case["method"], omega=case["omega"], tol=1e-9,
                    stop="delta", max_iter=20000, adi_form="inside")
    return dict(method=case["method"], precision=case["precision"], omega=case["omega"], tol=case["tol"],
                max_iter=case["iters"], check_every=case["check"])


def prepare(case, seed):
    if case["kind"] == "batch":
        probs = _batch_problems(case, seed)
        need = sum(lap.footprint(p[0].shape[1], p[0].shape[0], _alloc(case)) for p in probs)
        ctx = lap.Context(arena_bytes=need + (64 << 20), device=DEV)
        grids = [ctx.grid(*p, alloc=_alloc(case)) for p in probs]
        return dict(case=case, ctx=ctx, grids=grids, psi0=[p[0] for p in probs], options=_options(case))
    psi0, f, dx, dy = _problem(case, seed)
    need = lap.footprint(case["m"], case["n"], _alloc(case))
    ctx = lap.Context(arena_bytes=need + (64 << 20), device=DEV)
    state = dict(case=case, ctx=ctx, psi0=psi0, f=f, dx=dx, dy=dy, options=_options(case))
    if case["kind"] != "request":
        state["grid"] = ctx.grid(psi0, f, dx, dy, alloc=_alloc(case))
    return state


def run(state):
    kind, ctx = state["case"]["kind"], state["ctx"]
    if kind == "batch":
        for g, psi0 in zip(state["grids"], state["psi0"]):
            g.write(psi0)
        infos = ctx.solve_batch(state["grids"], **state["options"])
        return [g.read() for g in state["grids"]] + [np.array([i["iterations"] for i in infos])]
    if kind == "request":
        g = ctx.grid(state["psi0"], state["f"], state["dx"], state["dy"], alloc=_alloc(state["case"]))
        info = g.solve(**state["options"])
        out = g.read()
        g.destroy()
        return [out, info["iterations"]]
    g = state["grid"]
    g.write(state["psi0"])
    info = g.solve(**state["options"])
    return [g.read(), info["iterations"]]


# ---------------------------------------------------- what the work needs
def work(case):
    """Field (and source) read once, field written once; the operations of the
    method's own iterations (7 V(2,2) cycles, 5 V(1,1) line-smoothed ones, or the
    stated sweeps), counted at 7 per point update, 10 per line unknown."""
    if case["kind"] == "batch":
        nodes = sum(m * n for m, n, _ in _batch_shapes(case))
        source, iters = False, case["iters"]
        per = 10 * 2 * iters if case["method"] == "adi" else 4 / 3 * 7 * (4 * 7 + 18)
    else:
        nodes, source = case["m"] * case["n"], case.get("source", False)
        per = {"sor": 7 * case.get("iters", 0), "adi": 20 * case.get("iters", 0), "paper": 20 * 50}.get(
            case["kind"], 4 / 3 * (5 * (40 + 18) if case.get("smoother") == "zebra" else 7 * (4 * 7 + 18)))
    return {"bytes": nodes * (24 if source else 16), "flops": nodes * per}


# --------------------------------------------------------- 64-bit results
def _dst(x):
    """Sine transform (type I) of the rows of x."""
    r, k = x.shape
    z = torch.zeros((r, 2 * k + 2), dtype=x.dtype, device=x.device)
    z[:, 1:k + 1] = x
    z[:, k + 2:] = -x.flip(1)
    return -0.5 * torch.fft.rfft(z, dim=1).imag[:, 1:k + 1]


def _direct(psi0, f, dx, dy):
    """The discrete solution: sine transforms in both directions."""
    n, m = psi0.shape
    cx, cy = 1.0 / dx ** 2, 1.0 / dy ** 2
    b = torch.zeros((n - 2, m - 2), dtype=torch.float64, device=psi0.device) if f is None else f[1:-1, 1:-1].clone()
    b[:, 0] -= cx * psi0[1:-1, 0]
    b[:, -1] -= cx * psi0[1:-1, -1]
    b[0, :] -= cy * psi0[0, 1:-1]
    b[-1, :] -= cy * psi0[-1, 1:-1]
    lx = cx * 4 * torch.sin(torch.arange(1, m - 1, dtype=torch.float64, device=b.device) * math.pi / (2 * (m - 1))) ** 2
    ly = cy * 4 * torch.sin(torch.arange(1, n - 1, dtype=torch.float64, device=b.device) * math.pi / (2 * (n - 1))) ** 2
    b = _dst(_dst(b).T.contiguous())                    # [x mode, y mode]
    b = -b / (lx[:, None] + ly[None, :])
    b = _dst(_dst(b).T.contiguous()) * (4.0 / ((m - 1) * (n - 1)))
    out = psi0.clone()
    out[1:-1, 1:-1] = b
    return out


def _sor(psi0, f, dx, dy, omega, iters):
    n, m = psi0.shape
    cx, cy = 1.0 / dx ** 2, 1.0 / dy ** 2
    d = 2.0 * (cx + cy)
    u = psi0.clone()
    rhs = torch.zeros_like(u) if f is None else f
    rows = torch.arange(1, n - 1, device=u.device)[:, None]
    cols = torch.arange(1, m - 1, device=u.device)[None, :]
    w = [omega * ((rows + cols) % 2 == c).double() for c in (0, 1)]
    for _ in range(iters):
        for c in (0, 1):
            t = (cx * (u[1:-1, :-2] + u[1:-1, 2:]) + cy * (u[:-2, 1:-1] + u[2:, 1:-1]) - rhs[1:-1, 1:-1]) / d
            u[1:-1, 1:-1] += w[c] * (t - u[1:-1, 1:-1])
    return u


def _line_inverse(k, c, d):
    off = torch.full((k - 1,), c, dtype=torch.float64, device=DEV)
    return torch.linalg.inv(d * torch.eye(k, dtype=torch.float64, device=DEV) - torch.diag(off, 1) - torch.diag(off, -1))


def _adi(psi0, f, dx, dy, omega, iters):
    n, m = psi0.shape
    cx, cy = 1.0 / dx ** 2, 1.0 / dy ** 2
    u = psi0.clone()
    rhs = torch.zeros_like(u) if f is None else f
    ix, iy = _line_inverse(m - 2, cx, 2 * (cx + cy)), _line_inverse(n - 2, cy, 2 * (cx + cy))

    def half(v, g, inv, along, across):
        k = v.shape[0]
        for first in (1, 2):
            b = across * (v[first - 1:k - 2:2, 1:-1] + v[first + 1:k:2, 1:-1]) - g[first:k - 1:2, 1:-1]
            old = v[first:k - 1:2]
            b[:, 0] += along * old[:, 0]
            b[:, -1] += along * old[:, -1]
            old[:, 1:-1] += omega * (b @ inv - old[:, 1:-1])

    for _ in range(iters):
        half(u, rhs, ix, cx, cy)
        half(u.T, rhs.T, iy, cy, cx)
    return u


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        probs = _batch_problems(case, seed)
        fields = [_direct(*p) if case["method"] == "mg" else _adi(*p, case["omega"], case["iters"]) for p in probs]
        return fields + [None]
    psi0, f, dx, dy = _problem(case, seed)
    if kind == "sor":
        return [_sor(psi0, f, dx, dy, case["omega"], case["iters"]), None]
    if kind == "adi":
        return [_adi(psi0, f, dx, dy, case["omega"], case["iters"]), None]
    return [_direct(psi0, f, dx, dy), None]
