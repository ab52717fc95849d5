"""The calls whose speed matters to a user of this library, as cases that can be timed.

A case is one call, or the short sequence of calls a program makes together, through the public
entry points of paper_1405_0942_amd:

  step      resume from stored positions, take K accepted steps, fetch the positions
  gradient  K recorded steps, then the reverse pass (Relaxation.backward)
  energy    relax_energy, the differentiable form, on a new context (one iteration of a fit)
  analysis  the diagnostics, fields, velocity and breakdown monitors of one state
  noalloc   relax_diagnostics_noalloc on positions and a field in hand

Inputs are the library's test fields (single twist, IsoHelix, braid, ABC box), made on the GPU
from the seed: the seed sets the twist amplitudes or the displacement.

The adaptive runs are those where the step-size rule is limited by accuracy.  Where it is limited
by the explicit stability limit, as on fine grids, the error estimate is the amplified rounding of
the run itself: two evaluations of the same step in 64 bits then part within a few steps.  The
other runs take steps of fixed size, as the parity and gradient runs do.
"""
import itertools
import math
import types

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

import paper_1405_0942_amd as R

GAMMA, TAU = 1.0, 1e-12


def _case(name, kind, field, n, steps=0, precision="fp64", curl="nn", adaptive=False, every=0):
    nx, ny, nz = n
    c = {"kind": kind, "field": field, "nx": nx, "ny": ny, "nz": nz, "steps": steps, "precision": precision,
         "curl": curl, "adaptive": adaptive, "every": every}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest run of the test-suite and of smoke(): every launch and wait shows
        _case("step_twist_16", "step", "twist", (16, 16, 16), 50, adaptive=True),
        # the vertex grids (2^m + 1 nodes) of the IsoHelix and Pontin09 tables, small and large
        _case("step_helix_33", "step", "helix", (33, 33, 33), 30, adaptive=True),
        _case("step_helix_129", "step", "helix", (129, 129, 129), 10),
        # the braid: mixed boundaries, the long runs, rejected attempts among them
        _case("step_braid_64x64x192", "step", "braid", (64, 64, 192), 20, adaptive=True),
        # the throughput workload of bench.py in both precisions, and a larger box
        _case("step_abc_256", "step", "abc", (256, 256, 256), 10),
        _case("step_abc_256_mixed", "step", "abc", (256, 256, 256), 10, precision="mixed"),
        _case("step_abc_384", "step", "abc", (384, 384, 384), 4),
        # the octilateral current on a vertex grid
        _case("step_octilateral_65", "step", "helix", (65, 65, 65), 15, curl="nnn"),
        # gradients: one iteration of a fit on the smallest grid, and the braid gradients
        _case("energy_twist_16", "energy", "twist", (16, 16, 16), 20, every=10),
        _case("gradient_braid_64x64x192", "gradient", "braid", (64, 64, 192), 8, every=4),
        # what is looked at between runs: every field and monitor of a state
        _case("analysis_helix_65", "analysis", "helix", (65, 65, 65)),
        # the diagnostics of positions in hand, inside a serving loop
        _case("noalloc_abc_128", "noalloc", "abc", (128, 128, 128)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "gradient", "energy", "analysis", "noalloc"])
    field = rng.choice(["twist", "helix", "braid", "abc"])
    # a typical length, then axes up to 40 % either side of it, odd sizes among them
    top = {"step": 330, "gradient": 110, "energy": 40, "analysis": 200, "noalloc": 200}[kind]
    m = _log_int(rng, 14, top)
    n = [max(9, int(m * rng.uniform(0.7, 1.4))) for _ in range(3)]
    if field == "helix":  # vertex grids have the same count on every axis
        n = [m | 1] * 3
    if field == "braid":  # three times as many nodes along the braid
        n = [max(12, int(m * 0.7)), max(12, int(m * 0.7)), int(m * 2.1)]
    N = n[0] * n[1] * n[2]
    precision, curl, adaptive = "fp64", "nn", False
    if kind == "step":
        if m >= 96 and rng.random() < 0.4:  # the mixed mode is for large runs
            precision = "mixed"
        elif N < 5_000_000 and rng.random() < 0.25:
            curl = "nnn"
        else:
            adaptive = m <= (64 if field == "braid" else 36)
    steps = {"step": max(3, min(_log_int(rng, 6, 20 if m > 36 else 40), 100_000_000 // N)),
             "gradient": rng.randint(3, 8), "energy": rng.randint(5, 20)}.get(kind, 0)
    every = rng.randint(2, steps) if kind in ("gradient", "energy") else 0
    return _case(None, kind, field, n, steps, precision, curl, adaptive, every)


# ---- inputs ------------------------------------------------------------------------------------

LINE_TIED, PERIODIC = R.RELAX_LINE_TIED, R.RELAX_PERIODIC
BOX = {
    "twist": ([(-1.0, 1.0)] * 3, (LINE_TIED,) * 3),
    "helix": ([(-4.0, 4.0), (-4.0, 4.0), (-10.0, 10.0)], (LINE_TIED,) * 3),
    "braid": ([(-4.0, 4.0), (-4.0, 4.0), (-24.0, 24.0)], (PERIODIC, PERIODIC, LINE_TIED)),
    "abc": ([(0.0, 2 * math.pi)] * 3, (PERIODIC,) * 3),
}


def _grid(case):
    n = (case["nx"], case["ny"], case["nz"])
    spans, bc = BOX[case["field"]]
    h = tuple((hi - lo) / (n[a] if bc[a] == PERIODIC else n[a] - 1) for a, (lo, hi) in enumerate(spans))
    return types.SimpleNamespace(n=n, h=h, bc=bc, lo=tuple(s[0] for s in spans), N=n[0] * n[1] * n[2])


def _axes(g):
    ax = [g.lo[a] + g.h[a] * torch.arange(g.n[a], dtype=torch.float64, device="cuda") for a in range(3)]
    return ax[0].view(1, 1, -1), ax[1].view(1, -1, 1), ax[2].view(-1, 1, 1)


def _separable(tables, coef):
    """sum over (l, m, k) of coef[l, m, k] tz[:, l] ty[:, m] tx[:, k] as an (nz, ny, nx) tensor; the
    real part where the tables are complex."""
    tx, ty, tz = tables
    plane = np.einsum("ym,lmk,xk->lyx", ty, coef, tx, optimize=True)
    a, b = tz, plane.reshape(plane.shape[0], -1)
    if np.iscomplexobj(b):
        a, b = np.concatenate([a.real, -a.imag], 1), np.concatenate([b.real, b.imag], 0)
    out = torch.from_numpy(np.ascontiguousarray(a)).cuda() @ torch.from_numpy(np.ascontiguousarray(b)).cuda()
    return out.view(tz.shape[0], ty.shape[0], tx.shape[0])


def _displacement(case, g, rng):
    ax = [g.lo[a] + g.h[a] * np.arange(g.n[a]) for a in range(3)]
    if case["field"] == "twist":  # two sine modes per axis, zero on the walls
        tables = [np.stack([np.sin(m * math.pi * (v + 1.0) / 2.0) for m in (1, 2)], 1) for v in ax]
        coef, amp = rng.standard_normal((3, 2, 2, 2)), 0.02
    else:  # ABC box: divergence-free, 0 < |k| <= 3
        tables = [np.exp(1j * v[:, None] * np.arange(-3, 4)) for v in ax]
        coef, amp = np.zeros((3, 7, 7, 7), dtype=complex), 0.1
        for k in itertools.product(range(-3, 4), repeat=3):
            if 0 < sum(v * v for v in k) <= 9 and k > (0, 0, 0):
                kv = np.array(k, dtype=float)
                c = rng.standard_normal(3) - 1j * rng.standard_normal(3)
                coef[:, k[2] + 3, k[1] + 3, k[0] + 3] = c - kv * (kv @ c) / (kv @ kv)
    d = torch.stack([_separable(tables, coef[c]) for c in range(3)])
    return d * (amp / d.square().sum(0).max().sqrt())


def _inputs(case, seed):
    """(grid, x0, B0, dt0, tol) of a case, the tensors on the GPU."""
    g, rng = _grid(case), np.random.default_rng(seed)
    X, Y, Z = _axes(g)
    shape = (g.n[2], g.n[1], g.n[0])
    field, one = case["field"], torch.ones(shape, dtype=torch.float64, device="cuda")
    x0 = torch.stack([X.expand(shape), Y.expand(shape), Z.expand(shape)])
    r2 = X ** 2 + Y ** 2
    if field == "twist":
        a = 0.5
        amp = (2.0 * rng.uniform(0.5, 1.5) / a) * torch.exp(-r2 / a ** 2 - Z ** 2 / a ** 2)
        B0 = torch.stack([-Y * amp, X * amp, one])
    elif field == "helix":
        amp = 0.5 * Z * math.pi * rng.uniform(0.2, 0.3) * torch.exp(-r2 / 2.0 - Z ** 2 / 4.0)
        B0 = torch.stack([Y * amp, -X * amp, one])
    elif field == "braid":
        bx, by = torch.zeros_like(one), torch.zeros_like(one)
        for m, k in enumerate(rng.uniform(0.5, 1.5, 6)):
            s = float((-1) ** m)
            for ix, iy in itertools.product((-1, 0, 1), repeat=2):
                x, y = X - 8.0 * ix - s, Y - 8.0 * iy
                w = s * (2.0 * k / math.sqrt(2.0)) * torch.exp(-(x ** 2 + y ** 2) / 2.0 - (Z + 15.0 - 6.0 * m) ** 2 / 4.0)
                bx -= y * w
                by += x * w
        B0 = torch.stack([bx, by, one])
    else:
        B0 = torch.stack([torch.sin(Z) + torch.cos(Y) + 0 * X, torch.sin(X) + torch.cos(Z) + 0 * Y,
                          torch.sin(Y) + torch.cos(X) + 0 * Z])
    if field in ("twist", "abc"):
        x0 = x0 + _displacement(case, g, rng)
    # a step inside the explicit stability limit (about h^2 / 6 in the ABC box)
    return g, x0.contiguous(), B0.contiguous(), 0.1 * min(g.h) ** 2, 1e-7 if field in ("braid", "abc") else 1e-8


def _config(case, g, dt0, tol):
    return R.make_config(g, precision=R.RELAX_FP32_MIXED if case["precision"] == "mixed" else R.RELAX_FP64, gamma=GAMMA,
                         dt0=dt0, tol=tol, adaptive=case["adaptive"], record=case["every"] > 0,
                         checkpoint_every=max(1, case["every"]), xi_null_tau=TAU, safety=0.9,
                         curl=R.RELAX_CURL_NNN if case["curl"] == "nnn" else R.RELAX_CURL_NN)


def prepare(case, seed):
    g, x0, B0, dt0, tol = _inputs(case, seed)
    s = {"case": case, "x0": x0, "B0": B0, "dt0": dt0, "cfg": _config(case, g, dt0, tol)}
    if case["kind"] == "energy":
        x0.requires_grad_(True)
        B0.requires_grad_(True)
    elif case["kind"] == "noalloc":
        s["stream"] = torch.cuda.current_stream().cuda_stream
    else:
        s["relax"] = R.Relaxation(s["cfg"], x0, B0, K_record=case["steps"] if case["every"] else 0)
    return s


# ---- one pass ----------------------------------------------------------------------------------

PER_STEP = ("t", "dt", "E_M", "xi", "R2", "min_det")
OF_STATE = ("E_M", "xi", "R2", "min_det")


def _columns(records, case):
    """The per-step records as arrays.  Adaptive runs: with the error estimate, a cancellation that is
    good to about eight digits, as are the step sizes that follow from it, so in single precision;
    so are the records that FP32 sweeps make.  With fixed steps the estimate (1e-15 and below) is
    rounding alone and steers nothing."""
    kind = np.float32 if case["adaptive"] or case["precision"] == "mixed" else np.float64
    out = {f: np.array([d[f] for d in records], dtype=kind) for f in PER_STEP + (("Lambda",) if case["adaptive"] else ())}
    out["rejects"] = np.array([d["rejects"] for d in records], dtype=np.int64)
    return out


def _numbers(d):
    return {**{f: np.float64(d[f]) for f in OF_STATE}, "concave": int(d["concave"])}


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "energy":
        E, R2 = R.relax_energy(state["x0"], state["B0"], state["cfg"], case["steps"])
        gx, gb = torch.autograd.grad(E + 0.1 * R2, (state["x0"], state["B0"]))
        return {"E_M": E.detach(), "R2": R2.detach(), "grad_x0": gx, "grad_B0": gb}
    if kind == "noalloc":
        rc, d = R.relax_diagnostics_noalloc(state["cfg"], state["x0"].data_ptr(), state["B0"].data_ptr(), state["stream"])
        if rc != R.RELAX_OK:
            raise R.RelaxError(rc, "relax_diagnostics_noalloc")
        return _numbers({f: getattr(d, f) for f in R.DIAG_FIELDS})
    r = state["relax"]
    if kind == "analysis":
        d = r.diagnostics()
        B, J = r.fields()
        u = r.velocity()
        alpha, kappa = r.monitors()
        return {**_numbers(d), "B": B, "J": J, "u": u, "alpha": alpha, "kappa": kappa}
    r.set_state(state["x0"], 0.0, state["dt0"])
    if kind == "gradient":
        r.step(case["steps"], diag=False)
        gx, gb = r.backward(1.0, 0.1)
        return {"grad_x0": gx, "grad_B0": gb}
    records = r.step(case["steps"])
    x, t, dt = r.state()
    return {"steps": _columns(records, case), "x": x, "t": np.float32(t), "dt": np.float32(dt)}


def work(case):
    """Bytes: a step reads x and B0 and writes x (24 bytes a node each); the reverse of a step reads x,
    B0 and both cotangents and writes the cotangents.  Flops: about 200 a node and evaluation of the
    right-hand side (700 with the octilateral loops), three times that for its transpose."""
    N, K = case["nx"] * case["ny"] * case["nz"], case["steps"]
    rhs = (700 if case["curl"] == "nnn" else 200) * N
    if case["kind"] == "step":
        return {"bytes": 72 * N * K, "flops": 6 * rhs * K}
    if case["kind"] in ("energy", "gradient"):
        return {"bytes": (72 + 144) * N * K, "flops": 4 * 6 * rhs * K}
    if case["kind"] == "analysis":
        return {"bytes": (48 + 72 + 12) * N, "flops": rhs}
    return {"bytes": 48 * N, "flops": rhs}


# ---- the same in plain torch, 64 bits ------------------------------------------------------------

CK_A = [[], [1 / 5], [3 / 40, 9 / 40], [3 / 10, -9 / 10, 6 / 5], [-11 / 54, 5 / 2, -70 / 27, 35 / 27],
        [1631 / 55296, 175 / 512, 575 / 13824, 44275 / 110592, 253 / 4096]]
CK_B5 = [37 / 378, 0, 250 / 621, 125 / 594, 0, 512 / 1771]
CK_B4 = [2825 / 27648, 0, 18575 / 48384, 13525 / 55296, 277 / 14336, 1 / 4]


def _pad(v, g, shift):
    """v with one ghost node on both sides of every axis: the periodic image (positions move by the
    period), or zeros on line-tied axes."""
    for a in range(3):
        dim = 3 - a
        lo, hi = v.narrow(dim, v.shape[dim] - 1, 1), v.narrow(dim, 0, 1)
        if g.bc[a] == PERIODIC:
            if shift:
                e = torch.zeros((3, 1, 1, 1), dtype=v.dtype, device=v.device)
                e[a] = g.n[a] * g.h[a]
                lo, hi = lo - e, hi + e
        else:
            lo, hi = torch.zeros_like(lo), torch.zeros_like(hi)
        v = torch.cat([lo, v, hi], dim)
    return v


def _at(p, g, dx, dy, dz):
    return p[:, 1 + dz:1 + dz + g.n[2], 1 + dy:1 + dy + g.n[1], 1 + dx:1 + dx + g.n[0]]


def _difference(p, v, g, a, ends):
    """The central difference v(+e_a) - v(-e_a); with `ends`, the one-sided rows at line-tied ends."""
    e = [0, 0, 0]
    e[a] = 1
    d = _at(p, g, *e) - _at(p, g, *[-k for k in e])
    if ends and g.bc[a] == LINE_TIED:
        dim, n = 3 - a, g.n[a]
        s = [v.narrow(dim, k, 1) for k in (0, 1, 2, n - 1, n - 2, n - 3)]
        d = torch.cat([-3 * s[0] + 4 * s[1] - s[2], d.narrow(dim, 1, n - 2), 3 * s[3] - 4 * s[4] + s[5]], dim)
    return d


def _dot(u, v):
    return u[0] * v[0] + u[1] * v[1] + u[2] * v[2]


def _cross(u, v):
    return torch.stack([u[1] * v[2] - u[2] * v[1], u[2] * v[0] - u[0] * v[2], u[0] * v[1] - u[1] * v[0]])


def _interior(g):
    m = torch.ones((g.n[2], g.n[1], g.n[0]), dtype=torch.float64, device="cuda")
    for a in range(3):
        if g.bc[a] == LINE_TIED:
            m.narrow(2 - a, 0, 1).zero_()
            m.narrow(2 - a, g.n[a] - 1, 1).zero_()
    return m


def _octilateral(p, Bp, g):
    """Cramer's rule on the three octilateral loops of every node."""
    ring = [(1, 0), (1, 1), (0, 1), (-1, 1), (-1, 0), (-1, -1), (0, -1), (1, -1)]
    M, C = [], []
    for q in range(3):
        ab = ((q + 1) % 3, (q + 2) % 3)
        V, W = [], []
        for da, db in ring:
            e = [0, 0, 0]
            e[ab[0]], e[ab[1]] = da, db
            V.append(_at(p, g, *e))
            W.append(_at(Bp, g, *e))
        d = [V[(r + 1) % 8] - V[r] for r in range(8)]
        C.append(sum(_dot(0.5 * (W[r] + W[(r + 1) % 8]), d[r]) for r in range(8)))
        area = sum(0.5 * _cross(d[r], d[(r + 1) % 8]) for r in (1, 3, 5, 7))
        D = [V[3] - V[1], V[5] - V[3], V[7] - V[5], V[1] - V[7]]
        M.append(area + sum(0.25 * _cross(D[k], D[(k + 1) % 4]) for k in range(4)))
    x = [_cross(M[1], M[2]), _cross(M[2], M[0]), _cross(M[0], M[1])]
    det = _dot(M[0], x[0])
    return (C[0] * x[0] + C[1] * x[1] + C[2] * x[2]) / torch.where(det == 0, torch.ones_like(det), det)


def _evaluate(y, B0, g, curl, inner):
    """(u, B, J, det F) of the positions y."""
    p = _pad(y, g, True)
    F = [_difference(p, y, g, a, True) / (2 * g.h[a]) for a in range(3)]
    D = _dot(F[0], _cross(F[1], F[2]))
    B = (F[0] * B0[0] + F[1] * B0[1] + F[2] * B0[2]) / D
    Bp = _pad(B, g, False)
    if curl == "nnn":
        J = _octilateral(p, Bp, g) * inner
    else:
        G = [_difference(Bp, B, g, a, False) / (2 * g.h[a]) for a in range(3)]
        J = sum(F[q] * (_dot(F[(q + 2) % 3], G[(q + 1) % 3]) - _dot(F[(q + 1) % 3], G[(q + 2) % 3])) for q in range(3)) / D
        J = J * inner
    return GAMMA * _cross(J, B), B, J, D


def _measures(B, J, D, B0, g, inner):
    f2, b2 = _cross(J, B).square().sum(0), B.square().sum(0)
    zeta, dV = torch.ones_like(D), g.h[0] * g.h[1] * g.h[2]
    for a in range(3):
        if g.bc[a] == LINE_TIED:
            zeta.narrow(2 - a, 0, 1).mul_(0.5)
            zeta.narrow(2 - a, g.n[a] - 1, 1).mul_(0.5)
    on = (inner > 0) & (b2 > TAU * B0.square().sum(0).max())
    xi = torch.where(on, f2.sqrt() / b2, torch.zeros_like(b2)).max()
    return {"E_M": 0.5 * (zeta * b2 * D).sum() * dV, "xi": xi, "R2": 0.5 * (inner * D * f2).sum() * dV, "min_det": D.min()}


def _convex(x, g):
    p, ok = _pad(x, g, True), torch.ones(x.shape[1:], dtype=torch.bool, device=x.device)
    for s in itertools.product((-1, 1), repeat=3):
        e = [_at(p, g, *[s[a] if b == a else 0 for b in range(3)]) - x for a in range(3)]
        bad = ~(_dot(e[0], _cross(e[1], e[2])) * (s[0] * s[1] * s[2]) > 0)
        for a in range(3):
            if g.bc[a] == LINE_TIED:
                bad.narrow(2 - a, 0 if s[a] < 0 else g.n[a] - 1, 1).fill_(False)
        ok &= ~bad
    return ok


def _attempt(x, B0, dt, g, case, inner):
    """(x of the fifth order, max |x5 - x4|, the evaluation at x)."""
    k = []
    for s in range(6):
        y = x + dt * sum(CK_A[s][j] * k[j] for j in range(s)) if s else x
        u, *rest = _evaluate(y, B0, g, case["curl"], inner)
        if s == 0:
            first = rest
        k.append(u)
    err = dt * sum((CK_B5[j] - CK_B4[j]) * k[j] for j in range(6))
    return x + dt * sum(CK_B5[j] * k[j] for j in range(6)), err.abs().max(), first


def _march(x, B0, g, dt, tol, case, inner):
    """K accepted steps by the step-size rule (safety 0.9): positions, step sizes and records."""
    t, records, sizes = 0.0, [], []
    while len(records) < case["steps"]:
        rejects = 0
        while True:
            new, lam, (B, J, D) = _attempt(x, B0, dt, g, case, inner)
            lam = float(lam)
            size, other = dt, 0.9 * dt * abs(tol / lam) ** 0.2 if lam > 0 else 5 * dt
            if not case["adaptive"]:
                break
            if lam <= tol:
                dt = other if lam < 0.5 * tol else dt
                break
            rejects, dt = rejects + 1, other
        m = {f: float(v) for f, v in _measures(B, J, D, B0, g, inner).items()}
        records.append({"t": t, "dt": size, "Lambda": lam, "rejects": rejects, **m})
        sizes.append(size)
        t, x = t + size, new
    return x, t, dt, sizes, records


def exact(case, seed):
    g, x0, B0, dt0, tol = _inputs(case, seed)
    inner, kind = _interior(g), case["kind"]
    if kind in ("analysis", "noalloc"):
        u, B, J, D = _evaluate(x0, B0, g, case["curl"], inner)
        ok = _convex(x0, g)
        out = {f: np.float64(float(v)) for f, v in _measures(B, J, D, B0, g, inner).items()}
        out["concave"] = int((~ok).sum())
        if kind == "noalloc":
            return out
        b2 = B.square().sum(0)
        alpha = torch.where(b2 > 0, _dot(J, B) / b2, torch.zeros_like(b2))
        return {**out, "B": B, "J": J, "u": u, "alpha": alpha, "kappa": torch.where(ok, 1, -1).to(torch.int32)}
    with torch.no_grad():
        x, t, dt, sizes, records = _march(x0, B0, g, dt0, tol, case, inner)
    if kind == "step":
        return {"steps": _columns(records, case), "x": x, "t": np.float32(t), "dt": np.float32(dt)}
    x0.requires_grad_(True)
    B0.requires_grad_(True)
    x = x0
    for size in sizes:
        x = checkpoint(lambda v, b, d=size: _attempt(v, b, d, g, case, inner)[0], x, B0, use_reentrant=False)
    _, B, J, D = _evaluate(x, B0, g, case["curl"], inner)
    m = _measures(B, J, D, B0.detach(), g, inner)
    gx, gb = torch.autograd.grad(m["E_M"] + 0.1 * m["R2"], (x0, B0))
    out = {"grad_x0": gx, "grad_B0": gb}
    return out if kind == "gradient" else {"E_M": m["E_M"].detach(), "R2": m["R2"].detach(), **out}
