"""Performance cases: what programs have this library do, from the smallest call to
the largest.

    listed()            the fixed cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs (on the GPU, from the seed alone) and the plan, batch
                        or stepper that a program keeps between calls
    run(state)          one pass through the public entry points; returns its outputs
    work(case)          bytes and flops that a pass cannot do without
    exact(case, seed)   the outputs in plain 64-bit torch / numpy, without the library

A case is a dict of plain values.  `kind` names the call:
    solve     Plan.solve, with `lift` after Plan.lift_boundary on a copy of f
    spectral  Plan.apply_spectral
    refined   Plan.solve_refined in precision `prec` to `tol`
    pcg       Plan.pcg_solve, preconditioner precision `prec`
    batch     Batch.solve over `count` plans drawn from `plans_seed`
    ch        CahnHilliard.step, `steps` steps from a given pair of states
`k`, `nex`, `ney`, `nez` and `bc` (one condition per axis, comma separated) give the
mesh.  An axis has ne k - 1 (dirichlet), ne k + 1 (neumann) or ne k (periodic) unknowns.
"""
import functools
import math
import random

import numpy as np
import torch

import paper_2310_00226_amd as P

CH_EPS, CH_MOB, CH_DT = 0.05, 0.02, 1e-4  # interface width, mobility, time step
PCG_TOL = 1e-12


def listed():
    d3, n3, p3 = (",".join([b] * 3) for b in ("dirichlet", "neumann", "periodic"))
    return [
        # the smallest mesh of the accuracy tables, called again and again inside
        # a program of its own: launches and latency
        {"name": "solve_q4_n31", "kind": "solve", "k": 4, "nex": 8, "ney": 8, "nez": 8, "bc": d3, "alpha": 0.0},
        # a channel with boundary data: another condition on each axis, uneven sizes
        {"name": "solve_q5_mixed_lift", "kind": "solve", "k": 5, "nex": 20, "ney": 13, "nez": 16,
         "bc": "periodic,dirichlet,neumann", "alpha": 1.0, "lift": True},
        # a row of the accuracy tables (Q^6, 32^3 elements, Neumann)
        {"name": "solve_q6_n193", "kind": "solve", "k": 6, "nex": 32, "ney": 32, "nez": 32, "bc": n3, "alpha": 1.0},
        # the benchmark's FP64 solve: a billion unknowns
        {"name": "solve_q4_n999", "kind": "solve", "k": 4, "nex": 250, "ney": 250, "nez": 250, "bc": d3,
         "alpha": 1.0},
        # exponential time differencing on an uneven box
        {"name": "exp_q5_uneven", "kind": "spectral", "k": 5, "nex": 50, "ney": 41, "nez": 37, "bc": d3,
         "alpha": 1.0, "function": "exp", "param": 1e-3},
        # single precision with refinement at an ordinary size, odd extents
        {"name": "refined_f32_q4", "kind": "refined", "k": 4, "nex": 32, "ney": 41, "nez": 36, "bc": d3,
         "alpha": 0.0, "prec": "f32", "tol": 1e-11},
        # the default arguments of solve_refined
        {"name": "refined_bf16_q5_n119", "kind": "refined", "k": 5, "nex": 24, "ney": 24, "nez": 24, "bc": d3,
         "alpha": 1.0, "prec": "bf16", "tol": 1e-11},
        # split BF16 at an ordinary size, uneven axes
        {"name": "refined_bf16x3_q6", "kind": "refined", "k": 6, "nex": 43, "ney": 52, "nez": 38, "bc": d3,
         "alpha": 1.0, "prec": "bf16x3", "tol": 1e-11},
        # the benchmark's headline: a billion unknowns to 1e-10
        {"name": "refined_bf16x3_n999", "kind": "refined", "k": 4, "nex": 250, "ney": 250, "nez": 250, "bc": d3,
         "alpha": 1.0, "prec": "bf16x3", "tol": 1e-10},
        # a part of the benchmark's batch: uneven problems, k = 2..8, 8..64 elements per axis
        {"name": "batch_16_uneven", "kind": "batch", "count": 16, "plans_seed": 2311, "ne_lo": 8, "ne_hi": 64,
         "prec": "bf16x3", "tol": 1e-10},
        # the benchmark's Cahn-Hilliard configuration
        {"name": "ch_q4_n257", "kind": "ch", "k": 4, "nex": 64, "ney": 64, "nez": 64, "prec": "f32", "sweeps": 1,
         "steps": 4},
        # the first mesh of the paper's Schroedinger tables
        {"name": "pcg_q5_n250", "kind": "pcg", "k": 5, "nex": 50, "ney": 50, "nez": 50, "bc": p3, "alpha": 1.0,
         "prec": "bf16x3", "beta": 1.0},
    ]


def draw(rng):
    kind = rng.choice(("solve", "solve", "solve", "spectral", "refined", "refined", "refined", "batch", "ch", "pcg"))

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if kind == "batch":
        lo = rng.randint(4, 12)
        return {"kind": kind, "count": rng.randint(3, 24), "plans_seed": rng.randrange(1 << 20), "ne_lo": lo,
                "ne_hi": lo + log_int(4, 48), "prec": rng.choice(("f32", "bf16x3")), "tol": 1e-10}
    if kind == "ch":
        k = rng.randint(2, 6)
        ne = [max(2, log_int(24, 288) // k) for _ in range(3)]
        return {"kind": kind, "k": k, "nex": ne[0], "ney": ne[1], "nez": ne[2], "prec": rng.choice(("f32", "f64")),
                "sweeps": 1, "steps": rng.randint(1, 6)}
    k = rng.randint(3, 8) if kind == "pcg" else rng.randint(1, 8)
    top = {"pcg": 400, "refined": 480}.get(kind, 520)
    # the axes of a mesh are within a factor of about four of each other
    mid = math.exp(rng.uniform(math.log(14), math.log(top / 1.6)))
    ne = [max(2, int(round(mid * math.exp(rng.uniform(-0.47, 0.47)) / k))) for _ in range(3)]
    bcs = [rng.choice(("dirichlet", "dirichlet", "neumann", "periodic"))] * 3
    if rng.random() < 0.4:
        bcs = [rng.choice(("dirichlet", "neumann", "periodic")) for _ in range(3)]
    case = {"kind": kind, "k": k, "nex": ne[0], "ney": ne[1], "nez": ne[2], "bc": ",".join(bcs),
            "alpha": 0.0 if kind == "solve" and set(bcs) == {"dirichlet"} else round(rng.uniform(0.5, 10.0), 3)}
    if kind == "solve":
        case["lift"] = rng.random() < 0.3
    elif kind == "spectral":
        case["function"] = rng.choice(("exp", "power"))
        case["param"] = 10 ** rng.uniform(-4, -1) if case["function"] == "exp" else rng.choice((0.5, 0.75, 1.5))
    elif kind == "refined":
        case["prec"] = rng.choice(("f32", "bf16x3", "bf16x3", "bf16"))
        case["tol"] = rng.choice((1e-10, 1e-11))
    else:
        case["prec"] = rng.choice(("f64", "bf16x3"))
        case["alpha"], case["beta"] = 1.0, 1.0
    return case


# ---- meshes and inputs -------------------------------------------------------


def _bcs(case):
    return tuple(case["bc"].split(",")) if "bc" in case else ("neumann",) * 3


def _ne(case):
    return case["nex"], case["ney"], case["nez"]


def _box(case):
    lo, hi = {"ch": (0.0, 2 * math.pi), "pcg": (-16.0, 16.0)}.get(case["kind"], (-1.0, 1.0))
    return (lo, hi) * 3


def _dims(case):
    grow = {"dirichlet": -1, "neumann": 1, "periodic": 0}
    return tuple(n * case["k"] + grow[b] for n, b in zip(_ne(case), _bcs(case)))


def _problems(case):
    """The plans of a batch: any mix of degree, element counts and alpha, Dirichlet."""
    r = random.Random(case["plans_seed"])
    return [{"kind": "solve", "k": r.randint(2, 8), "nex": r.randint(case["ne_lo"], case["ne_hi"]),
             "ney": r.randint(case["ne_lo"], case["ne_hi"]), "nez": r.randint(case["ne_lo"], case["ne_hi"]),
             "bc": "dirichlet,dirichlet,dirichlet", "alpha": round(r.uniform(0.0, 10.0), 3)}
            for _ in range(case["count"])]


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _outer(a, b, c):
    return a[:, None, None] * b[None, :, None] * c[None, None, :]


def _grid(case):
    return [torch.from_numpy(_axis(case["k"], n, _box(case)[0], _box(case)[1], b).x).cuda()
            for n, b in zip(_ne(case), _bcs(case))]


def _inputs(case, seed):
    """The arrays of one pass, on the GPU, from the seed alone."""
    g = _generator(seed)
    if case["kind"] == "batch":  # right-hand sides ~ N(0, 1)
        return {"fs": [torch.randn(_dims(p), generator=g, device="cuda", dtype=torch.float64)
                       for p in _problems(case)]}
    dims = _dims(case)
    if case["kind"] == "ch":  # a quench: phi ~ U[-0.05, 0.05]
        return {"phi": (torch.rand(dims, generator=g, device="cuda", dtype=torch.float64) - 0.5) * 0.1}
    grid = _grid(case)
    amp = [float(v) for v in (0.5 + torch.rand(4, generator=g, device="cuda", dtype=torch.float64)).cpu()]
    if case["kind"] == "pcg":  # alpha u - Lap u + V u = f, V between 0 and beta
        s2 = [torch.sin(math.pi * t / 4) ** 2 for t in grid]
        c = [torch.cos(math.pi * t / 16) for t in grid]
        c2 = [torch.cos(math.pi * t / 8) for t in grid]
        v = case["beta"] * _outer(*s2)
        q = (math.pi / 16) ** 2
        f = amp[0] * (case["alpha"] + 3 * q + v) * _outer(*c)
        f += amp[1] * (case["alpha"] + 12 * q + v) * _outer(*c2)
        return {"v": v, "f": f}
    # a smooth solution plus noise of a thousandth
    f = torch.randn(dims, generator=g, device="cuda", dtype=torch.float64)
    f *= 1e-3
    s = [torch.sin(math.pi * t + w) for t, w in zip(grid, amp[1:])]
    f += amp[0] * (3 * math.pi**2 + case["alpha"]) * _outer(*s)
    out = {"f": f}
    if case.get("lift"):  # values or outward fluxes on the faces of the axes that take them
        out["faces"] = []
        for a, b in enumerate(_bcs(case)):
            rest = [d for i, d in enumerate(dims) if i != a]
            for _ in range(2):
                out["faces"].append(None if b == "periodic" else
                                    torch.randn(rest, generator=g, device="cuda", dtype=torch.float64))
    return out


def _plan(case):
    return P.Plan(case["k"], _ne(case), _box(case), case["alpha"], _bcs(case))


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    kind = case["kind"]
    if kind == "batch":
        s["batch"] = P.Batch([_plan(p) for p in _problems(case)])
        s["us"] = [torch.empty_like(f) for f in s["fs"]]
    elif kind == "ch":
        s["stepper"] = P.CahnHilliard(case["k"], _ne(case), _box(case), CH_EPS, CH_MOB, CH_DT, prec=case["prec"],
                                      refine_sweeps=case["sweeps"])
        s["phi_n"], s["phi_nm1"] = torch.empty_like(s["phi"]), torch.empty_like(s["phi"])
    else:
        s["plan"] = _plan(case)
        if case.get("prec", "f64") != "f64":
            s["plan"].tune(case["prec"])
        s["u"] = torch.empty_like(s["f"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        s["batch"].solve(s["fs"], s["us"], prec=case["prec"], tol=case["tol"])
        return s["us"]
    if kind == "ch":  # start from phi_0 at both levels
        s["phi_n"].copy_(s["phi"])
        s["phi_nm1"].copy_(s["phi"])
        s["stepper"].step(s["phi_n"], s["phi_nm1"], case["steps"])
        return s["phi_n"], s["phi_nm1"]
    plan, u = s["plan"], s["u"]
    if kind == "solve":
        f = s["f"]
        if case.get("lift"):
            f = plan.lift_boundary(s["faces"], f.clone())
        return plan.solve(f, u)
    if kind == "spectral":
        return plan.apply_spectral(case["function"], case["alpha"], case["param"], s["f"], u)
    if kind == "refined":
        return plan.solve_refined(s["f"], u, prec=case["prec"], tol=case["tol"])[0]
    return plan.pcg_solve(s["v"], s["f"], u, prec=case["prec"], tol=PCG_TOL)[0]


def _solve_flops(dims):
    """Six mode products, each as two half-size products (even and odd functions of
    the axis): half of 4 N (nx + ny + nz)."""
    return 2.0 * math.prod(dims) * sum(dims)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        dims = [_dims(p) for p in _problems(case)]
        return {"bytes": sum(16.0 * math.prod(d) for d in dims), "flops": sum(map(_solve_flops, dims))}
    dims = _dims(case)
    n = math.prod(dims)
    if kind == "ch":  # two states in, two out; a step is at least one solve
        return {"bytes": 32.0 * n, "flops": case["steps"] * _solve_flops(dims)}
    w = {"bytes": (24.0 if kind == "pcg" else 16.0) * n, "flops": _solve_flops(dims)}
    if case.get("lift"):
        w["bytes"] += sum(16.0 * n / d for d, b in zip(dims, _bcs(case)) if b != "periodic")
    return w


# ---- the same in plain 64-bit arithmetic -------------------------------------
# The 1D eigenpairs are needed beyond 64 bits: the eigenvalues of the smooth modes
# are 1e6 times smaller than the largest.  LAPACK's eigenpairs of the symmetric and
# antisymmetric halves of each axis get one Newton step (Ogita and Aishima, 2018)
# with residuals in long double; matrix products of long double matrices are
# sums of exact products of 21-bit slices.

LD = np.longdouble


def _gll(k):
    """Nodes and weights of the (k + 1)-point Gauss-Lobatto rule, and the derivative
    matrix of its Lagrange basis, in long double."""
    x = -np.cos(np.pi * np.arange(k + 1, dtype=LD) / k)

    def legendre(x):
        p0, p1 = np.ones_like(x), x.copy()
        for j in range(2, k + 1):
            p0, p1 = p1, ((2 * j - 1) * x * p1 - (j - 1) * p0) / LD(j)
        return p0, p1  # P_{k-1}, P_k

    for _ in range(12):  # Newton on (1 - x^2) P_k'
        p0, p1 = legendre(x[1:-1])
        dp = k * (p0 - x[1:-1] * p1) / (1 - x[1:-1] ** 2)
        d2p = (2 * x[1:-1] * dp - k * (k + 1) * p1) / (1 - x[1:-1] ** 2)
        x[1:-1] -= dp / d2p
    x = (x - x[::-1]) / 2
    p = legendre(x)[1]
    w = 2 / (LD(k) * (k + 1) * p**2)
    with np.errstate(divide="ignore"):
        d = p[:, None] / (p[None, :] * (x[:, None] - x[None, :]))
    np.fill_diagonal(d, 0)
    np.fill_diagonal(d, -d.sum(1))
    return x, w, d


def _slices(a, count=4):
    """a as a sum of 64-bit matrices of 21-bit integers times a power of two per column."""
    top = np.exp2(np.ceil(np.log2(np.maximum(np.abs(a).max(0), LD(1e-300)))))
    out = []
    for i in range(1, count + 1):
        unit = top * LD(2.0) ** (-21 * i)
        part = np.rint(a / unit) * unit
        out.append(part.astype(np.float64))
        a = a - part
    return out


def _tmul(a, b):
    """a^T b in long double."""
    a, b = _slices(a), _slices(b)
    total = LD(0)
    for i, x in enumerate(a):
        for y in b[:len(a) - i]:
            total = total + (x.T @ y).astype(LD)
    return total


def _eigenpairs(a):
    """Eigenvalues and vectors of a symmetric long double matrix."""
    lam, x = np.linalg.eigh(a.astype(np.float64))
    x = x.astype(LD)
    ax = _tmul(a, x)
    r = np.eye(len(lam), dtype=LD) - _tmul(x, x)
    s = _tmul(x, ax)
    lam = np.diag(s) / (1 - np.diag(r))
    off = s - np.diag(np.diag(s))
    near = 2 * (np.abs(off).max() + lam[-1] * np.abs(r).max())
    gap = lam[None, :] - lam[:, None]
    with np.errstate(divide="ignore", invalid="ignore"):
        e = np.where(np.abs(gap) > near, (s + lam[None, :] * r) / gap, r / 2)
    return lam, x + (x.astype(np.float64) @ e.astype(np.float64)).astype(LD)


class _Axis:
    """1D operators of one axis: x, mass, lam, S, F = S^T M, H = M^-1 K, and for the
    boundary terms the mass and H of the grid with both end nodes."""

    def __init__(self, k, ne, a, b, bc):
        gx, gw, gd = _gll(k)
        half = (LD(b) - LD(a)) / (2 * ne)
        ke = (gd.T * gw) @ gd / half
        ke = (ke + ke.T) / 2
        np.fill_diagonal(ke, 0)
        np.fill_diagonal(ke, -ke.sum(1))
        n = ne * k + 1
        kk, m, x = np.zeros((n, n), LD), np.zeros(n, LD), np.zeros(n, LD)
        for e in range(ne):
            at = slice(e * k, e * k + k + 1)
            kk[at, at] += ke
            m[at] += gw * half
            x[at] = LD(a) + half * (2 * e + 1 + gx)
        self.full_mass, self.full_h = m.astype(np.float64), (kk / m[:, None]).astype(np.float64)
        if bc == "dirichlet":
            kk, m, x = kk[1:-1, 1:-1], m[1:-1], x[1:-1]
        elif bc == "periodic":
            kk[0] += kk[-1]
            kk[:, 0] += kk[:, -1]
            m[0] += m[-1]
            kk, m, x = kk[:-1, :-1], m[:-1], x[:-1]
        n = len(m)
        self.n, self.x, self.mass = n, x.astype(np.float64), m.astype(np.float64)
        self.h = (kk / m[:, None]).astype(np.float64)
        root = np.sqrt(m)
        s1 = kk / root[:, None] / root[None, :]
        mirror = (n - np.arange(n)) % n if bc == "periodic" else n - 1 - np.arange(n)
        lam, vec = [], []
        for sign in (1, -1):
            rep = np.array([i for i in range(n) if i < mirror[i] or (i == mirror[i] and sign == 1)], int)
            if not len(rep):
                continue
            # basis vectors (e_i +- e_mirror(i)) / sqrt 2, or e_i where i is its own mirror
            fixed = mirror[rep] == rep
            norm = np.where(fixed, np.sqrt(LD(2)), LD(1))
            block = (s1[np.ix_(rep, rep)] + sign * s1[np.ix_(rep, mirror[rep])]) / norm[:, None] / norm[None, :]
            bl, bv = _eigenpairs(block)
            full = np.zeros((n, len(rep)), LD)
            full[mirror[rep]] = sign * bv / np.sqrt(LD(2))
            full[rep] = bv / np.where(fixed, LD(1), np.sqrt(LD(2)))[:, None]
            lam.append(bl)
            vec.append(full)
        vec = np.concatenate(vec, 1)
        self.lam = np.concatenate(lam).astype(np.float64)
        self.s = (vec / root[:, None]).astype(np.float64)
        self.f = (vec.T * root[None, :]).astype(np.float64)


class _Nodes:
    def __init__(self, k, ne, a, b, bc):
        gx = _gll(k)[0]
        half = (LD(b) - LD(a)) / (2 * ne)
        x = np.concatenate([LD(a) + half * (2 * e + 1 + gx[:k]) for e in range(ne)] + [np.array([LD(b)])])
        x = x[1:-1] if bc == "dirichlet" else x[:-1] if bc == "periodic" else x
        self.x = x.astype(np.float64)


@functools.lru_cache(maxsize=256)
def _axis(k, ne, a, b, bc, operators=False):
    return _Axis(k, ne, a, b, bc) if operators else _Nodes(k, ne, a, b, bc)


def _axes(case):
    lo, hi = _box(case)[:2]
    return [_axis(case["k"], n, lo, hi, b, True) for n, b in zip(_ne(case), _bcs(case))]


def _along(matrices, t):
    """Apply one matrix per axis of t."""
    mx, my, mz = (torch.from_numpy(m).to(t.device) for m in matrices)
    nx, ny, nz = t.shape
    t = torch.mm(t.reshape(nx * ny, nz), mz.T.contiguous()).reshape(nx, ny, nz)
    out = torch.empty_like(t)
    for i in range(nx):
        torch.mm(my, t[i], out=out[i])
    return torch.mm(mx, out.reshape(nx, ny * nz), out=t.view(nx, ny * nz)).view(nx, ny, nz)


def _eigen_sum(axes, like):
    lx, ly, lz = (torch.from_numpy(a.lam).to(like.device) for a in axes)
    return lx[:, None, None] + ly[None, :, None] + lz[None, None, :]


def _multiply(axes, f, g):
    c = _along([a.f for a in axes], f)
    c *= g(_eigen_sum(axes, c))
    return _along([a.s for a in axes], c)


def _laplace(axes, u):
    """(H_x + H_y + H_z) u."""
    hx, hy, hz = (torch.from_numpy(a.h).to(u.device) for a in axes)
    nx, ny, nz = u.shape
    out = torch.mm(u.reshape(nx * ny, nz), hz.T.contiguous()).reshape(nx, ny, nz)
    out += torch.mm(hx, u.reshape(nx, ny * nz)).reshape(nx, ny, nz)
    for i in range(nx):
        out[i] += torch.mm(hy, u[i])
    return out


def _lifted(case, axes, f, faces):
    f = f.clone()
    for a, b in enumerate(_bcs(case)):
        if b == "periodic":
            continue
        ax = axes[a]
        t = f.movedim(a, 0)
        for end, face in enumerate(faces[2 * a:2 * a + 2]):
            if b == "neumann":
                t[-end] += face / ax.full_mass[-end]
            else:
                col = torch.from_numpy(ax.full_h[1:-1, -end].copy()).to(f.device)
                t -= col[:, None, None] * face[None]
    return f


def _pcg(case, axes, v, f):
    alpha, shift = case["alpha"], case["alpha"] + case["beta"] / 2
    mass = _outer(*(torch.from_numpy(a.mass).to(f.device) for a in axes))

    def dot(a, b):
        return float((mass * a * b).sum())

    def precondition(r):
        return _multiply(axes, r, lambda s: 1 / (s + shift))

    u, r = torch.zeros_like(f), f.clone()
    z = precondition(r)
    p, rz, norm = z.clone(), dot(r, z), dot(f, f)
    for _ in range(100):
        q = _laplace(axes, p) + (alpha + v) * p
        step = rz / dot(p, q)
        u += step * p
        r -= step * q
        if dot(r, r) <= 1e-28 * norm:
            break
        z = precondition(r)
        rz, old = dot(r, z), rz
        p = z + (rz / old) * p
    return u


def exact(case, seed):
    data = _inputs(case, seed)
    kind = case["kind"]
    if kind == "batch":
        return [_multiply(_axes(p), f, lambda s, a=p["alpha"]: 1 / (s + a))
                for p, f in zip(_problems(case), data["fs"])]
    axes = _axes(case)
    if kind == "ch":
        old = now = data["phi"]
        c = CH_MOB * CH_DT
        for _ in range(case["steps"]):
            bar = 2 * now - old
            lam = _eigen_sum(axes, now)
            t = _along([a.f for a in axes], 2 * now - old / 2)
            t -= c / CH_EPS * lam * _along([a.f for a in axes], bar**3 - bar)
            old, now = now, _along([a.s for a in axes], t / (1.5 + c * CH_EPS * lam * lam))
        return now, old
    f = data["f"]
    if kind == "pcg":
        return _pcg(case, axes, data["v"], f)
    if case.get("lift"):
        f = _lifted(case, axes, f, data["faces"])
    if kind == "spectral":
        p, a = case["param"], case["alpha"]
        if case["function"] == "exp":
            return _multiply(axes, f, lambda s: torch.exp(-p * (s + a)))
        return _multiply(axes, f, lambda s: (s + a) ** -p)
    return _multiply(axes, f, lambda s: 1 / (s + case["alpha"]))
