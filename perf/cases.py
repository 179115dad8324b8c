"""Performance cases: what a user of the package has it do, through its public classes.

The path is V-cycle-preconditioned CG for curl(alpha curl u) + u = f on edge elements, used
in these ways: the operator or the V-cycle alone inside a caller's own Krylov method
("apply", "vcycle"), one solve ("solve", with its options: FP32 or FP64 V-cycle, subdomain
size, smoother, a coefficient with jumps, a domain that is not the cube, a box), many uneven
problems at once ("batch"), a gradient through the solve ("gradient") and implicit time
stepping ("step").  Sizes are c 2^j elements per axis (c = 2, 3, 5, 7), 8 to 128, the sizes
of the package's own benchmark, tests and time-stepping runs among them.

A case is a dict of plain values: "kind", "n" (elements per axis), "alpha", "precision" (of
the V-cycle; CG is always FP64) and the options of its kind.  Load vectors come from f ~
N(0, 1) at the 2 x 2 x 2 Gauss points of every element, as in the package's benchmark.

A solve returns its solution alone: iteration counts and recursive residuals say how it was
reached, and turn on the last bits of the preconditioner.

`exact` gives the outputs in FP64 torch: the operator written out on whole arrays; its
inverse by sine and cosine transforms (3 x 3 blocks per mode) where alpha is constant on the
cube, else CG preconditioned with that inverse.
"""
import math

import numpy as np
import torch

from paper_2205_05840_amd import BatchedSolver, Solver, solve, synth

DEV = "cuda:0"
RTOL = 1e-10
BATCH_SIZES = (8, 12, 16, 24, 32)


# ---- the cases ---------------------------------------------------------------------------

def listed():
    return [
        # the operator at the size of the headline solve, as a caller's own Krylov method or
        # a residual check calls it
        {"name": "apply-128", "kind": "apply", "n": 128, "alpha": 1.0, "precision": "fp64"},
        # the V-cycle alone, as the preconditioner of a caller's own Krylov method
        {"name": "vcycle-96-fp64", "kind": "vcycle", "n": 96, "alpha": 1.0, "precision": "fp64"},
        # the smallest solve in use: launches and latency
        {"name": "solve-8-fp64", "kind": "solve", "n": 8, "alpha": 1.0, "precision": "fp64"},
        # a small solve in mixed precision, a size that is no power of two (coarsest 5^3)
        {"name": "solve-40-fp32", "kind": "solve", "n": 40, "alpha": 0.01, "precision": "fp32"},
        # an ordinary solve: the 64^3 configuration at its stiffest coefficient, FP64
        {"name": "solve-64-fp64", "kind": "solve", "n": 64, "alpha": 100.0, "precision": "fp64"},
        # the headline: 128^3, mixed precision
        {"name": "solve-128-fp32", "kind": "solve", "n": 128, "alpha": 1.0, "precision": "fp32"},
        # the 64^3 configuration on subdomains of 4^3 elements
        {"name": "solve-64-s4-fp64", "kind": "solve", "n": 64, "alpha": 1.0, "precision": "fp64", "subdomain": 4},
        # a coefficient with jumps on 4^3 boxes, contrast up to 1e4 (coarsest level 4^3)
        {"name": "jumps-128-fp32", "kind": "solve", "n": 128, "alpha": 1.0, "precision": "fp32", "boxes": 4,
         "contrast": 1e4, "levels": 6},
        # a nonconvex domain: the cube less one octant, FP64
        {"name": "domain-64-fp64", "kind": "solve", "n": 64, "alpha": 1.0, "precision": "fp64", "cut": 2},
        # an inverse problem's gradient: 8 right-hand sides, forward and adjoint solve
        {"name": "gradient-64x8", "kind": "gradient", "n": 64, "alpha": 1.0, "precision": "fp64", "nrhs": 8},
        # many uneven problems with 4 right-hand sides each in one call
        {"name": "batch-512x4-fp32", "kind": "batch", "nprob": 512, "nrhs": 4, "pick": 3, "precision": "fp32"},
        # one implicit time step of Maxwell's equations, started from the predictor
        {"name": "step-96-fp32", "kind": "step", "n": 96, "dt": 0.01, "sigma": 1.0, "precision": "fp32"},
    ]


def draw(rng):
    """One more case of the ranges above: every kind, sizes spread over their logarithm."""
    def size(lo, hi, cs=(2, 3, 5, 7)):
        ns = sorted({c << j for c in cs for j in range(8) if lo <= c << j <= hi})
        x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        return min(ns, key=lambda n: (abs(math.log(n / x)), n))

    def alpha(lo, hi):
        return float("%.3g" % 10.0 ** rng.uniform(math.log10(lo), math.log10(hi)))

    prec = rng.choice(("fp32", "fp64"))
    kind = rng.choice(("apply", "vcycle", "solve", "solve", "solve", "option", "option", "option", "gradient", "batch",
                       "batch", "step"))
    if kind == "apply":
        return {"kind": "apply", "n": size(8, 128), "alpha": alpha(1e-2, 1e2), "precision": "fp64"}
    if kind == "vcycle":
        return {"kind": "vcycle", "n": size(8, 128), "alpha": alpha(1e-2, 1.0), "precision": "fp64"}
    if kind == "solve":
        return {"kind": "solve", "n": size(8, 128), "alpha": alpha(1e-2, 1e2), "precision": prec}
    if kind == "option":
        what = rng.choice(("subdomain", "edge", "jumps", "domain", "box"))
        if what == "subdomain":
            return {"kind": "solve", "n": size(16, 64, (2,)), "alpha": alpha(1e-2, 1e2), "precision": prec,
                    "subdomain": 4}
        if what == "edge":
            return {"kind": "solve", "n": size(8, 32, (2, 3)), "alpha": alpha(1e-2, 1.0), "precision": prec,
                    "smoother": "edge"}
        if what == "jumps":
            r = rng.choice((2, 3, 4))
            n = size(16, 96, (3,) if r == 3 else (2,))
            return {"kind": "solve", "n": n, "alpha": alpha(1e-1, 1e1), "precision": prec, "boxes": r,
                    "contrast": alpha(10.0, 1e4), "levels": int(round(math.log2(n // r))) + 1}
        if what == "domain":
            r = rng.choice((2, 3))
            return {"kind": "solve", "n": size(16, 96, (r,)), "alpha": alpha(1e-1, 1e1), "precision": prec, "cut": r}
        n = size(16, 96, (2,))
        return {"kind": "solve", "n": n, "ny": n // 2, "nz": rng.choice((n, n // 2)), "alpha": alpha(1e-1, 1e1),
                "precision": prec}
    if kind == "gradient":
        return {"kind": "gradient", "n": size(8, 64), "alpha": alpha(1e-1, 1e1), "precision": "fp64",
                "nrhs": rng.randint(1, 8)}
    if kind == "batch":
        return {"kind": "batch", "nprob": int(round(math.exp(rng.uniform(math.log(4), math.log(256))))),
                "nrhs": rng.choice((1, 2, 3, 4)), "pick": rng.randint(0, 99), "precision": prec}
    return {"kind": "step", "n": size(16, 128), "dt": alpha(3e-3, 3e-2), "sigma": rng.choice((0.0, 1.0)),
            "precision": prec}


# ---- inputs ------------------------------------------------------------------------------

def _randn(seed, count):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return torch.randn(count, generator=g, dtype=torch.float64, device=DEV)


def _dims(case):
    """Elements per axis (x, y, z)."""
    n = case["n"]
    return (n, case.get("ny", n), case.get("nz", n))


def _boxes(case):
    """Box factors of a coefficient with jumps (a property of the case: the material)."""
    if "boxes" not in case:
        return None
    r, c = case["boxes"], math.log10(case["contrast"]) / 2
    return 10.0 ** np.random.default_rng(3).uniform(-c, c, size=(r, r, r))


def _domain(case):
    """Flags of the boxes kept: the cube less its last box (r = 2: a Fichera corner)."""
    if "cut" not in case:
        return None
    keep = np.ones((case["cut"],) * 3, dtype=bool)
    keep[-1, -1, -1] = False
    return keep


def _alpha(case):
    if case["kind"] == "step":
        return case["dt"] ** 2 / (4 * (1.0 + 0.5 * case["sigma"] * case["dt"]))
    return case["alpha"]


def _problems(case):
    return synth.batched_problems(case["nprob"], seed=case["pick"], sizes=BATCH_SIZES)


def _solver(case, nrhs=1):
    opts = {k: case[k] for k in ("subdomain", "smoother", "levels") if k in case}
    dims = _dims(case)
    if len(set(dims)) > 1:
        return Solver(dims, _alpha(case), length=tuple(d / max(dims) for d in dims), precision=case["precision"], **opts)
    return Solver(case["n"], _alpha(case), precision=case["precision"], coef=_boxes(case), domain=_domain(case),
                  nrhs=nrhs, **opts)


def prepare(case, seed):
    """The solver and the right-hand side (or vector, or fields) on the GPU."""
    if case["kind"] == "batch":
        ns, alphas = _problems(case)
        S = BatchedSolver(ns, alphas, nrhs=case["nrhs"], precision=case["precision"])
        return {"kind": "batch", "S": S, "b": S.assemble_rhs(_randn(seed, S.sample_len()))}
    n, k = case["n"], case.get("nrhs", 1)
    S = _solver(case, k)
    st = {"kind": case["kind"], "S": S}
    if case["kind"] == "apply":
        st["b"] = _randn(seed, S.vec_len) * S.unknown_mask()
        return st
    st["b"] = S.assemble_rhs(_randn(seed, k * n ** 3 * 24))
    if case["kind"] == "gradient":
        st["alpha"] = torch.tensor(case["alpha"], dtype=torch.float64, device=DEV)
        st["target"] = _target(seed, k, S.vec_len) * S.unknown_mask()
        st["b"] = st["b"].reshape(k, -1)
    elif case["kind"] == "step":
        st.update(dt=case["dt"], sigma=case["sigma"], u=S.zeros(), v=S.zeros(), a=S.zeros())   # at rest
    return st


def _target(seed, k, vec_len):
    return 0.1 * _randn(seed + 1, k * vec_len).reshape(k, vec_len)


def run(state):
    S, kind, b = state["S"], state["kind"], state["b"]
    if kind == "apply":
        return S.apply(b)
    if kind == "vcycle":
        return S.vcycle(b)
    if kind in ("solve", "batch"):
        u, _, _ = S.solve(b, rtol=RTOL)
        return u
    if kind == "step":
        S.maxwell_step(b, state["u"], state["v"], state["a"], state["dt"], eps=1.0, sigma=state["sigma"], mu=1.0,
                       rtol=RTOL)
        return state["u"], state["v"], state["a"]
    B = b.detach().requires_grad_(True)
    alpha = state["alpha"].detach().requires_grad_(True)
    U = solve(B, alpha, S)
    loss = ((U - state["target"]) ** 2).sum()
    loss.backward()
    return {"u": U.detach(), "loss": loss.detach(), "grad_b": B.grad, "grad_alpha": alpha.grad}


# ---- the work of one pass ----------------------------------------------------------------

# Iterations to 1e-10 (26 at 128^3, alpha = 1, the same at every size: the V-cycle's
# contraction does not depend on h); with the edge spaces 60 and more.
ITERATIONS = 24
EDGE_ITERATIONS = 60


def _unknowns(case):
    nx, ny, nz = _dims(case)
    d = nx * (ny - 1) * (nz - 1) + (nx - 1) * ny * (nz - 1) + (nx - 1) * (ny - 1) * nz
    return d * (1 - case["cut"] ** -3) if "cut" in case else d


def _cycle_work(case):
    """Bytes and operations per unknown of one V-cycle (8/7: all levels): the residual read,
    the correction written, in its precision; two smoothing steps and two residuals (the patch
    products are 2 |patch|^2 operations each: per unknown 300 on subdomains of 2^3, 1000 on
    4^3; the residual 25)."""
    e = 4 if case["precision"] == "fp32" else 8
    patch = 1000 if case.get("subdomain", 2) == 4 else 30 if case.get("smoother") == "edge" else 300
    return 8 / 7 * 2 * e, 8 / 7 * (2 * patch + 50)


def _solve_work(case, unknowns):
    """Right-hand side in, solution out; per iteration the residual, the direction and the
    solution read and written once (FP64) and a V-cycle."""
    it = EDGE_ITERATIONS if case.get("smoother") == "edge" else ITERATIONS
    cb, cf = _cycle_work(case)
    return {"bytes": unknowns * (16 + it * (48 + cb)), "flops": unknowns * it * (40 + cf)}


def work(case):
    if case["kind"] == "batch":
        w = [_solve_work(case, 3 * int(n) * (int(n) - 1) ** 2 * case["nrhs"]) for n in _problems(case)[0]]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    N = _unknowns(case)
    if case["kind"] == "apply":
        return {"bytes": 16 * N, "flops": 25 * N}
    if case["kind"] == "vcycle":
        cb, cf = _cycle_work(case)
        return {"bytes": cb * N, "flops": cf * N}
    w = _solve_work(case, N)
    if case["kind"] == "step":   # the fields read and written, the load read
        return {"bytes": w["bytes"] + 56 * N, "flops": w["flops"] + 50 * N}
    if case["kind"] == "gradient":   # two solves per right-hand side, the loss and dL/dalpha
        k = case["nrhs"]
        return {"bytes": k * (2 * w["bytes"] + 40 * N), "flops": k * (2 * w["flops"] + 30 * N)}
    return w


# ---- exact outputs: FP64 torch on whole arrays -------------------------------------------
# A field is a list [x, y, z] of edge arrays [..., z, y, x], n entries along the edge and n + 1
# nodes across it.

def _axis(d):
    return -1 - d   # axis of coordinate d in an array [..., z, y, x]


def _diff(a, ax):
    n = a.shape[ax]
    return a.narrow(ax, 1, n - 1) - a.narrow(ax, 0, n - 1)


def _diff_t(a, ax):
    """Transpose of _diff."""
    shape = list(a.shape)
    shape[ax] += 1
    out = a.new_zeros(shape)
    out.narrow(ax, 1, a.shape[ax]).add_(a)
    out.narrow(ax, 0, a.shape[ax]).sub_(a)
    return out


def _mass(a, ax, c=None):
    """Linear elements' 1-D mass matrix along ax (unit cells, factor c per cell)."""
    n = a.shape[ax] - 1
    lo, hi = a.narrow(ax, 0, n), a.narrow(ax, 1, n)
    to_lo, to_hi = lo / 3 + hi / 6, lo / 6 + hi / 3
    if c is not None:
        to_lo, to_hi = c * to_lo, c * to_hi
    out = torch.zeros_like(a)
    out.narrow(ax, 0, n).add_(to_lo)
    out.narrow(ax, 1, n).add_(to_hi)
    return out


def _curl_curl(u, h, c=None):
    out = [torch.zeros_like(x) for x in u]
    for d in range(3):
        a, b = (d + 1) % 3, (d + 2) % 3
        F = _diff(u[b], _axis(a)) - _diff(u[a], _axis(b))   # flux through the faces of normal d
        G = h * _mass(F, _axis(d), c)
        out[b] += _diff_t(G, _axis(a))
        out[a] -= _diff_t(G, _axis(b))
    return out


def _mass_edges(u, h):
    return [h ** 3 * _mass(_mass(u[d], _axis((d + 1) % 3)), _axis((d + 2) % 3)) for d in range(3)]


def _edge_masks(cells):
    """Per direction: edges whose four cells are all inside."""
    n = cells.shape[0]
    out = []
    for d in range(3):
        shape = [n + 1] * 3
        shape[_axis(d)] = n
        m = torch.zeros(shape, dtype=torch.float64, device=DEV)
        a, b = _axis((d + 1) % 3), _axis((d + 2) % 3)
        inner = m.narrow(a, 1, n - 1).narrow(b, 1, n - 1)
        inner.fill_(1.0)
        for i in range(2):
            for j in range(2):
                inner.mul_(cells.narrow(a, i, n - 1).narrow(b, j, n - 1))
        out.append(m)
    return out


def _load(f, n, h):
    """Load vector of f at the Gauss points, f [..., n^3 elements, 8 points, 3 components]."""
    f = f.reshape(f.shape[:-3] + (n, n, n, 2, 2, 2, 3))   # [..., z, y, x, qz, qy, qx, component]
    x = torch.tensor(synth.GAUSS_1D, dtype=torch.float64, device=DEV)
    w = (1 - x, x)
    out = []
    for d in range(3):
        a, b = (d + 1) % 3, (d + 2) % 3
        shape = list(f.shape[:-7]) + [n + 1] * 3
        shape[_axis(d)] = n
        v = f.new_zeros(shape)
        fd = f[..., d].sum(_axis(d))                        # weight 1 along the edge
        across = [q for q in (2, 1, 0) if q != d]           # the two point axes left, in order
        for i in range(2):
            for j in range(2):
                pick = {a: w[i], b: w[j]}
                t = torch.einsum("...pq,p,q->...", fd, pick[across[0]], pick[across[1]])
                v.narrow(_axis(a), i, n).narrow(_axis(b), j, n).add_(h ** 3 / 8 * t)
        out.append(v)
    return out


class _Inverse:
    """A^{-1} on the cube at constant alpha: sine modes across an edge, cosine modes along it
    diagonalise the differences and the 1-D mass matrices, which leaves a 3 x 3 block a mode."""

    def __init__(self, n, alpha, h):
        self.n = n
        p = torch.arange(n, dtype=torch.float64, device=DEV)
        cell = torch.arange(n, dtype=torch.float64, device=DEV)
        node = torch.arange(n + 1, dtype=torch.float64, device=DEV)
        self.cos = math.sqrt(2 / n) * torch.cos(math.pi / n * p[:, None] * (cell[None, :] + 0.5))
        self.cos[0] /= math.sqrt(2)
        self.sin = math.sqrt(2 / n) * torch.sin(math.pi / n * p[:, None] * node[None, :])
        self.sin[0] = 0
        self.sin[:, n] = 0
        s, t = 2 * torch.sin(math.pi / (2 * n) * p), 2 / 3 + torch.cos(math.pi / n * p) / 3
        at = [(None, None, slice(None)), (None, slice(None), None), (slice(None), None, None)]
        s, t = [s[at[d]] for d in range(3)], [t[at[d]] for d in range(3)]
        A = [[None] * 3 for _ in range(3)]
        for d in range(3):
            a, b = (d + 1) % 3, (d + 2) % 3
            A[d][d] = h ** 3 * t[a] * t[b] + alpha * h * (s[a] ** 2 * t[b] + s[b] ** 2 * t[a])
            A[d][a] = A[a][d] = -alpha * h * s[d] * s[a] * t[b]
        l00 = torch.sqrt(A[0][0])
        l10, l20 = A[1][0] / l00, A[2][0] / l00
        l11 = torch.sqrt(A[1][1] - l10 ** 2)
        l21 = (A[2][1] - l20 * l10) / l11
        l22 = torch.sqrt(A[2][2] - l20 ** 2 - l21 ** 2)
        self.L = (l00, l10, l20, l11, l21, l22)

    def _basis(self, x, d, back):
        for ax in range(3):
            m = self.cos if ax == d else self.sin
            m = m.t() if back else m
            x = torch.matmul(x.movedim(_axis(ax), -1), m.t().contiguous()).movedim(-1, _axis(ax))
        return x

    def __call__(self, b):
        g = [self._basis(b[d], d, False) for d in range(3)]
        l00, l10, l20, l11, l21, l22 = self.L
        y0 = g[0] / l00
        y1 = (g[1] - l10 * y0) / l11
        y2 = (g[2] - l20 * y0 - l21 * y1) / l22
        z2 = y2 / l22
        z1 = (y1 - l21 * z2) / l11
        z0 = (y0 - l10 * z1 - l20 * z2) / l00
        return [self._basis(z, d, True) for d, z in enumerate((z0, z1, z2))]


def _pad(u, n):
    """Fields in the package's padded layout, [..., 3 (n + 1)^2 P]."""
    P = (n + 8) // 8 * 8
    lead = u[0].shape[:-3]
    out = torch.zeros(lead + (3, n + 1, n + 1, P), dtype=torch.float64, device=DEV)
    for d in range(3):
        z, y, x = u[d].shape[-3:]
        out[..., d, :z, :y, :x] = u[d]
    return out.reshape(lead + (-1,))


def _unpad(v, n):
    P = (n + 8) // 8 * 8
    v = v.reshape(v.shape[:-1] + (3, n + 1, n + 1, P))
    out = []
    for d in range(3):
        size = [n + 1] * 3
        size[_axis(d)] = n
        out.append(v[..., d, :size[0], :size[1], :size[2]].contiguous())
    return out


def _cells(case):
    """(inside flags, coefficient factors or None) per cell, [z][y][x]."""
    n = case["n"]

    def spread(a):
        for ax in range(3):
            a = a.repeat_interleave(n // a.shape[ax], ax)
        return a

    inside = torch.zeros(n, n, n, dtype=torch.float64, device=DEV)
    nx, ny, nz = _dims(case)
    inside[:nz, :ny, :nx] = 1.0
    if "cut" in case:
        inside = spread(torch.from_numpy(_domain(case).astype(np.float64)).to(DEV))
    if "boxes" in case:
        return inside, spread(torch.from_numpy(_boxes(case)).to(DEV))
    return inside, None


def _dot(a, b):
    return sum(float((x * y).sum()) for x, y in zip(a, b))


def _exact_pcg(case, b, h, cells, coef, masks):
    """A^{-1} b by CG for a coefficient with jumps or a domain inside the cube, preconditioned
    with the cube's inverse at the mean coefficient; None if it does not converge."""
    a = _alpha(case)
    c = coef if coef is not None else cells

    def apply(u):
        K, M = _curl_curl(u, h, c), _mass_edges(u, h)
        return [m * (a * k + v) for m, k, v in zip(masks, K, M)]

    mean = 1.0 if coef is None else float(torch.exp(torch.log(coef).mean()))
    B = _Inverse(case["n"], a * mean, h)
    u = [torch.zeros_like(x) for x in b]
    r = [x.clone() for x in b]
    stop = 1e-13 * math.sqrt(_dot(b, b))
    p, rz = None, 0.0
    for _ in range(5000):
        z = [m * x for m, x in zip(masks, B(r))]
        new = _dot(r, z)
        p = z if p is None else [x + new / rz * y for x, y in zip(z, p)]
        rz = new
        q = apply(p)
        s = rz / _dot(p, q)
        for x, y, w, v in zip(u, r, p, q):
            x.add_(w, alpha=s)
            y.sub_(v, alpha=s)
        if math.sqrt(_dot(r, r)) <= stop:
            return u
    return None


def exact(case, seed):
    kind = case["kind"]
    if kind == "vcycle":
        return None
    if kind == "batch":
        ns, alphas = _problems(case)
        k = case["nrhs"]
        f = _randn(seed, sum(24 * int(n) ** 3 * k for n in ns))
        out, at = [], 0
        for i in np.argsort(ns, kind="stable"):   # batch vectors hold the problems by size
            n, a = int(ns[i]), float(alphas[i])
            h = 1.0 / n
            count = 24 * n ** 3 * k
            b = _load(f[at:at + count].reshape(k, n ** 3, 8, 3), n, h)
            at += count
            out.append(_pad(_Inverse(n, a, h)(b), n).reshape(-1))
        return torch.cat(out)
    n, k, a = case["n"], case.get("nrhs", 1), _alpha(case)
    h = 1.0 / n
    cells, coef = _cells(case)
    masks = _edge_masks(cells)
    if kind == "apply":
        P = (n + 8) // 8 * 8
        u = [m * x for m, x in zip(masks, _unpad(_randn(seed, 3 * (n + 1) ** 2 * P), n))]
        K, M = _curl_curl(u, h), _mass_edges(u, h)
        return _pad([m * (a * x + y) for m, x, y in zip(masks, K, M)], n)
    b = [m * x for m, x in zip(masks, _load(_randn(seed, k * n ** 3 * 24).reshape(k, n ** 3, 8, 3), n, h))]
    if kind == "solve":
        if coef is not None and n > 64:
            return None   # thousands of iterations of a contrast of 1e4: more than 20 seconds
        if coef is not None or float(cells.min()) == 0.0:
            u = _exact_pcg(case, b, h, cells, coef, masks)
            return None if u is None else _pad(u, n)[0]
        return _pad(_Inverse(n, a, h)(b), n)[0]
    if kind == "step":   # from rest: (dt^2 / 4) f / d on the right, a = 4 / dt^2 u, v = dt / 2 a
        dt = case["dt"]
        d = 1.0 + 0.5 * case["sigma"] * dt
        u = _pad(_Inverse(n, a, h)([dt * dt / (4 * d) * x for x in b]), n)[0]
        acc = 4 / dt ** 2 * u
        return u, dt / 2 * acc, acc
    A = _Inverse(n, a, h)
    u = A(b)
    vec_len = _pad(u, n).shape[-1]
    t = [m * x for m, x in zip(masks, _unpad(_target(seed, k, vec_len), n))]
    diff = [x - y for x, y in zip(u, t)]
    lam = A([2 * x for x in diff])
    g_alpha = -_dot(lam, _curl_curl(u, h))
    one = lambda v: torch.tensor(v, dtype=torch.float64, device=DEV)  # noqa: E731
    return {"u": _pad(u, n), "loss": one(_dot(diff, diff)), "grad_b": _pad(lam, n), "grad_alpha": one(g_alpha)}
