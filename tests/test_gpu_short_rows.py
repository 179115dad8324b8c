"""The plane-marching operator with several rows per wave (two of 32 positions up to n = 32,
four of 16 up to n = 16, in batches) at the sizes around its limits: short rows, full ones
(the position i = n apart), tiles that end inside and at the last row.  Every launch variant
and plane count gives the same apply bit for bit; each mode agrees with the FP64 oracle, and
solves agree with single solvers, which take other kernels there.

Bounds: the apply's bar against the oracle, 1e-14 = 90 u, in either precision, relative to
|b| + |A| |x|; two solves to 1e-10 differ by no more than 3e-10 |b| / lambda_min each.
"""
import ctypes
import os

import numpy as np
import pytest

from layout import boundary_mask, from_padded, to_padded
from oracle import assemble, mesh

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("n,nrhs", [(10, 65), (12, 64), (14, 64), (16, 64), (20, 5), (24, 4), (28, 4), (32, 5)])
def test_apply_shapes(n, nrhs):
    from paper_2205_05840_amd import Solver, _lib
    print(f"[case] n={n} nrhs={nrhs}", flush=True)
    alpha = 2.5
    L = _lib.lib()
    S = Solver(n, alpha, nrhs=nrhs)
    cls = 4 if nrhs >= 64 else 2
    x = np.random.default_rng(n).standard_normal((nrhs, mesh.ndof(n)))
    xd = torch.from_numpy(np.stack([to_padded(n, S.P, S.B, v) for v in x])).cuda()
    outs = []
    try:
        for v in range(2):
            for kz in (2, 5, n):
                L.ndmg_tuning_clear()
                _lib.check(L.ndmg_tuning_set(f"stencil {n} fp64 0 {cls} {v} {kz}".encode()))
                y = torch.full_like(xd, float("nan"))
                outs.append(S.apply(xd, y).cpu().numpy())
    finally:
        L.ndmg_tuning_clear()
        if os.path.exists(_lib.TUNING_PATH):
            L.ndmg_tuning_load(_lib.TUNING_PATH.encode())
    assert all(np.array_equal(o, outs[0]) for o in outs)
    A = assemble.matrix_kron(n, 1.0 / n, alpha)
    for r in range(nrhs):
        assert _rel(from_padded(n, S.P, S.B, outs[0][r]), A @ x[r]) <= 1e-14, r
        assert np.all(outs[0][r][boundary_mask(n, S.P, S.B)] == 0.0)


@pytest.mark.parametrize("precision,mode", [("fp64", 1), ("fp64", 2), ("fp32", 0), ("fp32", 1)])
@pytest.mark.parametrize("n,count", [(12, 64), (16, 66), (24, 5), (32, 4)])
def test_modes(n, count, precision, mode):
    """The kernel alone, every variant: residual y = b - A x (mode 1), apply with the partial
    sums of x . A x (mode 2)."""
    from paper_2205_05840_amd import _lib
    print(f"[case] n={n} count={count} {precision} mode {mode}", flush=True)
    L = _lib.lib()
    P = (n + 8) // 8 * 8
    B = (n + 1) ** 2 * P
    dt = torch.float64 if precision == "fp64" else torch.float32
    rng = np.random.default_rng(n + mode)
    xs, bs = (rng.standard_normal((count, mesh.ndof(n))).astype(np.float32).astype(np.float64) for _ in range(2))
    x, b = (torch.from_numpy(np.stack([to_padded(n, P, B, v) for v in w])).to("cuda", dt) for w in (xs, bs))
    part = torch.zeros(count * (n * n + 64), dtype=torch.float64, device="cuda")
    alpha = torch.full((count,), 0.7, dtype=torch.float64, device="cuda")
    A = assemble.matrix_kron(n, 1.0 / n, 0.7)
    want = (bs if mode == 1 else 0.0) + (-1.0 if mode == 1 else 1.0) * (A @ xs.T).T
    size = (np.abs(bs) if mode == 1 else 0.0) + (abs(A) @ np.abs(xs).T).T
    tol = 90 * 2.0 ** (-53 if precision == "fp64" else -24)
    us = ctypes.c_double()
    for v in range(2):
        for kz in (2, 5, n):
            y = torch.full_like(x, float("nan"))
            part.fill_(0.0)
            _lib.check(L.ndmg_time_stencil(n, 0 if precision == "fp64" else 1, mode, count, v, kz, x.data_ptr(),
                                           b.data_ptr(), y.data_ptr(), part.data_ptr(), alpha.data_ptr(), 1, 1,
                                           torch.cuda.current_stream().cuda_stream, ctypes.byref(us)))
            got = y.double().cpu().numpy()
            dots = part.cpu().numpy()
            for r in range(count):
                assert np.all(got[r][boundary_mask(n, P, B)] == 0.0)
                err = np.linalg.norm(from_padded(n, P, B, got[r]) - want[r])
                assert err <= tol * np.linalg.norm(size[r]), (v, kz, r)
            if mode == 2:
                ps = ((n + 1) // 2) ** 2   # stride of the partial sums: two rows and planes per tile
                for r in range(count):
                    assert abs(dots[r * ps:(r + 1) * ps].sum() - xs[r] @ want[r]) <= tol * (np.abs(xs[r]) @ size[r])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", [(16, 130), (24, 8), (32, 5)])
def test_solve(n, nrhs, precision):
    from paper_2205_05840_amd import Solver
    print(f"[case] n={n} nrhs={nrhs} {precision}", flush=True)
    S = Solver(n, 0.6, nrhs=nrhs, precision=precision)
    S1 = Solver(n, 0.6, precision=precision)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    b = torch.randn(nrhs, S1.vec_len, generator=g, dtype=torch.float64, device="cuda") * S1.unknown_mask()
    u = S.solve(b, rtol=1e-10)[0]
    lam = (1.0 / n) ** 3 / 9.0   # lower bound of the spectrum (symbol of A)
    for r in (0, nrhs // 2, nrhs - 1):
        u1 = S1.solve(b[r].contiguous(), rtol=1e-10)[0]
        assert float((u[r] - u1).norm()) <= 6e-10 * float(b[r].norm()) / lam, r


@pytest.mark.parametrize("n,nrhs", [(16, 64), (24, 4), (32, 4)])
def test_domain(n, nrhs):
    from paper_2205_05840_amd import Solver
    print(f"[case] n={n} nrhs={nrhs} domain", flush=True)
    dom = np.ones((3, 3, 3) if n == 24 else (2, 2, 2), dtype=bool)
    dom[0, 1, 1] = False
    S, S1 = Solver(n, 1.7, domain=dom, nrhs=nrhs), Solver(n, 1.7, domain=dom)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(nrhs, S1.vec_len, generator=g, dtype=torch.float64, device="cuda") * S1.unknown_mask()
    y = S.apply(x, torch.full_like(x, float("nan")))
    for r in range(nrhs):
        y1 = S1.apply(x[r].contiguous())
        assert float((y[r] - y1).norm() / y1.norm()) <= 2e-14, r
