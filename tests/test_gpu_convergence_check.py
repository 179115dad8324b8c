"""The convergence test of CG for few and many pairs (one wavefront per pair, or one thread where
there are few partial sums): pairs stop on their own residuals, a zero right-hand side at once.

Bounds: the relative residual returned is at most rtol = 1e-10; the true one, which differs by
the rounding of the recursion, at most 3 rtol (the bar of the other solver tests).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", [(16, 2), (40, 1), (24, 8), (32, 9), (16, 17), (20, 40), (14, 700)])
def test_pairs_stop_on_their_own(n, nrhs, precision):
    from paper_2205_05840_amd import Solver
    print(f"[case] n={n} nrhs={nrhs} {precision}", flush=True)
    S = Solver(n, 0.8, nrhs=nrhs, precision=precision)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + nrhs)
    b = torch.randn(nrhs, S.vec_len, generator=g, dtype=torch.float64, device="cuda") * S.unknown_mask()
    b *= torch.logspace(-6, 6, nrhs, dtype=torch.float64, device="cuda")[:, None]
    zero = nrhs // 2 if nrhs > 1 else -1
    if zero >= 0:
        b[zero] = 0.0
    flat = b if nrhs > 1 else b[0].contiguous()
    u, it, rel = S.solve(flat, rtol=1e-10)
    it, rel = np.atleast_1d(np.asarray(it)), np.atleast_1d(np.asarray(rel))
    r = (flat - S.apply(u)).reshape(nrhs, -1)
    for p in range(nrhs):
        if p == zero:
            assert it[p] == 0 and not u.reshape(nrhs, -1)[p].any()
        else:
            assert it[p] > 0 and rel[p] <= 1e-10
            assert float(r[p].norm()) <= 3e-10 * float(b[p].norm()), p
