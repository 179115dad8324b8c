"""The exact solve on the coarsest level for few and many right-hand sides (a wavefront per row of
A_0^{-1}, or a thread per row), on either side of the rule 8 nrhs >= N
(N unknowns; one problem).

Both are sums of N products with the same matrix entries, so they differ by at most 2 (N + 1) u
sum_j |a_ij| |g_j| <= 2 (N + 1) u |g| / lambda_min(A_0) in any entry, u the unit roundoff."""
import numpy as np
import pytest

from layout import to_padded
from oracle import exact, mesh

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,n0,nrhs", [(2, 2, 3), (5, 5, 29), (5, 5, 30), (10, 5, 61), (20, 5, 300), (14, 7, 94), (14, 7, 95)])
def test_right_hand_sides_agree(n, n0, nrhs, precision):
    from paper_2205_05840_amd import Solver, _lib
    print(f"[case] n={n} nrhs={nrhs} {precision}", flush=True)
    alpha = 0.6
    S1, Sk = Solver(n, alpha, precision=precision), Solver(n, alpha, nrhs=nrhs, precision=precision)
    info = _lib.ndmg_layout(Sk.ctx, 0)
    assert info[0] == n0
    rng = np.random.default_rng(n)
    G = [rng.standard_normal(mesh.ndof(n0)) for _ in range(nrhs)]
    g = torch.from_numpy(np.stack([to_padded(n0, info[1], info[2], v) for v in G])).cuda()
    zk = Sk.level_op(0, "coarse", g.reshape(-1)).reshape(nrhs, -1)
    N, u = mesh.ndof(n0), 2.0 ** (-53 if precision == "fp64" else -24)
    lam = exact.eigenvalues(n0, 1.0 / n0, alpha).min()
    for r in range(nrhs):
        z1 = S1.level_op(0, "coarse", g[r])
        assert z1.abs().max() > 0
        assert float((zk[r] - z1).abs().max()) <= 2 * (N + 1) * u * np.linalg.norm(G[r]) / lam, r
