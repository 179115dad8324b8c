"""Small problems, whose CG iterations run as one launch between V-cycles (n <= 12; one block
per pair, unknowns dealt to 1024 lanes): every size that has a hierarchy, several
right-hand sides (the convergence test then a launch of its own), both V-cycle precisions
(the flexible beta), a warm start, and eager launches against graphs.

The solution against the oracle's exact one: ||e|| <= ||r|| / lambda_min(A) for a residual of
rtol ||b|| (factor 2 as in the PCG tests: the recursive residual may lie below the true one by
rounding)."""
import numpy as np
import pytest

from layout import from_padded, to_padded
from oracle import exact, mesh, rhs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", [(2, 1), (3, 2), (4, 1), (5, 1), (6, 3), (7, 1), (8, 1), (8, 5), (10, 1), (10, 2), (12, 1),
                                    (12, 4), (14, 1)])
def test_small_solves(n, nrhs, precision):
    from paper_2205_05840_amd import Solver, synth
    alpha, rtol = 0.4, 1e-10
    print(f"[case] n={n} nrhs={nrhs} {precision}", flush=True)
    b_o = [rhs.load_from_samples(n, 1.0 / n, synth.normal_samples(n, 10 * n + r)) for r in range(nrhs)]
    lam = exact.eigenvalues(n, 1.0 / n, alpha).min()
    ue = [exact.solve_fft(n, 1.0 / n, alpha, b) for b in b_o]
    sols = []
    for graphs in (None, True, False):
        S = Solver(n, alpha, precision=precision, nrhs=nrhs, use_graphs=graphs)
        b = torch.from_numpy(np.stack([to_padded(n, S.P, S.B, v) for v in b_o])).cuda()
        b = b if nrhs > 1 else b[0].contiguous()
        u, it, rel = S.solve(b, rtol=rtol)
        assert np.max(rel) <= rtol
        sols.append(u.clone())
        for r in range(nrhs):
            ur = u.reshape(nrhs, -1)[r].cpu().numpy()
            err = np.linalg.norm(from_padded(n, S.P, S.B, ur) - ue[r])
            assert err <= 2 * rtol * np.linalg.norm(b_o[r]) / lam, (r, err)
        # from the solution: at most the first step, which must not make it worse
        w, it2, rel2 = S.solve(b, rtol=rtol, u=u, warm=True)
        assert np.max(it2) <= 2 and np.max(rel2) <= rtol
    assert torch.equal(sols[0], sols[1]) and torch.equal(sols[0], sols[2])


def test_mesh_counts():
    """(the sizes above cover 2, 3 and 5 unknowns per lane of 1024)"""
    assert [-(-mesh.ndof(n) // 1024) for n in (8, 10, 12)] == [2, 3, 5]
