"""The small-level kernels (up to 17^3 vertices over all pairs: one block or wavefront per
vertex, subdomain and coarse node) against the FP64 oracle's V-cycle, at the sizes around
their limit, where a level has one or two subdomains per axis, without boundary patches, with
two smoothing steps (the mode without prolongation), and with several right-hand sides (the
pair offsets; 32^3 with two pairs is past the limit and takes the large-level kernels).

FP64: max(1e-12, 5 spread), the spread of the oracle's LU and Cholesky factors (the bar of
the V-cycle tests).  FP32: 12 u, every factor built in FP64 and rounded once.
"""
import numpy as np
import pytest

from layout import boundary_mask, from_padded, to_padded
from oracle import mesh, vcycle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [(4, 1, 2, True, 0), (6, 2, 1, False, 0), (12, 1, 2, False, 4), (20, 3, 1, True, None), (24, 1, 2, True, None),
         (32, 1, 1, False, None), (32, 2, 1, True, None)]


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs,m,boundary,dense", CASES)
def test_small_level_vcycle(n, nrhs, m, boundary, dense, precision):
    from paper_2205_05840_amd import Solver
    alpha = 0.6
    print(f"[case] n={n} nrhs={nrhs} m={m} boundary={boundary} dense={dense} {precision}", flush=True)
    S = Solver(n, alpha, m=m, boundary_patches=boundary, precision=precision, nrhs=nrhs, dense_n=dense)
    H = vcycle.Hierarchy(n, alpha, m=m, boundary=boundary, factored=True)
    H2 = vcycle.Hierarchy(n, alpha, m=m, boundary=boundary, factored=True, inverse="cholesky")
    g = np.random.default_rng(n).standard_normal((nrhs, mesh.ndof(n)))
    x = np.stack([to_padded(n, S.P, S.B, v) for v in g])
    z = S.vcycle(torch.from_numpy(x if nrhs > 1 else x[0]).cuda()).cpu().numpy().reshape(nrhs, -1)
    for r in range(nrhs):
        ref = H.precondition(g[r])
        tol = max(1e-12, 5.0 * _rel(H2.precondition(g[r]), ref)) if precision == "fp64" else 12 * 2.0 ** -24
        assert not z[r][boundary_mask(n, S.P, S.B)].any()
        assert _rel(from_padded(n, S.P, S.B, z[r]), ref) <= tol, (r, _rel(from_padded(n, S.P, S.B, z[r]), ref), tol)
