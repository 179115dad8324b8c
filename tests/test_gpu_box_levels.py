"""The vertex smoother's large-level kernels with coefficient boxes (blocks of subdomains of
one box, patch classes between the boxes) where their indexing has its edges: boxes of one
subdomain per axis, of an odd number, boxes that fill no whole block of 64 or 256 lanes, a
domain with boxes left out, two right-hand sides; and the 64-bit addressing form, bit for
bit the 32-bit one.

Oracle: the literal smoother on the cell-by-cell matrix.  FP64: 0.03 u kappa(A_T) kappa(S)
(the bar of the coefficient tests), FP32: 12 u.
"""
import numpy as np
import pytest

from layout import boundary_mask, from_padded, to_padded
from oracle import coefficient, domain, mesh, smoother

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# n, boxes per axis, levels, boundary patches, boxes left out of the domain, right-hand sides
CASES = [(8, 4, 2, True, False, 0), (12, 6, 2, True, True, 0), (12, 2, 2, False, True, 0), (20, 5, 3, True, False, 0),
         (24, 2, 3, True, True, 0), (16, 2, 0, True, False, 2)]


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("n,r,levels,boundary,cut,nrhs", CASES)
def test_box_smoother(n, r, levels, boundary, cut, nrhs):
    import os
    from paper_2205_05840_amd import Solver, _lib
    rng = np.random.default_rng(n + r)
    boxes = 10.0 ** rng.uniform(-1.5, 1.5, size=(r, r, r))
    active = np.ones((r, r, r), dtype=bool)
    if cut:
        active[rng.integers(r), rng.integers(r), rng.integers(r)] = False
        active[-1, -1, -1] = False
    kw = dict(coef=boxes, domain=active if cut else None, boundary_patches=boundary)
    kw.update(nrhs=nrhs) if nrhs else kw.update(levels=levels)
    print(f"[case] n={n} r={r} levels={levels} boundary={boundary} cut={cut} nrhs={nrhs}", flush=True)
    keep = domain.unknown_mask(n, active)
    cells = coefficient.cell_field(n, boxes)
    A = domain.matrix(n, 1.0 / n, cells, active)
    lit = smoother.LiteralSmoother(A, n, 2, boundary=boundary, **({"keep": keep} if cut else {}))
    k = max(nrhs, 1)
    x = np.zeros((k, mesh.ndof(n)))
    x[:, keep] = rng.standard_normal((k, int(keep.sum())))
    ref = [lit(v[keep]) for v in x]
    scale = 2.0 ** -53 * max(np.linalg.cond(a) for _, a in lit.T) * max(np.linalg.cond(p[3]) for p in lit.P)
    L = _lib.lib()
    for precision, tol in (("fp64", max(1e-13, 0.03 * scale)), ("fp32", 12 * 2.0 ** -24)):
        S = Solver(n, 1.0, precision=precision, **kw)
        g = torch.from_numpy(np.stack([to_padded(n, S.P, S.B, v) for v in x]).reshape(-1)).cuda()
        z = S.level_op(S.levels - 1, "smooth", g)
        for i, zi in enumerate(z.cpu().numpy().reshape(k, -1)):
            assert not zi[boundary_mask(n, S.P, S.B)].any()
            zc = from_padded(n, S.P, S.B, zi)
            assert not zc[~keep].any()
            err = _rel(zc[keep], ref[i])
            print(f"{precision} right-hand side {i}: err {err:.2e}, bound {tol:.2e}")
            assert err <= tol
        try:
            _lib.check(L.ndmg_tuning_set(f"patchaddr {n} {precision} 0 {0 if k == 1 else 1} 64 1".encode()))
            z64 = S.level_op(S.levels - 1, "smooth", g)
        finally:
            L.ndmg_tuning_clear()
            if os.path.exists(_lib.TUNING_PATH):
                L.ndmg_tuning_load(_lib.TUNING_PATH.encode())
        assert torch.equal(z, z64)
