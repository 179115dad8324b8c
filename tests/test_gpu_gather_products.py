"""The gathered products of the generic smoother (s = 4 and edge spaces) under different launch
shapes: many right-hand sides give each workgroup more row tiles (fewer blocks along the
rows), one gives it a single tile.  Every sum runs in the order of k, so each right-hand
side's smoothing step must equal the one of a solver of its own bit for bit (and that one is
held to the oracle elsewhere)."""
import numpy as np
import pytest

from layout import to_padded
from oracle import mesh

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,s,n,nrhs", [("vertex", 4, 8, 40), ("vertex", 4, 24, 7), ("edge", 2, 12, 9), ("edge", 4, 8, 17)])
def test_shapes_agree(kind, s, n, nrhs, precision):
    from paper_2205_05840_amd import Solver
    print(f"[case] {kind} s={s} n={n} nrhs={nrhs} {precision}", flush=True)
    kw = dict(smoother=kind, subdomain=s, precision=precision)
    S1, Sk = Solver(n, 0.7, **kw), Solver(n, 0.7, nrhs=nrhs, **kw)
    rng = np.random.default_rng(n)
    g = torch.from_numpy(np.stack([to_padded(n, S1.P, S1.B, rng.standard_normal(mesh.ndof(n))) for _ in range(nrhs)])).cuda()
    zk = Sk.level_op(Sk.levels - 1, "smooth", g.reshape(-1)).reshape(nrhs, -1)
    for r in range(nrhs):
        assert torch.equal(zk[r], S1.level_op(S1.levels - 1, "smooth", g[r])), r
