"""The gathered products of the generic smoother on either side of the rules that choose their
block form by the number of units in a launch (few pairs: 16 or 32 units per block; many: 32 or
64, FP32 the form that shares the matrix).  Every sum runs in the order of k in all of them, so
each right-hand side's smoothing step must equal the one of a solver of its own bit for bit (and that
one is held to the oracle elsewhere)."""
import numpy as np
import pytest

from layout import to_padded
from oracle import mesh

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,s,n,nrhs", [("edge", 2, 6, 40), ("edge", 2, 10, 100), ("edge", 2, 32, 3), ("vertex", 4, 16, 20),
                                           ("vertex", 4, 24, 33), ("edge", 4, 16, 30)])
def test_many_units(kind, s, n, nrhs, precision):
    from paper_2205_05840_amd import Solver
    print(f"[case] {kind} s={s} n={n} nrhs={nrhs} {precision}", flush=True)
    kw = dict(smoother=kind, subdomain=s, precision=precision)
    S1, Sk = Solver(n, 0.7, **kw), Solver(n, 0.7, nrhs=nrhs, **kw)
    rng = np.random.default_rng(n)
    g = torch.from_numpy(np.stack([to_padded(n, S1.P, S1.B, rng.standard_normal(mesh.ndof(n))) for _ in range(nrhs)])).cuda()
    zk = Sk.level_op(-1, "smooth", g.reshape(-1)).reshape(nrhs, -1)
    for r in range(nrhs):
        assert torch.equal(zk[r], S1.level_op(-1, "smooth", g[r])), r
