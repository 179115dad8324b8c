"""Interface sums of planes of up to 16 x 16 subdomains (one block per plane, from 8 pairs on)
against the one-subdomain-per-lane kernel that one pair takes: one smoothing step at planes
of 2 x 2 to 16 x 16 subdomains (and 20 x 20, past the limit), with and without boundary patches.

Bound: an interface value is a sum of at most 4 patch results, in another order (3 roundings
each side); through the harmonic extension and its own rounding 32 u relative.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs,boundary", [(4, 8, True), (6, 9, False), (14, 8, True), (20, 11, True), (28, 8, False),
                                             (32, 8, True), (40, 8, True)])
def test_smoothing_step(n, nrhs, boundary, precision):
    from paper_2205_05840_amd import Solver
    print(f"[case] n={n} nrhs={nrhs} boundary={boundary} {precision}", flush=True)
    kw = dict(precision=precision, boundary_patches=boundary, dense_n=0, bottom_n=0)
    S, S1 = Solver(n, 0.7, nrhs=nrhs, **kw), Solver(n, 0.7, **kw)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(nrhs, S1.vec_len, generator=g, dtype=torch.float64, device="cuda") * S1.unknown_mask()
    z = S.level_op(-1, "smooth", x.reshape(-1)).reshape(nrhs, -1)
    tol = 32 * 2.0 ** (-53 if precision == "fp64" else -24)
    for r in range(nrhs):
        z1 = S1.level_op(-1, "smooth", x[r].contiguous())
        assert not (z[r] * (1 - S1.unknown_mask())).any()
        assert float((z[r] - z1).norm()) <= tol * float(z1.norm()), r
