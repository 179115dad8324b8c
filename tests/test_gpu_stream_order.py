"""Calls of one context from two streams without any wait of the caller's: the later call finds the
earlier one's result, though a longer computation lies before that on its stream (a missing
wait would find the NaN that filled the buffer).  For one size class and for a batch of several,
whose classes fork from the caller's stream and join it again."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _solver(kind, precision):
    from paper_2205_05840_amd import BatchedSolver, Solver
    if kind == "one":
        S = Solver(32, 0.5, precision=precision)
        return S, S.unknown_mask()
    S = BatchedSolver([8, 20, 32, 14, 20], [0.5, 1.0, 0.2, 0.7, 0.3], nrhs=2, precision=precision)
    ones = torch.ones(S.sample_len(), dtype=torch.float64, device="cuda")
    return S, (S.assemble_rhs(ones) != 0).double()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["one", "batch"])
def test_later_calls_follow(kind, precision):
    S, mask = _solver(kind, precision)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    xs = [torch.randn(mask.numel(), generator=g, dtype=torch.float64, device="cuda") * mask for _ in range(4)]
    want = []
    for x in xs:
        z = S.vcycle(x)
        want.append((z, S.apply(z), S.solve(S.apply(z))[0]))
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    busy = {s: torch.randn(4096, 4096, generator=g, device="cuda") for s in (a, b)}
    work = {s: torch.empty_like(busy[s]) for s in (a, b)}
    zs = [S.zeros() for _ in xs]
    ys = [torch.full_like(x, float("nan")) for x in xs]
    us = [None] * len(xs)
    for z in zs:   # (the V-cycle writes unknowns only)
        z.masked_fill_(mask != 0, float("nan"))
    torch.cuda.synchronize()
    for i, x in enumerate(xs):
        first = a if i % 2 else b
        with torch.cuda.stream(first):
            for _ in range(20):
                torch.mm(busy[first], busy[first], out=work[first])
            S.vcycle(x, zs[i])
        with torch.cuda.stream(b if i % 2 else a):
            S.apply(zs[i], ys[i])
        with torch.cuda.stream(a):
            us[i] = S.solve(ys[i])[0]
    torch.cuda.synchronize()
    for i in range(len(xs)):
        assert torch.equal(zs[i], want[i][0]) and torch.equal(ys[i], want[i][1]) and torch.equal(us[i], want[i][2])
