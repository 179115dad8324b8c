"""Single steps on the caller's stream: apply writes every entry of its output (row padding
included, whatever the buffer held), calls from two streams in turn share the context's
level buffers in order, steps and solves mix, and a step captured into a caller's graph
replays as the eager one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _vec(S, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(S.vec_len, generator=g, dtype=torch.float64, device="cuda") * S.unknown_mask()


@pytest.mark.parametrize("n,coef", [(2, False), (12, False), (40, False), (64, False), (96, False), (128, False),
                                    (16, True), (64, True)])
def test_apply_writes_every_entry(n, coef):
    from paper_2205_05840_amd import Solver
    print(f"[case] n={n} coef={coef}", flush=True)
    S = Solver(n, 1.0, domain=np.array([[[1, 1], [1, 0]], [[1, 1], [1, 1]]], dtype=bool) if coef else None)
    x = _vec(S, n)
    y = torch.full_like(x, float("nan"))
    S.apply(x, y)
    ref = torch.zeros_like(x)
    S.apply(x, ref)
    assert torch.equal(y, ref)
    assert not (y * (1 - S.unknown_mask())).any()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_streams_share_a_context(precision):
    from paper_2205_05840_amd import Solver
    S = Solver(32, 0.5, precision=precision)
    g = [_vec(S, s) for s in range(6)]
    want = [S.vcycle(v).clone() for v in g]
    u_want = S.solve(g[0])[0].clone()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = []
    for i, v in enumerate(g):   # the level buffers pass from stream to stream
        with torch.cuda.stream(streams[i % 2]):
            got.append(S.vcycle(v))
            if i == 2:
                u = S.solve(g[0])[0]
    torch.cuda.synchronize()
    for z, w in zip(got, want):
        assert torch.equal(z, w)
    assert torch.equal(u, u_want)


def test_step_under_capture():
    from paper_2205_05840_amd import Solver
    S = Solver(16, 1.0)
    x, y, z = _vec(S, 1), S.zeros(), S.zeros()
    S.apply(x, y)
    S.vcycle(x, z)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        S.apply(x, y)
        S.vcycle(x, z)
    for seed in (2, 3, 4):
        x.copy_(_vec(S, seed))
        graph.replay()
        torch.cuda.synchronize()
        yr, zr = y.clone(), z.clone()
        assert torch.equal(yr, S.apply(x)) and torch.equal(zr, S.vcycle(x))
        S.solve(x)
        torch.cuda.synchronize()
