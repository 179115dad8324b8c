"""Steps on a stream that was made outside torch and is destroyed after its work: later calls on
other streams, and the end of the context, do not touch it."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_steps_on_a_stream_of_the_caller():
    from paper_2205_05840_amd import Solver
    S = Solver(16, 1.0)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn(S.vec_len, generator=g, dtype=torch.float64, device="cuda") * S.unknown_mask()
    y, z = S.apply(x), S.vcycle(x)
    hip = ctypes.CDLL("libamdhip64.so")
    handle = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0   # hipStreamNonBlocking
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.ExternalStream(handle.value)):
        ye, ze = S.apply(x), S.vcycle(x)
    torch.cuda.synchronize()
    assert hip.hipStreamDestroy(handle) == 0
    assert torch.equal(ye, y) and torch.equal(ze, z)
    assert torch.equal(S.vcycle(x), z)
    S.solve(x)
    S.close()
    torch.cuda.synchronize()
