"""The patch products with one 16-vertex group per wave (their own kernel in FP32) against other
launch shapes: V-cycles agree bit for bit (each vertex's product does not depend on its
place), on one pair and in classes of several right-hand sides (edges of the box spread over
right-hand sides), with and without boundary patches, with last groups that are partly filled.
"""
import os

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nrhs,boundary", [(24, 8, True), (28, 6, False), (40, 1, True), (48, 1, False), (64, 3, True)])
def test_one_group_per_wave(n, nrhs, boundary):
    from paper_2205_05840_amd import Solver, _lib
    print(f"[case] n={n} nrhs={nrhs} boundary={boundary}", flush=True)
    L = _lib.lib()
    cls = 0 if nrhs == 1 else 1 if nrhs < 4 else 2
    outs = []
    try:
        for shape in ("1 1", "2 1", "4 3"):
            L.ndmg_tuning_clear()
            _lib.check(L.ndmg_tuning_set(f"patch {n} fp32 0 {cls} {shape}".encode()))
            S = Solver(n, 0.7, precision="fp32", nrhs=nrhs, boundary_patches=boundary)
            g = torch.Generator(device="cuda")
            g.manual_seed(n)
            b = torch.randn(nrhs, S.vec_len, generator=g, dtype=torch.float64, device="cuda") * S.unknown_mask()
            outs.append(S.vcycle(b if nrhs > 1 else b[0].contiguous()).clone())
            S.close()
    finally:
        L.ndmg_tuning_clear()
        if os.path.exists(_lib.TUNING_PATH):
            L.ndmg_tuning_load(_lib.TUNING_PATH.encode())
    assert outs[0].abs().max() > 0
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
