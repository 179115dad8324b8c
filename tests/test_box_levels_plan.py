"""Domains of many boxes plan (CPU): a chessboard of 32^3 boxes has more class triples of vertices
with patches on its 128^3 level than the box form of the vertex kernels numbers; the level is
then served by the generic smoother."""
import ctypes

import numpy as np
import pytest

from paper_2205_05840_amd import _lib


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("r,n,levels", [(32, 128, 3), (16, 64, 3), (32, 64, 2)])
def test_chessboard_plans(r, n, levels, precision):
    i = np.arange(r)
    keep = np.ascontiguousarray((i[:, None, None] + i[None, :, None] + i) % 2 == 0, dtype=np.uint8)
    o = _lib.ndmg_default_opts()
    o.precision, o.coef_r = precision, r
    o.domain = keep.ctypes.data_as(ctypes.POINTER(ctypes.c_ubyte))
    ws, vl = _lib.ndmg_plan(n, 1.0, 1.0, o, levels)
    assert ws > 0 and vl == 3 * (n + 1) ** 2 * ((n + 8) // 8 * 8)
