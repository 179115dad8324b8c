"""The convergence test of CG on either side of its rule (a wavefront per pair up to 16 pairs and
as long as a pair has as many partial sums as there are pairs, else a thread per pair): 14^3
has 43 partial sums per pair, 16^3 with 64 and 65 pairs 64 and 63.  Checks and bounds as for the
other numbers of pairs."""
import pytest

import test_gpu_convergence_check as check

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", [(14, 43), (14, 44), (16, 64), (16, 65), (14, 200)])
def test_either_side(n, nrhs, precision):
    check.test_pairs_stop_on_their_own(n, nrhs, precision)
