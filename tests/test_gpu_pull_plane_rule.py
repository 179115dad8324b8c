"""Interface sums of many pairs of 8^3 on either side of the rule that leaves planes of 4 x 4
subdomains to the one-subdomain-per-lane kernel (FP64, 256 pairs).  Checks and bounds as for the
other planes."""
import pytest

import test_gpu_pull_plane as plane

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", [(8, 255), (8, 256), (10, 256)])
def test_either_side(n, nrhs, precision):
    plane.test_smoothing_step(n, nrhs, True, precision)
