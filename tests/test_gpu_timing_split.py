"""The launch-timing hook sees the work of a split cost at every size: one
launch (first halves of 2^10..2^14 points) or separate passes."""
import pytest
import torch

from paper_0808_0487_amd import fdwt, inputs
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m2", [9, 11, 13, 15, 16])
def test_split_cost_is_timed(m2):
    announce("split cost timing", m2)
    net = fdwt.Net(2, m2, 3, inputs.upper_triangular_generators(2, m2, 3, 1))
    f2 = torch.rand(2 ** m2, device="cuda")
    net.split_cost(f2, 2.0, 0.5, -2.0)
    fdwt.timing_enable(True)
    try:
        for want_sf in (False, True):
            net.split_cost(f2, 2.0, 0.5, -2.0, want_sf=want_sf)
        ms, n, work = fdwt.timing_query("pass_f64")
    finally:
        fdwt.timing_enable(False)
    # f~ and the second half's values are read in every form
    assert n >= 2 and ms > 0.0 and work >= 2 * 2 ** (m2 - 1) * 8.0
    net.close()
