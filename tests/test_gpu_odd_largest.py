"""The odd-p plans beyond those of test_gpu_odd_passes.py: three passes, and
the largest nets, against the fast CPU reference (oracle/fast, float64)."""
import numpy as np
import pytest
import torch

from oracle import fast
from paper_0808_0487_amd import fdwt, inputs
from tests.gpu_common import announce, nrel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,m,dtype,eps", [(3, 15, np.float32, 2.0 ** -24), (3, 15, np.float64, 2.0 ** -53),
                                           (3, 16, np.float32, 2.0 ** -24), (5, 11, np.float32, 2.0 ** -24),
                                           (5, 11, np.float64, 2.0 ** -53), (7, 9, np.float32, 2.0 ** -24),
                                           (7, 9, np.float64, 2.0 ** -53)])
def test_largest_plans(p, m, dtype, eps):
    """Forward of real data, inverse to real and back in place.  A radix-p
    stage (p <= 7) adds at most 8 eps normwise in either precision, the double
    reference as much of its own."""
    announce("odd largest", p, m, np.dtype(dtype).name)
    N = p ** m
    tol = 8 * m * (eps + 2.0 ** -53)
    x = np.random.default_rng(100 * p + m).standard_normal(N).astype(dtype)
    net = fdwt.Net(p, m, 1, inputs.identity_generators(p, m, 1))
    y = net.forward(torch.from_numpy(x).cuda())
    assert nrel(y.cpu().numpy(), fast.fwt(p, m, x.astype(np.float64))) <= tol
    assert nrel(net.inverse(y, real=True).cpu().numpy(), x) <= 3 * tol
    out = net.inverse(y, out=y)  # in place, to complex
    assert out is y and nrel(out.cpu().numpy().real, x) <= 3 * tol
    net.close()
