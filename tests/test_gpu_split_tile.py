"""The split cost in one launch (first halves of 2^10..2^14 points), and the
sizes beside it that run as separate passes, against the cost formula on the
oracle's kernel values with Walsh transforms of the fast CPU reference; one
handle used for several data sets, kernels and streams in turn."""
import numpy as np
import pytest
import torch

from oracle import fast, kernel, net as onet, tuning
from paper_0808_0487_amd import fdwt, inputs
from tests.gpu_common import announce, nrel

pytestmark = pytest.mark.gpu


def reference(m2, C2, f2, alpha, beta, q):
    """Sf at the second half and the cost, in float64."""
    s, N = C2.shape[0], 2 ** (m2 - 1)
    X2 = onet.net_int(2, m2, C2)
    K = kernel.kernel_K(2, alpha, tuning.weights(s, beta, q), m2, X2, np.zeros((s, 1), dtype=X2.dtype)).reshape(-1)
    fwt = lambda v: fast.fwt(2, m2 - 1, v) * N  # noqa: E731  (unnormalised)
    sf = fwt(fwt(f2[:N]) * fwt(K[N:]) / fwt(K[:N])) / N
    return sf, float(np.sum((f2[N:] - sf) ** 2))


@pytest.mark.parametrize("m2,s", [(10, 3), (11, 1), (11, 5), (12, 20), (13, 2), (14, 10), (15, 7), (15, 64), (16, 4)])
def test_split_cost_tiles(m2, s):
    """Sf to 1e-5 normwise (float32 coefficients of the data); the cost to
    1e-5 of the size of f, as its square root."""
    announce("split tile", m2, s)
    C2 = inputs.upper_triangular_generators(2, m2, s, 10 * m2 + s)
    net = fdwt.Net(2, m2, s, C2)
    x = onet.net_points(2, m2, C2)
    N = 2 ** (m2 - 1)
    side = torch.cuda.Stream()
    for i, prm in enumerate([(2.0, 0.5, -2.0), (1.5, 0.3, -1.5), (2.0, 0.5, -2.0)]):
        f2 = np.prod(1.0 + (x - 0.3 - 0.1 * i) / np.arange(1, s + 1)[:, None] ** 2, axis=0).astype(np.float32)
        with torch.cuda.stream(side if i == 1 else torch.cuda.current_stream()):
            cost, sf = net.split_cost(torch.from_numpy(f2).cuda(), *prm, want_sf=True)
        torch.cuda.synchronize()
        ref, rc = reference(m2, C2, f2.astype(np.float64), *prm)
        assert nrel(sf.cpu().numpy(), ref) <= 1e-5
        assert abs(np.sqrt(cost) - np.sqrt(rc)) <= 1e-5 * np.linalg.norm(f2[N:])
    net.close()
