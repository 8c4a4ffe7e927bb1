"""Interpolant evaluation by table rows (csrc/eval.hip) at the largest net of
each prime, where every digit position of the rows' point words is in use:
coefficients on a random set of points, the direct sum over those points."""
import numpy as np
import pytest
import torch

from oracle import kernel
from paper_0808_0487_amd import fdwt, inputs
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


def points(p, m, C, idx):
    """X_{j,n} (m-digit integers) of the points idx."""
    nd = np.stack([(idx // p ** i) % p for i in range(m)])
    X = np.zeros((C.shape[0], idx.size), dtype=np.int64)
    for j in range(C.shape[0]):
        y = (C[j].astype(np.int64) @ nd) % p
        X[j] = (y * p ** np.arange(m - 1, -1, -1, dtype=np.int64)[:, None]).sum(0)
    return X


@pytest.mark.parametrize("p,m,s", [(2, 26, 3), (3, 15, 4), (3, 16, 1), (3, 16, 5), (5, 10, 3), (7, 9, 3)])
def test_largest_nets(p, m, s):
    announce("eval rows largest", p, m, s)
    D, N, k = inputs.QUERY_DEPTH[p], p ** m, 3000
    C = inputs.upper_triangular_generators(p, m, s, 10 * p + m + s)
    g = np.random.default_rng(m + s)
    idx = np.unique(np.concatenate([[0, N - 1], g.integers(0, N, k)]))
    cv = g.uniform(-1.0, 1.0, size=idx.size).astype(np.float32)
    c = torch.zeros(N, dtype=torch.float32, device="cuda")
    c[torch.from_numpy(idx).cuda()] = torch.from_numpy(cv).cuda()
    X = points(p, m, C, idx)
    # Queries at points of the set: the same, then with their last digits
    # changed (all digits up to some depth agree), then anywhere.
    Q = inputs.queries(p, s, 12, m).astype(np.int64)
    near = kernel.to_depth(p, m, D, X[:, g.integers(0, idx.size, 8)]).astype(np.int64)
    for i in range(1, 8):
        low = p ** min(D - 1, D - m + 2 * i - 2)
        near[:, i] += g.integers(0, low, size=s) - near[:, i] % low
    Q[:, :8] = near
    gam = inputs.kernel_weights(s)
    net = fdwt.Net(p, m, s, C)
    qd = torch.from_numpy(np.ascontiguousarray(Q.astype(np.uint32)).view(np.int32)).cuda()
    sf = net.spline_eval(fdwt.Kernel(2.0, gam), c, qd).cpu().numpy().astype(np.float64)
    net.close()
    ref = kernel.spline_eval(p, m, 2.0, gam, X, cv.astype(np.float64), Q, D)
    # Every factor (positive: gamma_j <= 1) is rounded to float, s products
    # and at most 64 float additions follow; the pair sums add nothing.
    bound = (2 * s + 66) * 2.0 ** -24 * kernel.spline_eval(p, m, 2.0, gam, X, np.abs(cv).astype(np.float64), Q, D)
    assert np.all(np.abs(sf - ref) <= bound)
