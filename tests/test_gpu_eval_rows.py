"""Interpolant evaluation by table rows (csrc/eval.hip) against the oracle's
direct sum, with arbitrary coefficients: the smallest nets, ragged numbers of
blocks and queries, queries that agree with net points in every digit the
rows see, and nets outside the rows' rule."""
import numpy as np
import pytest
import torch

from oracle import kernel, net as onet
from paper_0808_0487_amd import fdwt, inputs
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


def near_points(p, m, D, X, seed):
    """Queries at net points: exactly, and with the last 1..D - m digits
    changed, so that all digits up to D - 1, D - 2, ... agree."""
    g = np.random.default_rng(seed)
    idx = g.integers(0, X.shape[1], size=12)
    base = kernel.to_depth(p, m, D, X[:, idx]).astype(np.int64)
    for i in range(1, 12):
        base[:, i] += g.integers(0, p ** min(i, D - m), size=X.shape[0])
    return base


def check(p, m, s, nq, C, seed):
    D = inputs.QUERY_DEPTH[p]
    X = onet.net_int(p, m, C)
    g = np.random.default_rng(seed)
    c = g.uniform(-1.0, 1.0, size=p ** m).astype(np.float32)
    Q = np.concatenate([near_points(p, m, D, X, seed), inputs.queries(p, s, nq, seed).astype(np.int64)], axis=1)[:, :nq]
    gam = inputs.kernel_weights(s)
    net = fdwt.Net(p, m, s, C)
    qd = torch.from_numpy(np.ascontiguousarray(Q.astype(np.uint32)).view(np.int32)).cuda()
    sf = net.spline_eval(fdwt.Kernel(2.0, gam), torch.from_numpy(c).cuda(), qd).cpu().numpy().astype(np.float64)
    ref = kernel.spline_eval(p, m, 2.0, gam, X, c.astype(np.float64), Q, D)
    # Every factor (positive: gamma_j <= 1) is rounded to float, s products
    # and at most 64 float additions follow; the pair sums add nothing.
    bound = (2 * s + 66) * 2.0 ** -24 * kernel.spline_eval(p, m, 2.0, gam, X, np.abs(c).astype(np.float64), Q, D)
    assert np.all(np.abs(sf - ref) <= bound)
    net.close()


@pytest.mark.parametrize("p,m,s,nq", [
    (2, 2, 1, 1), (2, 3, 5, 64), (2, 7, 4, 65), (2, 9, 13, 129), (2, 12, 3, 300), (2, 13, 33, 40), (2, 5, 64, 257),
    (3, 1, 1, 3), (3, 2, 4, 66), (3, 4, 9, 128), (3, 7, 14, 70), (3, 8, 2, 300), (3, 3, 64, 20),
    (5, 1, 2, 5), (5, 2, 8, 65), (5, 4, 25, 129), (5, 5, 3, 260), (5, 2, 64, 33),
    (7, 1, 3, 2), (7, 3, 6, 67), (7, 4, 2, 130), (7, 2, 43, 40), (7, 2, 44, 40)])
def test_rows_against_the_direct_sum(p, m, s, nq):
    announce("eval rows", p, m, s, nq)
    check(p, m, s, nq, inputs.upper_triangular_generators(p, m, s, 100 * p + m + s), m + s + nq)


@pytest.mark.parametrize("p,m,s,nq", [(2, 8, 5, 70), (3, 5, 4, 70), (5, 3, 4, 70), (7, 2, 3, 70)])
def test_singular_and_general_generators(p, m, s, nq):
    """Random matrices (the first columns not zero below the leading block),
    with a zero leading block, with non-singular leading blocks, and those
    over zeros (the rows' rule, the other columns still random)."""
    announce("eval general generators", p, m, s, nq)
    C = inputs.random_generators(p, m, s, 7 * p + m)
    check(p, m, s, nq, C, 1)
    C[0, :2, :2] = 0
    check(p, m, s, nq, C, 2)
    C[:, :2, :2] = [[1, 1], [1, 0]]
    check(p, m, s, nq, C, 3)
    C[:, 2:, :2] = 0
    check(p, m, s, nq, C, 4)
    C[:, 1:, 0] = 0
    check(p, m, s, nq, C, 5)
