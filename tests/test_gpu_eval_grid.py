"""Divisions of the row evaluation (csrc/eval.hip, eval_rows_grid) where the
workspace's bound on partial sums lets fewer than 256 queries share a workgroup
and more of its waves divide the points; and both sides of the rows' LDS limit
for p = 7 (44 coordinates fit, 45 take the general kernel)."""
import pytest

from paper_0808_0487_amd import inputs
from tests.gpu_common import announce
from tests.test_gpu_eval_rows import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,m,s,nq", [(2, 8, 4, 300), (2, 9, 1, 700), (2, 10, 5, 130), (2, 12, 2, 150), (2, 9, 40, 130),
                                      (3, 6, 3, 200), (3, 7, 3, 140), (3, 8, 1, 300), (3, 8, 2, 120),
                                      (5, 4, 30, 140), (5, 5, 4, 130), (7, 3, 30, 175),
                                      (7, 2, 45, 40), (7, 2, 64, 70), (7, 3, 44, 20)])
def test_against_the_direct_sum(p, m, s, nq):
    announce("eval grid", p, m, s, nq)
    check(p, m, s, nq, inputs.upper_triangular_generators(p, m, s, 100 * p + m + s), m + s + nq)
