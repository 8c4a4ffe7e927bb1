"""p = 2 passes whose digits 4 and 5 run between lanes (contiguous tiles: lanes
of a quad; strided tiles: register swaps between rows and halves of a wave),
at the sizes where the tile shapes change."""
import numpy as np
import pytest

from paper_0808_0487_amd import fdwt, inputs
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [10, 13, 14, 15, 17, 18, 19, 22, 23, 24])
@pytest.mark.parametrize("dtype", ["int32", "float32", "float64"])
def test_delta_gives_its_walsh_function(m, dtype):
    """The transform of a delta at n is the Walsh function wal_n, exactly: +-1
    (times p^-m, a power of two, in floating point), and +-inf for an infinite
    delta (its butterflies only add zeros to it)."""
    import torch
    announce("delta", m, dtype)
    N = 2 ** m
    net = fdwt.Net(2, m, 1, inputs.upper_triangular_generators(2, m, 1, 1))
    h = np.arange(N, dtype=np.uint32)
    for n in (1, 16, 32, 48, N // 2 + 33, N - 1):
        par = h & np.uint32(n)
        for k in (16, 8, 4, 2, 1):
            par ^= par >> np.uint32(k)
        sign = 1 - 2 * (par & 1).astype(np.int64)
        x = torch.zeros(N, dtype=getattr(torch, dtype), device="cuda")
        x[n] = 1
        scale = 1.0 if dtype == "int32" else 1.0 / N
        y = net.forward(x).cpu().numpy()
        assert np.array_equal(y, (sign * scale).astype(y.dtype))
        if dtype != "int32":
            x[n] = float("inf")
            y = net.forward(x).cpu().numpy()
            assert np.array_equal(y, np.where(sign > 0, np.inf, -np.inf).astype(y.dtype))
    net.close()
