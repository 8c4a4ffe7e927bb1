"""Calls that return host results wait for their stream (include/fdwt.h): when
they return, nothing is left running on it, and the next call may come on
another stream."""
import numpy as np
import pytest
import torch

from paper_0808_0487_amd import fdwt, inputs
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


def idle_after(call, stream):
    """How often the stream is idle when the call returns, of 100 calls, with
    work of the stream's own before each."""
    w = torch.zeros(1 << 18, device="cuda")
    stream.wait_stream(torch.cuda.current_stream())
    n = 0
    with torch.cuda.stream(stream):
        for _ in range(100):
            w += 1.0
            call()
            n += stream.query()
    torch.cuda.synchronize()
    return n


@pytest.mark.parametrize("side", [False, True])
@pytest.mark.parametrize("p,m,s", [(2, 6, 3), (2, 10, 4), (2, 15, 5), (3, 6, 4), (5, 4, 30)])
def test_eff_dim(p, m, s, side):
    announce("wait eff_dim", p, m, s, side)
    net = fdwt.Net(p, m, s, inputs.upper_triangular_generators(p, m, s, 1))
    kern = fdwt.Kernel(2.0, inputs.kernel_weights(s))
    ft = net.forward(net.sample("product", inputs.family_params("product", s, seed=1)))
    st = torch.cuda.Stream() if side else torch.cuda.current_stream()
    assert idle_after(lambda: net.eff_dim(kern, ft), st) == 100
    net.close()


@pytest.mark.parametrize("m2,s", [(8, 3), (11, 4), (14, 10), (16, 3)])
def test_split_cost(m2, s):
    announce("wait split cost", m2, s)
    net = fdwt.Net(2, m2, s, inputs.upper_triangular_generators(2, m2, s, 1))
    f2 = torch.rand(2 ** m2, device="cuda")
    st = torch.cuda.current_stream()
    assert idle_after(lambda: net.split_cost(f2, 2.0, 0.5, -2.0), st) == 100
    assert idle_after(lambda: net.split_cost(f2, 2.0, 0.5, -2.0, want_sf=True), st) == 100
    net.close()


def test_streams_in_turn():
    """One handle from two streams in turn, every result that of one stream."""
    announce("wait streams in turn")
    p, m, s = 2, 12, 6
    net = fdwt.Net(p, m, s, inputs.upper_triangular_generators(p, m, s, 1))
    kern = fdwt.Kernel(2.0, inputs.kernel_weights(s))
    fts = [net.forward(net.sample("product", inputs.family_params("product", s, seed=i))) for i in range(4)]
    f2 = [torch.rand(2 ** m, device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    want = [(net.eff_dim(kern, ft)["var_trc"], net.split_cost(g, 2.0, 0.5, -2.0)) for ft, g in zip(fts, f2)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for r in range(40):
        with torch.cuda.stream(streams[r % 2]):
            i = r % 4
            v, c = net.eff_dim(kern, fts[i])["var_trc"], net.split_cost(f2[i], 2.0, 0.5, -2.0)
        assert np.array_equal(v, want[i][0]) and c == want[i][1]
    net.close()
