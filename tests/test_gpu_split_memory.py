"""Device memory after a split cost: the call works in the net's workspace, so
that a handle which has computed an effective dimension on its points (a larger
workspace) holds no more after it than the tables of the half net."""
import pytest
import torch

from paper_0808_0487_amd import fdwt, inputs
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,s", [(22, 4), (20, 3)])
def test_split_cost_keeps_no_buffers_of_its_own(m, s):
    announce("split memory", m, s)
    net = fdwt.Net(2, m, s, inputs.upper_triangular_generators(2, m, s, 1))
    kern = fdwt.Kernel(2.0, inputs.kernel_weights(s))
    f2 = torch.rand(2 ** m, device="cuda")
    want = net.eff_dim(kern, f2)["var_trc"]
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    cost = net.split_cost(f2, 2.0, 0.5, -2.0)
    net.kernel_tune(f2, (2.0, 0.5, -2.0), 8)
    torch.cuda.synchronize()
    # the half net's tables take less than one 2 MiB page of device memory
    assert free0 - torch.cuda.mem_get_info()[0] <= 2 << 20
    assert (net.eff_dim(kern, f2)["var_trc"] == want).all()
    assert net.split_cost(f2, 2.0, 0.5, -2.0) == cost
    net.close()
