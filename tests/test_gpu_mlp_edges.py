"""Edges of the one-launch prediction: batch sizes around each workgroup size's
limits and every protocol length (needs an MI355X).  Predictions of 300 rows
(16 protocols per workgroup) and 16,600 (64) are compared with the float64
oracle elsewhere; a protocol's sums do not depend on the batch, so the other
sizes have to agree with those bit for bit."""
import numpy as np
import pytest
import torch

from paper_2303_08123_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gga():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08123_amd as g
    return g


@pytest.mark.parametrize("K", [1, 10, 40, 43])
def test_a_protocol_predicts_the_same_in_every_batch(gga, K):
    net = gga.mlp_net(seed=11)
    most = 16500
    dose, gap, nfrac = workloads.random_protocols(most, K, seed=K, kmin=0)
    dd = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (dose, gap, nfrac)]
    whole = gga.mlp_predict(net, *dd)
    small = torch.cat([gga.mlp_predict(net, *(x[k:k + 300].contiguous() for x in dd)) for k in range(0, most, 300)])
    assert torch.equal(whole, small)
    for B in (1, 15, 16, 17, 31, 33, 63, 65, 4095, 4096, 4097, 4129, 8191, 8192, 8193, 8257):
        assert torch.equal(gga.mlp_predict(net, *(x[:B].contiguous() for x in dd)), whole[:B]), B
